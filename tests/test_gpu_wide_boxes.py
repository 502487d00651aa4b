"""Clusters far apart in a wide box: wavefronts that span two or more of them take
their queries in parts.  Rows against the oracle, with one to many gaps in a
wavefront, and the time of a list against that of the same clusters close together.
"""
import numpy as np
import pytest

import oracle
import paper_1901_08088_amd as Q
import workloads as W

from nlist_check import batch_buffers, batch_results, compare_rows, require_gpu, run_nlist

pytestmark = pytest.mark.gpu


def _clusters(n, count, L, ntypes=1, rc=2.5, seed=71):
    """n particles in `count` balls of density 0.8 anywhere in a box of edge L."""
    rng = np.random.default_rng(seed)
    u = rng.normal(size=(n, 3))
    ball = u / np.linalg.norm(u, axis=1, keepdims=True) * (0.75 * n / count / 0.8 / np.pi) ** (1.0 / 3.0) * \
        rng.uniform(0, 1, (n, 1)) ** (1.0 / 3.0)
    pos = rng.uniform(0, L, (count, 3))[rng.integers(0, count, n)] + ball
    box = np.full(3, L, np.float32)
    types = rng.integers(0, ntypes, n).astype(np.int32) if ntypes > 1 else None
    r = np.full((ntypes, ntypes), rc, np.float32)
    if ntypes > 1:
        r[0, 1] = r[1, 0] = 0.5 * rc
    return W.Config(pos=W.wrap_f32(pos, box), box=box, rcut=r, skin=0.3, types=types, name=f"{count} clusters L={L:g}")


def _some(n):
    return np.random.default_rng(72).choice(n, 3000, replace=False)


@pytest.mark.parametrize("opts", [{}, {"queries_per_wave": 32, "block_size": 192, "leaf_size": 5}])
@pytest.mark.parametrize("n, count, L, ntypes", [(70001, 40, 3e3, 1), (70001, 40, 3e4, 1), (70001, 3000, 3e4, 1),
                                                 (70001, 30000, 3e4, 1), (90001, 500, 1e4, 3), (66000, 2, 1e6, 2)])
def test_rows(n, count, L, ntypes, opts):
    cfg = _clusters(n, count, L, ntypes)
    tree, nbr, cnt, ovf = run_nlist(cfg, max_nbr=512, opts=opts)
    Q.qbvh_free(tree)
    compare_rows(cfg, nbr, cnt, ovf, 512, queries=_some(n), method="brute")


def test_rows_cut_and_fp64():
    cfg = _clusters(70001, 300, 2e4)
    tree, nbr, cnt, ovf = run_nlist(cfg, max_nbr=37)
    Q.qbvh_free(tree)
    compare_rows(cfg, nbr, cnt, ovf, 37, queries=_some(cfg.n), method="brute")
    cfg = W.as_f64(cfg, seed=73)
    tree, nbr, cnt, ovf = run_nlist(cfg, max_nbr=512)
    Q.qbvh_free(tree)
    compare_rows(cfg, nbr, cnt, ovf, 512, queries=_some(cfg.n), method="brute")


def test_paper_mode():
    # cells of 0.09 of a radius of 1.5 in a box of edge 6000: every row between the
    # exact one and that of a radius larger by the pad and a cell's diagonal
    import test_gpu_paper as P
    cfg = _clusters(70001, 700, 6e3, rc=1.2)
    nbr, cnt, ovf = P._paper_rows(cfg, {"qbits": 16}, max_nbr=512)
    assert ovf == 0
    h = 6e3 / 65535.0
    q = _some(cfg.n)[:800]
    rp, cols = oracle.neighbor_lists(cfg.pos, cfg.box, cfg.rcut, cfg.skin, queries=q, method="brute")
    rp2, cols2 = oracle.neighbor_lists(cfg.pos, cfg.box, cfg.rcut, cfg.skin + (3.0 ** 0.5 + 0.05) * h, queries=q,
                                       method="brute")
    for k, i in enumerate(q):
        got = set(nbr[i, :cnt[i]].tolist())
        assert len(got) == cnt[i]
        assert set(cols[rp[k]:rp[k + 1]].tolist()) <= got <= set(cols2[rp2[k]:rp2[k + 1]].tolist())


def test_batch_of_wide_and_ordinary_boxes():
    # one shape, boxes that change from call to call: ordinary, one wide, ordinary
    opts = dict(leaf_size=16, qbits=16, block_size=64)
    for L in (300.0, 3e4, 300.0, 3e4):
        cfgs = [W.lj_fluid(30000, seed=74), _clusters(40000, 30, L), _clusters(35001, 400, L, 2)]
        systems = batch_buffers(cfgs, max_nbr=512)
        Q.nlist_build_many(systems, opts)
        for c, (nbr, cnt, ovf) in zip(cfgs, batch_results(systems, cfgs)):
            compare_rows(c, nbr, cnt, ovf, 512, queries=_some(c.n), method="brute")


def _time(cfg):
    """Shortest of ten lists of a built tree, in ms."""
    torch = require_gpu()
    tree = Q.qbvh_build(torch.from_numpy(cfg.pos).cuda(), None, cfg.box, 1)
    nbr = torch.empty((cfg.n, 256), dtype=torch.int32, device="cuda")
    cnt = torch.empty(cfg.n, dtype=torch.int32, device="cuda")
    ovf = torch.empty(1, dtype=torch.int32, device="cuda")
    best = np.inf
    for _ in range(10):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        Q.nlist_build(tree, cfg.rcut, cfg.skin, 256, nbr, cnt, ovf)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    Q.qbvh_free(tree)
    return best


def test_time_in_a_wide_box():
    # (ten times as long when a wavefront that spans two clusters leaves all its
    # pairs to the exact test)
    t = [_time(_clusters(200_000, 100, L)) for L in (1e4, 500.0)]
    print(f"[wide] edge 1e4 {t[0]:.3f} ms, 500 {t[1]:.3f} ms", flush=True)
    assert t[0] < 5.0 * t[1]
