"""Wavefronts whose queries lie far apart: types with few particles, the vapour
around a droplet, a compact tree far smaller than the box.  Their rows equal the
oracle's, and they do not search what lies between the queries: a list with
such queries takes about the time of one without.
"""
import numpy as np
import pytest

import paper_1901_08088_amd as Q
import workloads as W

from nlist_check import batch_buffers, batch_results, compare_rows, require_gpu, run_nlist

pytestmark = pytest.mark.gpu


def _sparse(n, few, ntypes=2, rho=0.85, seed=61):
    """A fluid with `few` particles each of the further types, anywhere in it."""
    pos, box = W.lj_lattice(n, rho, seed)
    types = np.zeros(n, np.int32)
    which = np.random.default_rng(seed).permutation(n)
    for t in range(1, ntypes):
        types[which[(t - 1) * few:t * few]] = t
    rc = np.full((ntypes, ntypes), 2.6, np.float32)
    rc[-1, -1] = 3.0
    return W.Config(pos=pos, box=box, rcut=rc, skin=0.4, types=types, name=f"{few} of {n}")


def _droplet(n, vapour, rc=2.5, edge=5.0, seed=62):
    """A droplet of density 0.8 in a box `edge` times as wide, a share `vapour` outside it."""
    rng = np.random.default_rng(seed)
    L = edge * (n / 0.8) ** (1.0 / 3.0)
    u = rng.normal(size=(n, 3))
    pos = 0.5 * L + u / np.linalg.norm(u, axis=1, keepdims=True) * (0.75 * n / 0.8 / np.pi) ** (1.0 / 3.0) * \
        rng.uniform(0, 1, (n, 1)) ** (1.0 / 3.0)
    gas = rng.uniform(size=n) < vapour
    pos[gas] = rng.uniform(0, L, (int(gas.sum()), 3))
    box = np.full(3, L, np.float32)
    return W.Config(pos=W.wrap_f32(pos, box), box=box, rcut=np.array([[rc]], np.float32), skin=0.3, name="droplet")


def _compact(n, few, L=100.0, seed=63):
    """`few` particles over a box of edge L, n of a second type in a ball of radius 2 at its corner."""
    rng = np.random.default_rng(seed)
    u = rng.normal(size=(n, 3))
    ball = u / np.linalg.norm(u, axis=1, keepdims=True) * 2.0 * rng.uniform(0, 1, (n, 1)) ** (1.0 / 3.0)
    pos = np.concatenate([rng.uniform(0, L, (few, 3)), np.mod(ball + 0.25, L)])
    types = np.concatenate([np.zeros(few, np.int32), np.ones(n, np.int32)])
    which = rng.permutation(n + few)
    box = np.full(3, L, np.float32)
    return W.Config(pos=W.wrap_f32(pos, box)[which], box=box, rcut=np.array([[5.0, 20.0], [20.0, 0.3]], np.float32),
                    skin=0.0, types=types[which], name="compact")


@pytest.mark.parametrize("qpw", [0, 4, 64])
@pytest.mark.parametrize("n, few, ntypes", [(9000, 1, 2), (9000, 17, 4), (30011, 2, 2), (30011, 15, 2), (30011, 16, 3),
                                            (30011, 60, 2), (30011, 300, 4), (70001, 130, 2)])
def test_sparse_types(n, few, ntypes, qpw):
    cfg = _sparse(n, few, ntypes)
    tree, nbr, cnt, ovf = run_nlist(cfg, max_nbr=256, opts={"queries_per_wave": qpw})
    Q.qbvh_free(tree)
    compare_rows(cfg, nbr, cnt, ovf, 256, method="cells")


@pytest.mark.parametrize("opts", [{}, {"leaf_size": 3, "qbits": 8}, {"queries_per_wave": 16, "block_size": 256}])
@pytest.mark.parametrize("vapour", [0.003, 0.03])
def test_droplets(vapour, opts):
    cfg = _droplet(70001, vapour)
    tree, nbr, cnt, ovf = run_nlist(cfg, max_nbr=256, opts=opts)
    Q.qbvh_free(tree)
    compare_rows(cfg, nbr, cnt, ovf, 256, method="cells")


@pytest.mark.parametrize("few", [40, 900])
def test_compact_tree(few):
    # its bins are far below the rounding of a position in the box
    cfg = _compact(5000, few)
    tree, nbr, cnt, ovf = run_nlist(cfg, max_nbr=5120)
    Q.qbvh_free(tree)
    compare_rows(cfg, nbr, cnt, ovf, 5120, method="brute")


def test_fp64_data():
    for cfg in (_sparse(30011, 60), _droplet(30011, 0.01)):
        cfg = W.as_f64(cfg, seed=64)
        tree, nbr, cnt, ovf = run_nlist(cfg, max_nbr=256)
        Q.qbvh_free(tree)
        compare_rows(cfg, nbr, cnt, ovf, 256)


@pytest.mark.parametrize("qpw", [16, 64])
def test_paper_mode(qpw):
    import test_gpu_paper as P
    for cfg in (_sparse(30011, 60), _compact(3000, 60)):
        width = 512 if cfg.name != "compact" else 4096
        nbr, cnt, ovf = P._paper_rows(cfg, {"queries_per_wave": qpw, "qbits": 10}, max_nbr=width)
        few = np.nonzero(cfg.types == (0 if cfg.name == "compact" else 1))[0]
        P._check(cfg, 10, nbr, cnt, ovf, width, queries=np.concatenate([few, np.arange(0, cfg.n, 101)]))


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_beside_positions_that_are_not_numbers(bad):
    # the root box of the first type, and with a bad position of their own the
    # few, have no bounds
    for mine in (False, True):
        cfg = _sparse(30011, 60)
        few = np.nonzero(cfg.types == 1)[0]
        gone = np.array([few[7] if mine else np.nonzero(cfg.types == 0)[0][7]])
        cfg.pos[gone[0], 1] = bad
        tree, nbr, cnt, ovf = run_nlist(cfg, max_nbr=256)
        Q.qbvh_free(tree)
        rest = np.setdiff1d(np.arange(cfg.n), gone)
        alone = W.Config(pos=cfg.pos[rest], box=cfg.box, rcut=cfg.rcut, skin=cfg.skin, types=cfg.types[rest], name="rest")
        stored = np.arange(256)[None, :] < cnt[rest][:, None]
        assert cnt[gone[0]] == 0 and not np.any(stored & (nbr[rest] == gone[0]))
        rows = np.where(stored, nbr[rest] - (nbr[rest] > gone[0]), -7).astype(np.int32)
        compare_rows(alone, rows, cnt[rest], ovf, 256, method="cells")


def test_batch():
    cfgs = [_sparse(30011, 60), W.lj_fluid(20000, seed=65), _sparse(70001, 130, 3), _droplet(30011, 0.01)]
    systems = batch_buffers(cfgs, max_nbr=256)
    Q.nlist_build_many(systems, dict(leaf_size=16, qbits=16, block_size=64))
    for c, (nbr, cnt, ovf) in zip(cfgs, batch_results(systems, cfgs)):
        compare_rows(c, nbr, cnt, ovf, 256, method="cells")


def _time(cfg):
    """Shortest of ten lists of a built tree, in ms."""
    torch = require_gpu()
    pos = torch.from_numpy(cfg.pos).cuda()
    types = None if cfg.types is None else torch.from_numpy(cfg.types).cuda()
    tree = Q.qbvh_build(pos, types, cfg.box, cfg.ntypes)
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


def test_time_of_scattered_queries():
    # the time of the same particles of one type, and of the droplet without its
    # vapour, where every wavefront's queries lie together.  Searching all that
    # lies between a few dozen queries takes ten times as long at this size.
    n = 1_000_000
    sparse = _sparse(n, 60)
    one = W.Config(pos=sparse.pos, box=sparse.box, rcut=np.array([[2.6]], np.float32), skin=0.4, name="one")
    t = [_time(c) for c in (sparse, one, _droplet(n, 0.01), _droplet(n, 0.0))]
    print(f"[scattered] 60 of 1M {t[0]:.3f} ms, one type {t[1]:.3f} ms; droplet {t[2]:.3f} ms, without vapour "
          f"{t[3]:.3f} ms", flush=True)
    assert t[0] < 3.0 * t[1] and t[2] < 3.0 * t[3]
