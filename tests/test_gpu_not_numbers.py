"""Positions that are not numbers, many and few: whole wavefronts of them, lists in
all modes, and the time of a list that holds some.
"""
import numpy as np
import pytest

import paper_1901_08088_amd as Q
import workloads as W

from nlist_check import batch_buffers, batch_results, compare_rows, require_gpu, run_nlist

pytestmark = pytest.mark.gpu


def _fluid(n, bad, value, ntypes=1, f64=False, seed=81):
    """A fluid in which the particles `bad` have `value` for every coordinate, and the rest of it alone."""
    pos, box = W.lj_lattice(n, 0.6, seed)
    if f64:
        pos, box = pos.astype(np.float64), box.astype(np.float64)
    pos = pos.copy()
    pos[bad] = value
    types = np.random.default_rng(seed).integers(0, ntypes, n).astype(np.int32) if ntypes > 1 else None
    rest = np.setdiff1d(np.arange(n), bad)
    make = lambda k: W.Config(pos=pos[k], box=box, rcut=np.full((ntypes, ntypes), 2.0, np.float32), skin=0.3,
                              types=None if types is None else types[k], name=f"{len(bad)} of {n}")
    return make(np.arange(n)), make(rest), rest


def _check(cfg, alone, rest, nbr, cnt, ovf):
    gone = np.setdiff1d(np.arange(cfg.n), rest)
    assert np.all(cnt[gone] == 0) and np.all(nbr[gone] == -7)
    number = np.full(cfg.n, -1, np.int32)
    number[rest] = np.arange(rest.size, dtype=np.int32)
    stored = np.arange(nbr.shape[1])[None, :] < cnt[rest][:, None]
    rows = np.where(stored, number[np.where(stored, nbr[rest], 0)], -7).astype(np.int32)
    assert not np.any(rows == -1)
    compare_rows(alone, rows, cnt[rest], ovf, nbr.shape[1])


@pytest.mark.parametrize("qpw", [0, 2, 16, 64])
@pytest.mark.parametrize("n, bad, ntypes", [(65, 65, 1), (65, 64, 1), (500, 130, 1), (4001, 700, 1), (4001, 30, 3),
                                            (20001, 1, 2)])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_rows(n, bad, ntypes, qpw, value):
    cfg, alone, rest = _fluid(n, np.random.default_rng(n).choice(n, bad, replace=False), value, ntypes)
    tree, nbr, cnt, ovf = run_nlist(cfg, max_nbr=128, opts={"queries_per_wave": qpw}, fill=-7)
    Q.qbvh_free(tree)
    if rest.size == 0:
        assert np.all(cnt == 0) and ovf == 0
    else:
        _check(cfg, alone, rest, nbr, cnt, ovf)


def test_fp64_data_and_batch():
    bad = np.arange(0, 9000, 60)
    cfg, alone, rest = _fluid(9000, bad, np.nan, f64=True)
    tree, nbr, cnt, ovf = run_nlist(cfg, max_nbr=128, fill=-7)
    Q.qbvh_free(tree)
    _check(cfg, alone, rest, nbr, cnt, ovf)
    made = [_fluid(9000, bad, np.nan), _fluid(70001, np.arange(3, 70001, 900), np.nan, 2)]
    systems = batch_buffers([m[0] for m in made], max_nbr=128, fill=-7)
    Q.nlist_build_many(systems, dict(leaf_size=16, qbits=16, block_size=64))
    for m, (nbr, cnt, ovf) in zip(made, batch_results(systems, [m[0] for m in made])):
        _check(*m, nbr, cnt, ovf)


@pytest.mark.parametrize("qpw", [4, 64])
def test_paper_mode_queries(qpw):
    # (what such a particle's own cell is, and so who lists it, is not defined)
    import test_gpu_paper as P
    cfg, alone, rest = _fluid(3000, np.arange(0, 3000, 40), np.nan)
    nbr, cnt, ovf = P._paper_rows(cfg, {"queries_per_wave": qpw, "qbits": 10})
    assert np.all(cnt[::40] == 0)
    number = np.full(cfg.n, -1, np.int32)
    number[rest] = np.arange(rest.size, dtype=np.int32)
    rows = np.full((rest.size, 512), -7, np.int32)
    keep = [number[nbr[i, :cnt[i]]] for i in rest]
    keep = [k[k >= 0] for k in keep]
    for k, r in enumerate(keep):
        rows[k, :r.size] = r
    P._check(alone, 10, rows, np.array([k.size for k in keep], np.int32), ovf, 512)


def test_time_beside_them():
    # (more than a thousand times as long when such a query searches the whole system)
    torch = require_gpu()
    best = []
    for bad in (np.zeros(0, int), np.arange(7, 20001, 4000)):
        cfg, _, _ = _fluid(20001, bad, np.nan)
        tree = Q.qbvh_build(torch.from_numpy(cfg.pos).cuda(), None, cfg.box, 1)
        nbr = torch.empty((cfg.n, 128), dtype=torch.int32, device="cuda")
        cnt = torch.empty(cfg.n, dtype=torch.int32, device="cuda")
        ovf = torch.empty(1, dtype=torch.int32, device="cuda")
        t = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            Q.nlist_build(tree, cfg.rcut, cfg.skin, 128, nbr, cnt, ovf)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b))
        Q.qbvh_free(tree)
        best.append(min(t))
    print(f"[not numbers] none {best[0]:.3f} ms, 6 of 20001 {best[1]:.3f} ms", flush=True)
    assert best[1] < 4.0 * best[0]
