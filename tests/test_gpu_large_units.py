"""Boxes in very small units (edges up to 1e17, and down to 1e-17): the same system
scaled, its rows against the oracle's and its time against that of edge 100.
"""
import numpy as np
import pytest

import paper_1901_08088_amd as Q
import workloads as W

from nlist_check import compare_rows, require_gpu, run_nlist

pytestmark = pytest.mark.gpu


def _scaled(n, L):
    rng = np.random.default_rng(101)
    box = np.full(3, L, np.float32)
    return W.Config(pos=W.wrap_f32(rng.uniform(0, 1, (n, 3)) * L, box), box=box, rcut=np.array([[0.08 * L]], np.float32),
                    skin=0.0, name=f"L={L:g}")


@pytest.mark.parametrize("qpw", [1, 16, 64])
@pytest.mark.parametrize("L", [1e-17, 1e-6, 2e13, 9e13, 1.1e14, 9e16, 1.1e17])
def test_rows(L, qpw):
    cfg = _scaled(3001, L)
    tree, nbr, cnt, ovf = run_nlist(cfg, max_nbr=64, opts={"queries_per_wave": qpw})
    Q.qbvh_free(tree)
    compare_rows(cfg, nbr, cnt, ovf, 64)


def test_time():
    # (six times as long when all pairs go to the exact test)
    torch = require_gpu()
    best = []
    for L in (100.0, 1e15):
        cfg = _scaled(200_000, L)
        tree = Q.qbvh_build(torch.from_numpy(cfg.pos).cuda(), None, cfg.box, 1)
        cnt = torch.empty(cfg.n, dtype=torch.int32, device="cuda")
        ovf = torch.empty(1, dtype=torch.int32, device="cuda")
        t = []
        for _ in range(10):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            Q.nlist_build(tree, cfg.rcut, cfg.skin, 0, None, cnt, ovf)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b))
        Q.qbvh_free(tree)
        best.append(min(t))
    print(f"[units] edge 100 {best[0]:.3f} ms, 1e15 {best[1]:.3f} ms", flush=True)
    assert best[1] < 1.5 * best[0]
