"""Trees that cannot tell their particles apart: positions that all fall in one
Morton bin (outside the box, which the library does not ask to be checked), where
neither boxes nor spheres around a wavefront's queries leave much out.
"""
import numpy as np
import pytest

import paper_1901_08088_amd as Q
import workloads as W

from nlist_check import compare_rows, require_gpu, run_nlist

pytestmark = pytest.mark.gpu


def _outside(n, rho=0.3, seed=91):
    """An ideal gas from -L/2 to L/2: an eighth of it has its own bins."""
    pos, box = W.uniform(n, np.full(3, (n / rho) ** (1.0 / 3.0)), seed)
    return W.Config(pos=(pos - 0.5 * box).astype(np.float32), box=box, rcut=np.array([[2.5]], np.float32), skin=0.3,
                    name="outside")


@pytest.mark.parametrize("opts", [{}, {"queries_per_wave": 16}, {"leaf_size": 2, "qbits": 8}])
@pytest.mark.parametrize("n", [9000, 70001])
def test_rows(n, opts):
    cfg = _outside(n)
    tree, nbr, cnt, ovf = run_nlist(cfg, max_nbr=128, opts=opts)
    Q.qbvh_free(tree)
    q = np.random.default_rng(92).choice(n, 3000, replace=False)
    compare_rows(cfg, nbr, cnt, ovf, 128, queries=q, method="brute")


def test_time():
    # every wavefront tests a sizeable part of the system, which takes about 70
    # times as long as the same gas inside the box; 350 times when each node is
    # compared with every query to no avail
    torch = require_gpu()
    cfg = _outside(500_000)
    best = []
    for pos in (cfg.pos, np.mod(cfg.pos, cfg.box).astype(np.float32)):
        tree = Q.qbvh_build(torch.from_numpy(pos).cuda(), None, cfg.box, 1)
        nbr = torch.empty((cfg.n, 128), dtype=torch.int32, device="cuda")
        cnt = torch.empty(cfg.n, dtype=torch.int32, device="cuda")
        ovf = torch.empty(1, dtype=torch.int32, device="cuda")
        t = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            Q.nlist_build(tree, cfg.rcut, cfg.skin, 128, nbr, cnt, ovf)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b))
        Q.qbvh_free(tree)
        best.append(min(t))
    print(f"[one bin] outside {best[0]:.3f} ms, inside {best[1]:.3f} ms", flush=True)
    assert best[0] < 150.0 * best[1]
