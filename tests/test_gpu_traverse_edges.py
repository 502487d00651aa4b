"""Edges of the traversal, row by row against the oracle: ragged wavefronts at
every queries-per-wavefront setting, runs and batches that fill exactly or
overflow (coincident particles: every slot of a batch accepted, more waiting
words than a wavefront keeps), exact ties (pairs that only the fp64 arithmetic
decides, several per part), spreads that widen the matrix-core band until it
covers most pairs, and coordinates whose squares would overflow in fp32.
"""
import numpy as np
import pytest

import workloads as W

from nlist_check import compare_rows, run_nlist

pytestmark = pytest.mark.gpu


def _config(pos, L, rc, skin=0.0, types=None, name="edge"):
    box = np.full(3, L, np.float32)
    rc = np.atleast_2d(np.asarray(rc, np.float32))
    return W.Config(pos=W.wrap_f32(np.asarray(pos, np.float64), box), box=box, rcut=rc, skin=skin, types=types,
                    name=name)


@pytest.mark.parametrize("qpw", [0, 1, 2, 16, 32, 64])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 63, 64, 65, 129, 1000])
def test_ragged_wavefronts(n, qpw):
    rng = np.random.default_rng(1000 + n)
    cfg = _config(rng.uniform(0, 8.0, (n, 3)), 8.0, 2.5, 0.4)
    _, nbr, cnt, ovf = run_nlist(cfg, max_nbr=256, opts={"queries_per_wave": qpw})
    compare_rows(cfg, nbr, cnt, ovf, 256)


@pytest.mark.parametrize("leaf", [1, 8, 11, 16])
@pytest.mark.parametrize("m", [17, 64, 300])
def test_coincident_particles(m, leaf):
    rng = np.random.default_rng(7 + m)
    pos = np.concatenate([np.full((m, 3), 5.125), rng.uniform(0, 12.0, (500, 3)), np.full((m, 3), 11.999)])
    cfg = _config(pos[rng.permutation(len(pos))], 12.0, 1.5)
    for width in (512, 96, 30, 0):  # rows that fit, that end on and off a 16-byte store, none
        _, nbr, cnt, ovf = run_nlist(cfg, max_nbr=width, opts={"leaf_size": leaf})
        compare_rows(cfg, nbr, cnt, ovf, width)


@pytest.mark.parametrize("opts", [{}, {"queries_per_wave": 64}, {"leaf_size": 5, "block_size": 256}])
@pytest.mark.parametrize("side, r", [(8, 3.0), (13, 5.0)])
def test_exact_ties(side, r, opts):
    # integer lattice: the shells at distance r (and every other one) are met exactly
    g = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3).astype(np.float64)
    g = g[np.random.default_rng(3).permutation(len(g))]
    cfg = _config(g, float(side), r)
    _, nbr, cnt, ovf = run_nlist(cfg, max_nbr=768, opts=opts)
    compare_rows(cfg, nbr, cnt, ovf, 768)


@pytest.mark.parametrize("L, r", [(3000.0, 1.0), (1e5, 2.0), (1e15, 1e13)])
def test_wide_spreads(L, r):
    # pairs near the cutoff whose wavefront spans the box
    rng = np.random.default_rng(11)
    base = rng.uniform(0, L, (700, 3))
    u = rng.normal(size=base.shape)
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    pos = np.concatenate([base, base + u * r * rng.uniform(0.9, 1.1, (700, 1)), base[:200]])
    types = rng.integers(0, 2, len(pos)).astype(np.int32)
    for qpw in (4, 64):
        cfg = _config(pos, L, r)
        _, nbr, cnt, ovf = run_nlist(cfg, max_nbr=64, opts={"queries_per_wave": qpw})
        compare_rows(cfg, nbr, cnt, ovf, 64)
        two = _config(pos, L, [[r, 0.5 * r], [0.5 * r, 0.0]], types=types)
        _, nbr, cnt, ovf = run_nlist(two, max_nbr=64, opts={"queries_per_wave": qpw})
        compare_rows(two, nbr, cnt, ovf, 64)


@pytest.mark.parametrize("n, qpw, edges, r, qbits", [
    (1, 0, (8, 8, 8), 2.5, 10), (17, 16, (8, 8, 8), 2.5, 8), (65, 64, (10, 10, 40), 1.0, 8),
    (700, 64, (10, 10, 40), 0.3, 8), (1500, 0, (40, 9, 12), 0.05, 8), (900, 32, (12, 12, 12), 3.0, 16),
])
def test_paper_mode(n, qpw, edges, r, qbits):
    # cells from far below the radius to three times it: few or all pairs fall
    # between "surely within R" and "surely beyond the cell's diagonal"
    import test_gpu_paper as P
    rng = np.random.default_rng(n)
    box = np.asarray(edges, np.float32)
    cfg = W.Config(pos=W.wrap_f32(rng.uniform(0, 1, (n, 3)) * box.astype(np.float64), box), box=box,
                   rcut=np.array([[r]], np.float32), skin=0.0, name="paper_edge")
    nbr, cnt, ovf = P._paper_rows(cfg, {"queries_per_wave": qpw, "qbits": qbits, "leaf_size": 7})
    P._check(cfg, qbits, nbr, cnt, ovf, 512)


@pytest.mark.parametrize("flat", [1.0, 0.5, 0.0])
@pytest.mark.parametrize("qpw", [8, 64])
def test_paper_mode_flat_cells(flat, qpw):
    # unit bins and a share of particles exactly on them: their cells have no
    # width, so that only the list radius itself is a sure accept
    import test_gpu_paper as P
    rng = np.random.default_rng(21)
    pos = rng.uniform(0, 255.0, (3000, 3))
    pos = np.where(rng.uniform(size=(3000, 1)) < flat, np.round(pos), pos)
    pos[0], pos[1] = 0.0, 255.0
    cfg = _config(pos, 260.0, 20.0)
    nbr, cnt, ovf = P._paper_rows(cfg, {"queries_per_wave": qpw, "qbits": 8})
    P._check(cfg, 8, nbr, cnt, ovf, 512)


@pytest.mark.parametrize("sizes", [(1, 300, 17), (700, 65, 1500), (4000, 129, 2500), (12000, 9000, 5000)])
def test_small_batches(sizes):
    # batches small enough for 1, 2, 4 and 16 queries per wavefront
    from nlist_check import batch_buffers
    import paper_1901_08088_amd as Q
    import torch
    rng = np.random.default_rng(sum(sizes))
    cfgs = []
    for n in sizes:
        L = max(8.0, (n / 0.6) ** (1.0 / 3.0))
        cfgs.append(_config(rng.uniform(0, L, (n, 3)), L, 2.2, 0.3))
    bufs = batch_buffers(cfgs, max_nbr=128)
    Q.nlist_build_many(bufs)
    torch.cuda.synchronize()
    for cfg, b in zip(cfgs, bufs):
        compare_rows(cfg, b["nbr"].cpu().numpy(), b["count"].cpu().numpy(), int(b["overflow"].item()), 128)
