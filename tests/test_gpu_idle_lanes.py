"""Wavefronts with idle lanes whose pairs all go to the exact test: coordinates
so large that the products say nothing, and positions that are not numbers.  An
idle lane stands beside its wavefront's last query and shares that query's row,
so every row is compared to its end: the entries with the oracle's, the slots
past them with what was there before the call.
"""
import numpy as np
import pytest

import paper_1901_08088_amd as Q
import workloads as W

from nlist_check import compare_rows, run_nlist

pytestmark = pytest.mark.gpu

FILL = -7


def _untouched(nbr, cnt):
    past = np.arange(nbr.shape[1])[None, :] >= cnt[:, None]
    bad = np.nonzero((past & (nbr != FILL)).any(axis=1))[0]
    assert bad.size == 0, f"{bad.size} rows written past their entries, first {bad[:5].tolist()}"


def _spread(n, L, r, seed):
    """Particles over a box of edge L, half of them near the distance r of another."""
    rng = np.random.default_rng(seed)
    base = rng.uniform(0, L, ((n + 1) // 2, 3))
    u = rng.normal(size=base.shape)
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    pos = np.concatenate([base, base + u * r * rng.uniform(0.9, 1.1, (len(base), 1))])[:n]
    return pos[rng.permutation(n)]


@pytest.mark.parametrize("qpw", [4, 16, 64])
@pytest.mark.parametrize("n", [1001, 1602])
@pytest.mark.parametrize("L", [1e15, 1e16, 1e17, 1e19])
def test_huge_boxes(L, n, qpw):
    r = 0.01 * L
    box = np.full(3, L, np.float32)
    pos = W.wrap_f32(_spread(n, L, r, 31), box)
    types = np.random.default_rng(32).integers(0, 3, n).astype(np.int32)
    for rc, ty in (([[r]], None), ([[r, 0.5 * r, r], [0.5 * r, 0.0, r], [r, r, 0.7 * r]], types)):
        cfg = W.Config(pos=pos, box=box, rcut=np.array(rc, np.float32), skin=0.0, types=ty, name="huge")
        tree, nbr, cnt, ovf = run_nlist(cfg, max_nbr=64, opts={"queries_per_wave": qpw}, fill=FILL)
        Q.qbvh_free(tree)
        compare_rows(cfg, nbr, cnt, ovf, 64)
        _untouched(nbr, cnt)


@pytest.mark.parametrize("qpw", [8, 64])
@pytest.mark.parametrize("n", [301, 602])
def test_huge_boxes_paper_mode(n, qpw):
    import test_gpu_paper as P
    L = 1e17
    box = np.full(3, L, np.float32)
    cfg = W.Config(pos=W.wrap_f32(_spread(n, L, 0.1 * L, 41), box), box=box, rcut=np.array([[0.1 * L]], np.float32),
                   skin=0.0, name="huge_paper")
    nbr, cnt, ovf = P._paper_rows(cfg, {"queries_per_wave": qpw, "qbits": 10})
    P._check(cfg, 10, nbr, cnt, ovf, 512)
    _untouched(nbr, cnt)


def _nan(sign):
    return np.array([0x7FC00000 if sign > 0 else 0xFFC00000], np.uint32).view(np.float32)[0]


@pytest.mark.parametrize("bad", [_nan(1), _nan(-1), np.float32(np.inf), np.float32(-np.inf)],
                         ids=["nan", "-nan", "inf", "-inf"])
@pytest.mark.parametrize("qpw", [1, 4, 16, 32, 64])
@pytest.mark.parametrize("axes, ntypes", [((0,), 1), ((0, 1, 2), 1), ((0,), 3), ((1, 2), 3)])
def test_positions_that_are_not_numbers(axes, ntypes, qpw, bad):
    # listed by nobody, list nobody, and every other row is that of the rest
    # alone.  The rest keeps out of the last corner of the box, so that the bad
    # positions of the first case, numbers there on their other axes, come
    # last in Z order: beside them the last wavefront's idle lanes
    rng = np.random.default_rng(51)
    n, L = 1001, 12.0
    box = np.full(3, L, np.float32)
    pos = W.wrap_f32(rng.uniform(0, 0.8 * L, (n, 3)), box)
    types = rng.integers(0, ntypes, n).astype(np.int32) if ntypes > 1 else None
    rc = np.full((ntypes, ntypes), 1.6, np.float32)
    if ntypes > 1:
        rc[0, 1] = rc[1, 0] = 0.0
    gone = rng.choice(n, 9, replace=False)
    pos[gone] = np.float32(0.95 * L)
    for d in axes:
        pos[gone, d] = bad
    rest = np.setdiff1d(np.arange(n), gone)
    cfg = W.Config(pos=pos, box=box, rcut=rc, skin=0.2, types=types, name="bad")
    tree, nbr, cnt, ovf = run_nlist(cfg, max_nbr=128, opts={"queries_per_wave": qpw}, fill=FILL)
    Q.qbvh_free(tree)
    assert np.all(cnt[gone] == 0)
    _untouched(nbr, cnt)
    # the rest in its own numbering
    number = np.full(n, -1, np.int32)
    number[rest] = np.arange(rest.size, dtype=np.int32)
    stored = np.arange(128)[None, :] < np.minimum(cnt[rest], 128)[:, None]
    rows = np.where(stored, number[np.where(stored, nbr[rest], 0)], FILL)
    assert not np.any(rows == -1), "a position that is not a number is listed"
    alone = W.Config(pos=pos[rest], box=box, rcut=rc, skin=0.2, types=None if types is None else types[rest],
                     name="rest")
    compare_rows(alone, rows.astype(np.int32), cnt[rest], ovf, 128)
