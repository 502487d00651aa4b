"""The build's rules and upper tree levels at their edges, step by step against the
oracle: sizes around one chunk and around a level's fanout (with and without
the cost model, whose fanout differs), and systems of several types whose
smaller trees end inside a chunk, so that a level's frontier has gaps.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, radius", [(1024, 0.0), (1025, 0.0), (1025, 3.4), (24 * 1024 + 1, 3.4),
                                       (32 * 1024, 0.0), (32 * 1024 + 1, 0.0)])
def test_chunk_borders(n, radius):
    from test_gpu_parity import _step_parity
    pos, box = W.lj_lattice(n, 0.85, 5)
    cfg = W.Config(pos=pos, box=box, rcut=np.array([[3.0]], np.float32), skin=0.4, name="levels")
    _step_parity(cfg, leaf_size=16, collapse_radius=radius)


@pytest.mark.parametrize("counts, radius", [((1, 3000, 1, 2), 0.0), ((1500, 700, 600, 1300), 0.0),
                                            ((1023, 1, 1024, 2), 2.5), ((5, 2042, 5, 1), 0.0)])
def test_trees_ending_inside_chunks(counts, radius):
    from test_gpu_parity import _step_parity
    rng = np.random.default_rng(sum(counts))
    n = sum(counts)
    types = rng.permutation(np.repeat(np.arange(4, dtype=np.int32), counts))
    pos, box = W.uniform(n, np.full(3, 20.0, np.float32), 17)
    cfg = W.Config(pos=pos, box=box, rcut=np.full((4, 4), 2.0, np.float32), skin=0.4, types=types, name="gaps")
    _step_parity(cfg, leaf_size=7, collapse_radius=radius)


@pytest.mark.parametrize("n", [2, 3, 15, 17, 255, 4097, 8191, 8192, 8193, 11263, 11264, 11265, 12289])
@pytest.mark.parametrize("kind", ["spread", "ties"])
def test_order_and_layout_rules(n, kind):
    # both sides of the lines where keys are sorted by ranks or by radix passes
    # and the emit scans the kept counts itself or not; ties: few distinct keys,
    # the largest among them (all bits set), in four types
    from test_gpu_parity import _step_parity
    rng = np.random.default_rng(n)
    box = np.full(3, 30.0, np.float32)
    if kind == "spread":
        pos, types = W.wrap_f32(rng.uniform(0, 30.0, (n, 3)), box), None
    else:
        corners = np.array([[0, 0, 0], [29.99, 29.99, 29.99], [29.99, 0, 15.0]], np.float32)
        pos, types = corners[rng.integers(0, 3, n)], rng.integers(0, 4, n).astype(np.int32)
    nt = 1 if types is None else 4
    _step_parity(W.Config(pos=np.ascontiguousarray(pos), box=box, rcut=np.ones((nt, nt), np.float32), skin=0.2,
                          types=types, name="order"), leaf_size=16)


@pytest.mark.parametrize("n", [20000, 126 * 4096 + 5, 129 * 4096 - 7])
def test_sort_tile_counts(n):
    # few tiles (their counts summed by the scatter) and more (scanned by a launch)
    from nlist_check import export, require_gpu
    import oracle.tree as T
    import paper_1901_08088_amd as Q
    torch = require_gpu()
    rng = np.random.default_rng(n)
    box = np.full(3, 50.0, np.float32)
    pos = W.wrap_f32(rng.uniform(0, 50.0, (n, 3)) ** 1.5 / 50.0 ** 0.5, box)
    tree = Q.qbvh_build(torch.from_numpy(pos).cuda(), None, box, 1)
    keys = export(tree, "keys", n, torch.int32).view(np.uint32)
    perm = export(tree, "perm", n, torch.int32).view(np.uint32)
    want = T.morton_keys(pos, box)
    order = np.argsort(want, kind="stable")
    assert np.array_equal(perm, order.astype(np.uint32)) and np.array_equal(keys, want[order].astype(np.uint32))
