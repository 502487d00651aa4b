"""The tree build's upper levels at their edges, step by step against the
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
