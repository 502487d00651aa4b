"""Systems without particles: the traversal's query mapping on the CPU
(csrc/launch_geometry.h, compiled with g++), and batches that hold an empty
system of several types where an earlier batch of the same stream had
particles."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_empty_system_mapping(tmp_path):
    exe = tmp_path / "empty_system_test"
    src = os.path.join(HERE, "empty_system_test.cpp")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror", src, "-o", str(exe)], check=True)
    proc = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert proc.returncode == 0, proc.stdout + proc.stderr
    assert "all checks passed" in proc.stdout


def _system(n, ntypes, seed):
    pos, box = W.uniform(n, [14.0, 14.0, 14.0], seed=seed)
    types = np.random.default_rng(seed).integers(0, ntypes, n).astype(np.int32) if ntypes > 1 else None
    return W.Config(pos=pos.reshape(-1, 3), box=box, rcut=np.full((ntypes, ntypes), 1.5, np.float32), skin=0.3,
                    types=types, name=f"{ntypes} types N={n}")


@pytest.mark.gpu
@pytest.mark.parametrize("eager", [0, 1])
@pytest.mark.parametrize("ntypes", [2, 4])
def test_empty_system_where_particles_were(ntypes, eager):
    import paper_1901_08088_amd as Q
    from nlist_check import batch_buffers, batch_results, compare_rows, require_gpu
    torch = require_gpu()
    opts = dict(leaf_size=8, qbits=16, block_size=64, eager=eager)
    stream = torch.cuda.Stream()
    # (sizes of the systems: the second loses its particles behind a larger
    # first one, then all do, then they come back)
    with torch.cuda.stream(stream):
        for sizes in ((100, 500, 300), (5000, 0, 300), (0, 0, 0), (100, 500, 300), (200, 0, 0)):
            cfgs = [_system(n, 1 if k == 0 else ntypes, 10 * k + n) for k, n in enumerate(sizes)]
            systems = batch_buffers(cfgs, max_nbr=64)
            print(f"[batch] sizes {sizes}", flush=True)
            Q.nlist_build_many(systems, opts)
            for c, s, (nbr, cnt, ovf) in zip(cfgs, systems, batch_results(systems, cfgs)):
                if c.n == 0:
                    assert ovf == 0
                    assert torch.all(s["nbr"] == -7) and torch.all(s["count"] == -1)
                else:
                    compare_rows(c, nbr, cnt, ovf, 64)
    Q.nlist_batch_release(stream)
