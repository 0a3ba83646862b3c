"""Workgroups exchange iterates through buffers in which each one's part begins a
cache line: also where the caller's allocator returns memory that does not."""
import pathlib
import shutil
import subprocess

import numpy as np
import pytest

import paper_2608_09159_amd as G
from instances import synth

ROOT = pathlib.Path(__file__).resolve().parents[1]


def test_start_of_a_ring_buffer(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = tmp_path / "probe"
    subprocess.run([cxx, "-O1", "-std=gnu++17", "-w", f"-I{ROOT / 'include'}", f"-I{ROOT / 'paper_2608_09159_amd' / 'csrc'}",
                    str(ROOT / "tests" / "ring_start_probe.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True)
    assert int(out.stdout) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("offset", [16, 64, 144])
def test_allocator_of_unaligned_memory(offset):
    """Results equal those of hipMalloc'd memory bit for bit."""
    import torch
    held = {}

    @G._ALLOC_FN
    def alloc(size, stream, ctx):
        t = torch.empty(size + 512, dtype=torch.uint8, device="cuda")
        p = (t.data_ptr() + 255) // 256 * 256 + offset
        held[p] = t
        return p

    @G._FREE_FN
    def free(p, stream, ctx):
        held.pop(p)

    for prob in (synth.mixed_cone_scaled(seed=4, scale=0.05), synth.large_sparse_qp(seed=2, n=9_000, m=4_000)):
        kw = dict(max_iter=200)
        ref = G.solve(prob, **kw)
        assert ref["grid_dim"] > 1
        h = G.setup(prob, dev_alloc=alloc, dev_free=free, **kw)
        try:
            runs = [h.solve() for _ in range(3)]
        finally:
            h.free()
        assert not held
        for r in runs:
            np.testing.assert_array_equal(r["x"], ref["x"])
            np.testing.assert_array_equal(r["y"], ref["y"])
