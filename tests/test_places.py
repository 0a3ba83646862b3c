"""Solver launches from several threads on one device: they are let in together
only where all their workgroups are resident."""
import pathlib
import shutil
import subprocess
import threading

import numpy as np
import pytest

import paper_2608_09159_amd as G
from instances import synth

ROOT = pathlib.Path(__file__).resolve().parents[1]


def test_never_more_than_is_resident(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = tmp_path / "probe"
    subprocess.run([cxx, "-O1", "-std=c++17", "-pthread", f"-I{ROOT / 'paper_2608_09159_amd' / 'csrc'}",
                    str(ROOT / "tests" / "places_probe.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=120)
    assert out.stdout.split() == ["0", "1800", "1", "1"]


@pytest.mark.gpu
def test_solves_on_two_streams():
    """Two threads with a handle and a stream each: 176 workgroups of the
    register-resident core, one a CU, and a general grid; every result is that
    of a solve by itself."""
    import torch
    probs = [synth.large_sparse_qp(seed=1, n=60_000, m=30_000), synth.large_sparse_qp(seed=2, n=55_000, m=28_000)]
    kw = dict(max_iter=600, host_poll=64)
    alone = [G.solve(p, **kw) for p in probs]
    assert sum(a["grid_dim"] for a in alone) > 256
    streams = [torch.cuda.Stream() for _ in probs]
    handles = [G.setup(p, stream=s, **kw) for p, s in zip(probs, streams)]
    got = [[], []]
    start = threading.Barrier(2)

    def work(k):
        start.wait()
        for _ in range(6):
            got[k].append(handles[k].solve())

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for h in handles:
        h.free()
    for runs, a in zip(got, alone):
        assert len(runs) == 6
        for r in runs:
            assert r["status"] == a["status"] and r["iterations"] == a["iterations"]
            np.testing.assert_array_equal(r["x"], a["x"])
