"""The EXP and POW root-finders from warm starts, on the CPU: the root must not
depend on where the search starts.  The slot of a block may hold the root of
another iterate, a value of any size, or none.

Tolerance: that of the projections against the oracle, 1e-9 max(1, ||r||_inf):
cold and warm searches end at the same root, to the resolution of their last
Newton step."""
import pathlib
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]
TOL = 1e-9


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("cone_roots")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text("")
    exe = d / "probe"
    subprocess.run([cxx, "-O2", "-w", f"-I{d}", f"-I{ROOT / 'paper_2608_09159_amd' / 'csrc'}",
                    str(ROOT / "tests" / "cone_roots_probe.cpp"), "-o", str(exe)], check=True)
    return exe


@pytest.mark.parametrize("pow_block", [0, 1])
def test_root_does_not_depend_on_the_start(probe, pow_block):
    out = subprocess.run([str(probe), str(pow_block), "60000"], check=True, capture_output=True, text=True)
    assert float(out.stdout) <= TOL
