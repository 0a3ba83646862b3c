"""POW: membership (of the cone and of its dual) within a few ulps of the boundary, at
coordinates from 1e-80 to 1e80, on the CPU.  A comparison of powers is right
beyond 4 ulps (two powers and their product); one of logarithms alone only beyond
as many ulps as the logarithms are large."""
import pathlib
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]


def test_sides_of_the_boundary(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text("")
    exe = tmp_path / "probe"
    subprocess.run([cxx, "-O2", "-std=gnu++17", "-w", f"-I{tmp_path}", f"-I{ROOT / 'paper_2608_09159_amd' / 'csrc'}",
                    str(ROOT / "tests" / "cone_member_probe.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe), "100000"], check=True, capture_output=True, text=True)
    assert int(out.stdout) == 0
