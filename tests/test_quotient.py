"""The resident core divides by the metric and the step sizes through their
reciprocals: the corrected product has the bits of the division."""
import pathlib
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]


def test_quotient_has_the_bits_of_the_division(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text("")
    exe = tmp_path / "probe"
    subprocess.run([cxx, "-O2", "-std=gnu++17", "-w", f"-I{tmp_path}", f"-I{ROOT / 'paper_2608_09159_amd' / 'csrc'}",
                    str(ROOT / "tests" / "quotient_probe.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe), "2000000"], check=True, capture_output=True, text=True)
    assert int(out.stdout) == 0
