"""The cone root-finders from warm roots that are nearly right, on the CPU: a
step of less than 1e-9 from the previous root says nothing about the error it
leaves when the block's metric spreads over many decades.

SOC and RSOC are compared with the secular equation solved in 128 bits.
Tolerance, relative to ||r||_inf: 16 eps times the spread S of the metric in
the block, since m_j + lambda is a difference of numbers of the metric's
size; and 1e-9, the projections' tolerance against the oracle, for the slot
carried along a converging sequence at spreads up to 1e8.  EXP and POW, from
roots off by up to 1e-9 against the projection from the root itself: 1e-9."""
import pathlib
import shutil
import subprocess

import numpy as np
import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]
EPS = float(np.finfo(float).eps)


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("cone_warm")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text("")
    exe = d / "probe"
    subprocess.run([cxx, "-O2", "-std=gnu++17", "-w", f"-I{d}", f"-I{ROOT / 'paper_2608_09159_amd' / 'csrc'}",
                    str(ROOT / "tests" / "cone_warm_probe.cpp"), "-o", str(exe)], check=True)
    return exe


def _worst(probe, mode, count, spread):
    out = subprocess.run([str(probe), mode, str(count), str(spread)], check=True, capture_output=True, text=True)
    return float(out.stdout)


@pytest.mark.parametrize("spread", [1e2, 1e4, 1e6, 1e8, 1e12])
@pytest.mark.parametrize("kind", ["soc", "rsoc"])
def test_wide_metric_from_a_nearly_right_root(probe, kind, spread):
    assert _worst(probe, kind, 4000, spread) <= 16.0 * EPS * spread


@pytest.mark.parametrize("spread", [1e4, 1e6, 1e8])
@pytest.mark.parametrize("kind", ["soc_path", "rsoc_path"])
def test_slot_along_a_converging_sequence(probe, kind, spread):
    assert _worst(probe, kind, 60, spread) <= 1e-9


@pytest.mark.parametrize("spread", [1e2, 1e6, 1e12])
@pytest.mark.parametrize("kind", ["exp", "pow"])
def test_exp_and_pow_from_a_nearly_right_root(probe, kind, spread):
    assert _worst(probe, kind, 20000, spread) <= 1e-9
