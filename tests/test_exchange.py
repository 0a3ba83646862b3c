"""The grid's all-reduce when a wait ends by its limit, on the CPU: a sum that
lacks a partial is never stored as a total, so a workgroup that arrives late
leaves the kernel as well; and a launch with a raised abort word counts as
aborted whatever status workgroup 0 stored."""
import pathlib
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("exchange")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text("")
    exe = d / "probe"
    subprocess.run([cxx, "-O1", "-std=gnu++17", "-w", f"-I{d}", f"-I{ROOT / 'include'}",
                    f"-I{ROOT / 'paper_2608_09159_amd' / 'csrc'}", str(ROOT / "tests" / "exchange_probe.cpp"),
                    "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60)
    return [[float(x) for x in line.split()] for line in out.stdout.splitlines()]


def test_all_arrive(lines):
    assert lines[0] == [1, 1, 7.0, 0, 1]


@pytest.mark.parametrize("scenario", [1, 2])
def test_late_workgroup_leaves_too(lines, scenario):
    zero, late, _, abort, stored = lines[scenario]
    assert (zero, late, abort, stored) == (0, 0, 1, 0)


def test_raised_abort_word_decides(lines):
    assert lines[3] == [1, 1]
