"""CPU check of the HiF4 quantizers' element arithmetic: device_fp4.h itself, compiled for the host
(tests/host), against the comparison with every rounding midpoint, the level-1 thresholds, and
zeros, infinities and NaN; mistakes planted in the reference must be reported."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("hif4") / "hif4_round_check")
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wno-unknown-pragmas", "-I", os.path.join(ROOT, "tests", "host"),
                        "-I", os.path.join(ROOT, "paper_2607_26515_amd", "csrc"),
                        os.path.join(ROOT, "tests", "hif4_round_check.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def test_every_midpoint_threshold_and_special_value(checker):
    r = subprocess.run([checker], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:]
    assert r.stdout.strip().endswith(" 0 errors")


@pytest.mark.parametrize("plant,what", [(1, "round"), (2, "c1 at its threshold")])
def test_planted_mistakes_are_reported(checker, plant, what):
    r = subprocess.run([checker, str(plant)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 1
    assert f"FAIL {what}" in r.stdout
