"""CPU checks of the HiF4 GEMM: its LDS stage protocol for every configuration (the kernel's own
geometry, paper_2607_26515_amd/csrc/gemm_hif4_geo.h, compiled for the host; planted mistakes
must be reported), and the exactness of its operand encodings (device_fp4.h): every activation
magnitude V = k (4+m) 2^(2-b) is 32 hi + 2 lo with the table's E2M3 and E2M1 codes, and every
weight magnitude k 2^-b is its E2M3 code's value."""
import os
import re
import subprocess

import pytest

from oracle.formats import E2M1_MAGNITUDES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_26515_amd", "csrc")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("hif4") / "hif4_protocol_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC,
                        os.path.join(ROOT, "tests", "hif4_protocol_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def test_every_configuration_keeps_the_protocol(checker):
    r = subprocess.run([checker], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:]
    assert "12 configurations, 0 errors" in r.stdout


@pytest.mark.parametrize("plant,what", [(1, "complete"), (2, "before every wave is done reading"),
                                        (3, "written by 2 copies")])
def test_planted_mistakes_are_reported(checker, plant, what):
    r = subprocess.run([checker, str(plant)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 1
    assert what in r.stdout


def _e2m3(code):
    e, m = code >> 3, code & 7
    return m / 8 if e == 0 else 2.0 ** (e - 1) * (1 + m / 8)


def _bytes(lo, hi):
    return list(int(lo, 16).to_bytes(4, "little") + int(hi, 16).to_bytes(4, "little"))


def test_operand_encodings_are_exact():
    src = open(os.path.join(CSRC, "device_fp4.h")).read()
    tab = src[src.index("kHiSplitTab[kHiSplitEntries]"):]
    rows = re.findall(r"\{(0x\w+)u, (0x\w+)u, (0x\w+)u, (0x\w+)u\}", tab)
    assert len(rows) == 12
    for m in range(4):
        for b in range(3):
            r = rows[3 * m + b]
            hi, lo = _bytes(r[0], r[1]), _bytes(r[2], r[3])
            for k in range(8):
                assert hi[k] < 32 and lo[k] < 8
                assert 32 * _e2m3(hi[k]) + 2 * E2M1_MAGNITUDES[lo[k]] == k * (4 + m) * 2 ** (2 - b), (m, b, k)
    weight = re.findall(r"b == 0u \? (0x\w+)u : b == 1u \? (0x\w+)u : (0x\w+)u;", src)
    assert len(weight) == 2  # codes of k = 0..3, then 4..7
    for b in range(3):
        codes = _bytes(weight[0][b], weight[1][b])
        assert [_e2m3(c) for c in codes] == [k * 2.0 ** -b for k in range(8)], b
