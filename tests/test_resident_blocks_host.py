"""Blocks of a resident launch (csrc/resident_plan.cpp) on the CPU: at least one per share
and at most one per compute unit, also where the units are no multiple of the eight XCDs
(the plan deals the shares to that many blocks), and as few XCDs as hold the shares."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1401_1112_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("blocks") / "blocks_dump")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-I", CSRC,
                    os.path.join(ROOT, "tests", "host", "res_blocks_dump.cpp"),
                    os.path.join(CSRC, "resident_plan.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("n_cu", [1, 3, 8, 12, 20, 32, 60, 64, 76, 110, 128, 255, 256, 304])
def test_blocks(harness, n_cu):
    out = subprocess.run([harness, str(n_cu)], check=True, capture_output=True, text=True).stdout.split()
    for g, b in enumerate(map(int, out), 1):
        assert g <= b <= n_cu, (g, b)
        if n_cu == 256 and 1 < g <= 32:
            assert b == 8 * g  # one XCD's blocks of a round-robin over eight
