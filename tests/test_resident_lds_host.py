"""LDS layout of a resident share (csrc/resident_plan.h) on the CPU: the arrays that the
kernel reads in pairs begin on 16-byte boundaries whatever the number of halo units, and no
array reaches into the next."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1401_1112_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("lds") / "lds_dump")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC,
                    os.path.join(ROOT, "tests", "host", "resident_lds_dump.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("cap", [1024, 5120, 8192])
@pytest.mark.parametrize("held", [0, 1])
@pytest.mark.parametrize("coarse", [0, 1, 3, 6])
def test_layout(harness, cap, held, coarse):
    for units in (0, 1, 2, 3, 4, 5, 6, 7, 333, 1022):
        run = subprocess.run([harness, str(cap), str(units), str(coarse), str(held)], check=True, capture_output=True,
                             text=True)
        p, rh, ex, diag, fine, partner, size = map(int, run.stdout.split())
        sizes = [(p, cap + 4 * units), (rh, 4 * units), (ex, 4 * units), (diag, cap if held else 0), (fine, 4 * coarse)]
        end = 0
        for at, n in sizes:
            assert at % 2 == 0 and at >= end, (units, at)
            end = at + n
        assert partner >= end and size >= 8 * partner + 4 * units
        assert size <= 8 * (2 * cap + 12 * units + 4 * coarse) + 4 * units + 8  # nothing wasted
