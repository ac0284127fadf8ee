"""The plan of the resident CG (csrc/resident_plan.cpp) made by several threads is the one
that a single thread makes, table by table; plain and with ThreadSanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1401_1112_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module", params=["plain", "tsan"])
def harness(request, tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / f"threads_{request.param}")
    extra = ["-g", "-fsanitize=thread"] if request.param == "tsan" else []
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread"] + extra + ["-I", CSRC,
                    os.path.join(ROOT, "tests", "host", "resident_plan_threads.cpp"),
                    os.path.join(CSRC, "resident_plan.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("threads", [2, 3, 8])
@pytest.mark.parametrize("n_blocks,target,boxes", [(1, 512, [1]), (16, 512, [12]), (256, 512, [20, 7, 3, 1]),
                                                   (8, 2048, [9] * 12), (256, 5120, [32, 2])])
def test_threads_make_the_same_plan(harness, threads, n_blocks, target, boxes):
    run = subprocess.run([harness, str(threads), str(n_blocks), str(target)] + [str(m) for m in boxes],
                         capture_output=True, text=True)
    assert run.returncode == 0, run.stderr[-3000:]
    assert run.stdout.startswith("same"), run.stdout
