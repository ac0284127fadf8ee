"""Device memory that is missing for the tables of resident solves only: levels, batches and
composite systems are built all the same and solved in sweeps. In a process of its own, with
a hipMalloc in front of the runtime's that fails for chosen sizes."""
import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")]

CHILD = """
import ctypes, json, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lo, hi = ctypes.c_size_t.in_dll(shim, "fail_lo"), ctypes.c_size_t.in_dll(shim, "fail_hi")
sys.path[:0] = [sys.argv[2], sys.argv[2] + "/tests"]
import numpy as np
import torch
from paper_1401_1112_amd.solver import BatchSolver, solver_from_problem, to_numpy
from synth.configs import config_uniform, patch_batch
out = {}

def fail(size):
    lo.value, hi.value = (size, size) if size else (1, 0)

def both(name, size, make, solve):
    got = []
    for on in (False, True):
        fail(size if on else 0)
        before = ctypes.c_int.in_dll(shim, "failed").value
        s = make()
        if not on:
            s.set_resident(False)
        got.append(solve(s))
        s.close()
        fail(0)
    out[name] = {"failed": ctypes.c_int.in_dll(shim, "failed").value - before, "resident": got[1][1],
                 "same": all(np.array_equal(a, b) for a, b in zip(got[0][0], got[1][0]))}

def level_solve(level, dt):
    def f(s):
        s.solve_level(level, dt, 0, 1e-8)
        st = s.stats()
        return [to_numpy(s.E(level))], sorted({x["resident"] for x in st})
    return f

def unique(s):
    s.advance_unique(12.0 / 32 ** 2, 1e-8)
    return [to_numpy(s.E(l)) for l in s.levels], sorted({x["resident"] for x in s.stats()})

p5 = config_uniform(5, kmode="lp", seed=3)
both("level", 12, lambda: solver_from_problem(p5), level_solve(5, 12.0 / 32 ** 2))
both("streamed", 256 * 11 * 4096 * 8, lambda: solver_from_problem(config_uniform(7, kmode="const", seed=3)),
     level_solve(7, 12.0 / 128 ** 2))
from synth.configs import config_tiny
two = config_tiny(11, base_level=4, max_level=5, p_refine=0.4, kmode="lp", tol=1e-12)
both("composite", 12, lambda: solver_from_problem(two), unique)
patches, alpha = patch_batch(4100, 5, n_min=4, n_max=48)

def batch(s):
    res, _ = s.solve(patches, 2, 1e-10)
    return res, sorted({x["resident"] for x in s.stats()})
both("batch", 4 * (2 * 5 + 1), lambda: BatchSolver(robin_alpha=alpha), batch)
print(json.dumps(out))
"""


def test_solves_without_memory_for_resident_tables(tmp_path):
    shim = str(tmp_path / "fail_malloc.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "host", "fail_malloc.c"), "-o", shim,
                    "-ldl"], check=True)
    run = subprocess.run([sys.executable, "-c", CHILD, shim, ROOT], capture_output=True, text=True, timeout=100, cwd=ROOT)
    assert run.returncode == 0, run.stderr[-3000:]
    out = json.loads(run.stdout.strip().splitlines()[-1])
    assert set(out) == {"level", "streamed", "composite", "batch"}
    for name, x in out.items():
        assert x["failed"] > 0 and x["resident"] == [0] and x["same"], (name, x)
