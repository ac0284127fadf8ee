"""Resident launches whose blocks give up their waits for each other: the bound on the
waits is set to one poll, every kernel leaves normally, and the call's answer is that of
the sweeps, which repeat the solve from the state before it."""
import numpy as np
import pytest

from synth.configs import config_uniform
from synth.hierarchy import Hierarchy

pytestmark = pytest.mark.gpu


def _problem(k=1200, base=5, coupled=True, seed=7):
    """A uniform base level and one finer level of k octs drawn at random: both levels in
    several shares, which have to wait for each other."""
    p = config_uniform(base, kmode="lp", seed=seed)
    n = 1 << base
    cells = np.stack(np.meshgrid(*[np.arange(n, dtype=np.int32)] * 3, indexing="ij"), -1).reshape(-1, 3)
    pick = np.random.default_rng(seed).permutation(len(cells))[:k]
    p.hierarchy = Hierarchy(base, {base: p.hierarchy.octs[base], base + 1: np.ascontiguousarray(cells[pick])})
    if coupled:
        E = p.E
        p.T = lambda level, ijk: E(level, ijk) ** 0.25
    return p


def _fields(s, p):
    from paper_1401_1112_amd.solver import to_numpy
    out = []
    for l in p.hierarchy.levels:
        if p.T is None:
            out.append(to_numpy(s.E(l)))
        else:
            out += [to_numpy(x) for x in s.E(l, with_T=True)]
    return out


def _levels(p, mode, resident, wait_limit, precision, unique=False, steps=1, level=None, **kw):
    from paper_1401_1112_amd.solver import solver_from_problem
    s = solver_from_problem(p, precision=precision, **kw)
    if level is not None:
        s.set_resident(False)
        s.advance(p.dt_coarse, mode, 1e-10)
    s.set_resident(resident, wait_limit)
    st = []
    for _ in range(steps):
        if level is not None:
            s.solve_level(level, p.dt_coarse, mode, 1e-10)
        elif unique:
            s.advance_unique(p.dt_coarse, 1e-10)
        else:
            s.advance(p.dt_coarse, mode, 1e-10)
        st += s.stats()
    out = _fields(s, p), st
    s.close()
    return out


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("mode", [0, 2])
@pytest.mark.parametrize("coupled", [False, True])
def test_level_solves_that_give_up_equal_sweeps(precision, mode, coupled):
    # energies, temperatures and (through the coarse solve) the flux register, bit for bit
    p = _problem(coupled=coupled)
    ref, st_ref = _levels(p, mode, False, 0, precision)
    got, st = _levels(p, mode, True, 1, precision)
    assert all(x["resident"] == 0 for x in st_ref)
    assert [x["resident"] for x in st] == [2] + [0] * (len(st) - 1)  # the others do not try
    assert all(x["launch_blocks"] == x["sweep_blocks"] for x in st)
    assert [x["iters"] for x in st] == [x["iters"] for x in st_ref]
    for a, b in zip(got, ref):
        assert np.array_equal(a, b)
    # one level's solve alone, after a step in sweeps (and with its register)
    for level in p.hierarchy.levels:
        ref, st_ref = _levels(p, mode, False, 0, precision, level=level)
        got, st = _levels(p, mode, True, 1, precision, level=level)
        assert [x["resident"] for x in st] == [2] and st[0]["iters"] == st_ref[0]["iters"]
        for a, b in zip(got, ref):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("precision", [0, 1])
def test_captured_step_that_gave_up_starts_clean_again(precision):
    # no launch of a replay takes the words of one that gave up for its own: the step
    # fails as a whole, every time, and after it the same context makes the step it would
    # have made, bit for bit
    from paper_1401_1112_amd import _lib as L
    from paper_1401_1112_amd.solver import sample_problem_fields, solver_from_problem
    p = _problem()
    ref, st_ref = _levels(p, 2, True, 0, precision, steps=2, persistent=True, graph=True)
    s = solver_from_problem(p, precision=precision, persistent=True, graph=True)
    s.set_resident(True, 1)
    for _ in range(3):
        sample_problem_fields(s, p)
        assert s.advance(p.dt_coarse, 2, 1e-10, raise_on_error=False) == L.E_DEVICE
        assert "did not meet" in s.last_error() and "not finished" in s.last_error()
        assert not any(x["converged"] for x in s.stats())
    s.set_resident(True)
    sample_problem_fields(s, p)
    st = []
    for _ in range(2):
        s.advance(p.dt_coarse, 2, 1e-10)
        st += s.stats()
    assert [x["iters"] for x in st] == [x["iters"] for x in st_ref]
    for a, b in zip(_fields(s, p), ref):
        assert np.array_equal(a, b)
    s.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("graph", [False, True])
def test_batch_launches_that_gave_up_start_clean_again(precision, graph):
    from paper_1401_1112_amd import _lib as L
    from paper_1401_1112_amd.solver import BatchSolver
    from synth.configs import patch_batch
    patches, alpha = patch_batch(4100, 5, n_min=4, n_max=48)
    ref = BatchSolver(robin_alpha=alpha, persistent=True, graph=graph)
    want, _ = ref.solve(patches, 3, 1e-10, precision=precision)
    ref.close()
    b = BatchSolver(robin_alpha=alpha, persistent=True, graph=graph)
    b.set_resident(True, 1)
    for _ in range(2):
        assert b.solve(patches, 3, 1e-10, precision=precision, raise_on_error=False)[1] == L.E_DEVICE
        assert "did not meet" in b.last_error()
    b.set_resident(True)
    got, _ = b.solve(patches, 3, 1e-10, precision=precision)
    b.close()
    for x, y in zip(got, want):
        assert np.array_equal(x, y)


def test_composite_and_batch_that_give_up_equal_sweeps():
    from paper_1401_1112_amd.solver import BatchSolver
    from synth.configs import patch_batch
    p = _problem(coupled=False)
    ref, st_ref = _levels(p, 0, False, 0, 0, unique=True)
    got, st = _levels(p, 0, True, 1, 0, unique=True)
    assert all(x["resident"] == 0 for x in st_ref)
    assert [x["resident"] for x in st] == [2] + [0] * (len(st) - 1)
    assert [x["iters"] for x in st] == [x["iters"] for x in st_ref]
    for a, b in zip(got, ref):
        assert np.array_equal(a, b)
    patches, alpha = patch_batch(4100, 5, n_min=4, n_max=48)
    for precision in (0, 1):
        out = []
        for resident, wait_limit in ((False, 0), (True, 1), (True, 0)):
            s = BatchSolver(robin_alpha=alpha)
            s.set_resident(resident, wait_limit)
            res, _ = s.solve(patches, 2, 1e-10, precision=precision)
            out.append((res, {x["resident"] for x in s.stats()}))
            s.close()
        assert [x[1] for x in out] == [{0}, {2}, {1}]
        for a, b in zip(out[0][0], out[1][0]):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("form", ["polled", "persistent", "graph"])
def test_blocks_wait_for_earlier_patches_of_a_batch(form):
    # more shares than blocks, one patch that iterates until its residual is zero and the
    # others at rest: blocks that come to a patch early wait for those still at the slow
    # one, however short the bound on the waits within a solve
    from paper_1401_1112_amd.solver import BatchSolver
    from synth.configs import patch_batch
    patches, alpha = patch_batch(4300, 200, n_min=18, n_max=26)
    slow = max(patches, key=lambda p: p.n)  # worked on first
    for p in patches:
        if p is not slow:
            p.E, p.face_mode, p.face_flux = np.ones_like(p.E), np.ones(6, dtype=np.int32), np.zeros(6)
    s = BatchSolver(robin_alpha=alpha, abs_floor=1e-12, persistent=form != "polled", graph=form == "graph")
    s.set_resident(True, 300)
    _, status = s.solve(patches, 1, 0.0, raise_on_error=False)
    st = s.stats()
    s.close()
    assert status in (0, -5) and {x["resident"] for x in st} == {1}
    its = sorted(x["iters"] for x in st)
    assert its[-2] <= 1 and its[-1] > 1000  # at 3 us or more each: longer than the bound


def test_solves_after_one_that_gave_up_do_not_try_again_at_once():
    from paper_1401_1112_amd.solver import solver_from_problem
    p = config_uniform(5, kmode="lp", seed=3)
    s = solver_from_problem(p)

    def forms(n):
        out = []
        for _ in range(n):
            s.solve_level(5, 1e-3 / 32 ** 2, 0, 1e-6)
            out.append(s.stats()[0]["resident"])
        return out

    s.set_resident(True, 1)
    assert forms(1 + 16 + 1 + 32 + 1) == [2] + [0] * 16 + [2] + [0] * 32 + [2]
    s.set_resident(True)  # starts anew
    assert forms(3) == [1] * 3
    s.close()
