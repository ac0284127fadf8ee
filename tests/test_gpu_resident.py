"""The resident CG of FP64 level solves (csrc/resident.hip) against the oracle at the
sizes where its shares change: one oct, the largest share of one block and one oct more,
whole and ragged last pairs of a thread, one and several waves of share words, faces
between shares on every side; and contexts on several streams and threads at once, whose
launches have to take turns on the device.

Bar: relative L2 <= 1e-12 with equal iteration counts (a near-tie of a residual with its
threshold: both sides again with tol 0 at the larger count)."""
import threading

import numpy as np
import pytest

from _util import align, oracle_from_problem
import oracle as ora
from synth.configs import config_uniform
from synth.hierarchy import Hierarchy

pytestmark = pytest.mark.gpu


def _problem(k, seed=1, base=4, compact=False):
    """A uniform base level and one finer level of k octs: the first k base cells in
    Morton-like blocks (compact) or k cells drawn at random."""
    p = config_uniform(base, kmode="lp", seed=seed)
    n = 1 << base
    rng = np.random.default_rng(seed)
    cells = np.array([[i, j, l] for i in range(n) for j in range(n) for l in range(n)], dtype=np.int32)
    pick = np.arange(k) if compact else rng.permutation(len(cells))[:k]
    p.hierarchy = Hierarchy(base, {base: p.hierarchy.octs[base], base + 1: np.ascontiguousarray(cells[pick])})
    return p


def _solve(p, level, dt, tol, max_iter=10000, **kw):
    from paper_1401_1112_amd.solver import solver_from_problem, to_numpy
    s = solver_from_problem(p, max_iter=max_iter, **kw)
    s.solve_level(level, dt, 0, tol, raise_on_error=False)
    out = to_numpy(s.E(level)), s.cells(level), s.stats()[0]
    s.close()
    return out


def _check(p, level, dt, tol):
    o = oracle_from_problem(p)
    h = o.solve_level(level, dt, ora.DIRICHLET, tol)
    e, cells, st = _solve(p, level, dt, tol)
    if st["iters"] != h["iters"]:  # near-tie: the larger count on both sides
        n = max(st["iters"], h["iters"])
        o = oracle_from_problem(p, max_iter=n, abs_floor=0.0)
        h = o.solve_level(level, dt, ora.DIRICHLET, 0.0)
        e, cells, st = _solve(p, level, dt, 0.0, max_iter=n, abs_floor=0.0)
    assert st["iters"] == h["iters"]
    ref = align(level, o.cells(level), o.E[level], cells)
    assert np.linalg.norm(e - ref) <= 1e-12 * np.linalg.norm(ref)
    assert np.isclose(st["min_E"], h["min_E"], rtol=1e-10)
    assert abs(st["true_rel_res"] * st["rnorm0"] - h["true_res"]) <= 0.05 * h["true_res"] + 1e-14 * h["bnorm"]
    return st


@pytest.mark.parametrize("k", [1, 2, 127, 128, 129, 640, 641, 1000, 2049, 4095])
@pytest.mark.parametrize("compact", [False, True])
def test_sizes_against_oracle(k, compact):
    p = _problem(k, seed=k, compact=compact)
    st = _check(p, 5, 12.0 / 32 ** 2, 1e-10)
    assert (st["launch_blocks"] == 1) == (k <= 640)


@pytest.mark.parametrize("level", [1, 2, 3, 6])
def test_uniform_levels_against_oracle(level):
    p = config_uniform(level, kmode="lp", seed=level)
    _check(p, level, 12.0 / 4 ** level, 1e-10)


def test_fixed_counts_and_no_linf_test():
    p = _problem(700, seed=5)
    for kw in ({"linf_test": False}, {"true_residual": False}):
        o = oracle_from_problem(p, **({"linf_test": False} if "linf_test" in kw else {}))
        h = o.solve_level(5, 12.0 / 32 ** 2, ora.DIRICHLET, 1e-8)
        e, cells, st = _solve(p, 5, 12.0 / 32 ** 2, 1e-8, **kw)
        assert st["iters"] == h["iters"]
        ref = align(5, o.cells(5), o.E[5], cells)
        assert np.linalg.norm(e - ref) <= 1e-12 * np.linalg.norm(ref)
        assert (st["true_rel_res"] == -1.0) == ("true_residual" in kw)


def test_contexts_on_streams_and_threads():
    # several contexts, each with a stream and a thread of its own, on levels of many
    # blocks: their launches wait for each other on the device and every result is the
    # one of the context alone, bit for bit
    import torch
    from paper_1401_1112_amd.solver import solver_from_problem, to_numpy
    ps = [_problem(k, seed=20 + k) for k in (3000, 4096, 900, 4000)]
    alone = [_solve(p, 5, 12.0 / 32 ** 2, 1e-10)[0] for p in ps]
    streams = [torch.cuda.Stream() for _ in ps]
    solvers = []
    for p, st in zip(ps, streams):
        with torch.cuda.stream(st):
            solvers.append(solver_from_problem(p, stream=st))
    torch.cuda.synchronize()
    out, errors = [None] * len(ps), []

    def work(k):
        try:
            p, s = ps[k], solvers[k]
            with torch.cuda.stream(streams[k]):
                for _ in range(4):
                    for l in (4, 5):
                        c = s.cells(l)
                        s.set_fields(l, p.rho(l, c), p.E(l, c), kmode=1)
                    s.solve_level(5, 12.0 / 32 ** 2, 0, 1e-10)
                out[k] = s.E(5)
            streams[k].synchronize()
        except Exception as e:  # reported below, in the main thread
            errors.append((k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(ps))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k, s in enumerate(solvers):
        assert np.array_equal(to_numpy(out[k]), alone[k]), k
        s.close()


@pytest.mark.parametrize("k", [163841, 200000, 262144])
def test_streamed_coefficients_against_oracle(k):
    # shares of six to eight pairs per thread, the last one full
    p = _problem(k, seed=3, base=6, compact=True)
    kw = dict(max_iter=20, abs_floor=0.0)
    o = oracle_from_problem(p, **kw)
    h = o.solve_level(7, 12.0 / 128 ** 2, ora.DIRICHLET, 0.0)
    e, cells, st = _solve(p, 7, 12.0 / 128 ** 2, 0.0, **kw)
    assert st["iters"] == h["iters"] == 20 and st["launch_blocks"] == 256
    ref = align(7, o.cells(7), o.E[7], cells)
    assert np.linalg.norm(e - ref) <= 1e-12 * np.linalg.norm(ref)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("n_big", [112, 136])
def test_batch_of_resident_and_swept_patches(precision, graph, n_big):
    # one patch of streamed coefficients (112^3 cells) or above the resident size (136^3)
    # among small ones, two steps: the small ones against the oracle, the large one by its
    # true residual; no sweep of the large patch may touch the others' energies
    from oracle.patch_oracle import patch_advance
    from paper_1401_1112_amd import FP64, MIXED
    from paper_1401_1112_amd.solver import BatchSolver
    from synth.configs import patch_batch
    small, alpha = patch_batch(5100, 6, n_min=2, n_max=40)
    big, _ = patch_batch(5200, 1, n_min=n_big, n_max=n_big)
    patches = small[:3] + big + small[3:]
    s = BatchSolver(robin_alpha=alpha, persistent=graph, graph=graph)
    res, status = s.solve(patches, 2, 1e-10, precision=MIXED if precision == "mixed" else FP64)
    st = s.stats()
    s.close()
    assert status == 0 and all(x["converged"] == 1 for x in st)
    for x in st:
        thr = max(1e-10 * x["rnorm0"], 1e-14 * x["bnorm"])
        assert x["true_rel_res"] * x["rnorm0"] <= (1.0 + 1e-12 if precision == "mixed" else 2.5) * thr
    for q, p in enumerate(patches):
        if p.n > 100:
            assert np.isfinite(res[q]).all()
            continue
        e, _ = patch_advance(p.rho, p.E, p.dx, p.dt, p.face_mode, p.face_ghost, p.face_flux, 2, 1e-10, alpha=alpha)
        assert np.linalg.norm(res[q] - e) <= 1e-9 * np.linalg.norm(e), q


@pytest.mark.parametrize("base,top,refine", [(2, 3, 0.2), (3, 5, 0.5), (4, 6, 0.4)])
def test_composite_of_levels_against_oracle(base, top, refine):
    # couplings within a share, between shares of one and of several XCDs; fixed counts
    from paper_1401_1112_amd.solver import solver_from_problem, to_numpy
    from synth.configs import config_tiny
    p = config_tiny(11, base_level=base, max_level=top, p_refine=refine, kmode="lp", tol=1e-12)
    o = oracle_from_problem(p, max_iter=25, abs_floor=0.0)
    o.advance_unique(p.dt_coarse, 0.0)
    s = solver_from_problem(p, max_iter=25, abs_floor=0.0)
    s.advance_unique(p.dt_coarse, 0.0, raise_on_error=False)
    st = s.stats()
    assert all(x["iters"] == 25 for x in st)
    slots = sum(-(-8 * len(p.hierarchy.octs[l]) // 256) * 256 for l in p.hierarchy.levels)
    assert all(x["launch_blocks"] == max(2, min(256, shares(slots))) for x in st)
    for l in p.hierarchy.levels:
        e = to_numpy(s.E(l))
        ref = align(l, o.cells(l), o.E[l], s.cells(l))
        assert np.linalg.norm(e - ref) <= 1e-12 * np.linalg.norm(ref)
    s.close()


def shares(slots):
    n = -(-slots // 512)  # about 512 slots each, as many on every XCD from nine on
    return n if n <= 8 else -(-n // 8) * 8


def test_timed_sweeps_beside_slow_resident_patches():
    # the timed sweeps are those of the patch that is swept, however many iterations the
    # resident patches take
    from paper_1401_1112_amd.solver import BatchSolver
    from synth.configs import patch_batch
    small, alpha = patch_batch(5100, 3, n_min=30, n_max=40)
    big, _ = patch_batch(5200, 1, n_min=136, n_max=136)
    for p in small:
        p.dt *= 300.0  # 17 times the iterations
    big[0].dt *= 0.1
    for period in (1, 4):
        s = BatchSolver(robin_alpha=alpha, time_sweeps=period)
        _, status = s.solve(small + big, 2, 1e-10)
        st = s.stats()
        s.close()
        assert status == 0 and len(st) == 8
        for k in (0, 4):
            assert min(x["iters"] for x in st[k:k + 3]) > st[k + 3]["iters"]
            assert all(x["n_timed"] == 0 for x in st[k:k + 3])
            assert st[k + 3]["n_timed"] == st[k + 3]["iters"] // period
            assert st[k + 3]["n_timed"] == 0 or st[k + 3]["sweep_ms"] > 0


def test_time_per_iteration_of_a_resumed_solve():
    # a threshold below what rounding allows: the refined solve is resumed until its
    # launches are used up, and its time per iteration is that of a solve of one launch
    from paper_1401_1112_amd import MIXED
    p = config_uniform(5, kmode="lp", seed=9)
    us = {}
    for precision in (0, MIXED):
        kw = dict(time_sweeps=1, abs_floor=0.0, precision=precision, linf_test=False)
        for _ in range(3):
            _, _, st = _solve(p, 5, 12.0 / 32 ** 2, 1e-10 if precision == 0 else 1e-17, **kw)
        us[precision] = 1e3 * st["sweep_ms"] / st["n_timed"]
        assert st["n_timed"] == st["iters"]
    assert st["converged"] == 0
    assert 0.6 * us[0] <= us[MIXED] <= 1.7 * us[0], us


@pytest.mark.parametrize("inner_tol", [3e-3, 1e-1])
@pytest.mark.parametrize("form", ["polled", "graph"])
def test_refined_solve_ends_a_segment_below_its_threshold(inner_tol, form):
    # every segment of a refined solve reduces the residual by inner_tol, the stopping rule
    # looks at their ends only, and max_outer caps them: as in the sweeps.  (FP64 segments
    # overshoot inner_tol by other amounts than FP32 ones: one segment's leave.)
    from paper_1401_1112_amd import MIXED
    from paper_1401_1112_amd import _lib as L
    from paper_1401_1112_amd.solver import solver_from_problem
    p = config_uniform(5, kmode="lp", seed=13)
    kw = dict(precision=MIXED, inner_tol=inner_tol, persistent=form == "graph", graph=form == "graph")
    for max_outer in (30, 2, 1):
        got, linf = {}, {}
        for resident in (True, False):
            s = solver_from_problem(p, max_outer=max_outer, **kw)
            s.set_resident(resident)
            status = s.advance(12.0 / 32 ** 2, 0, 1e-10, raise_on_error=False)
            st = s.stats()[0]
            s.close()
            got[resident] = st["outer_iters"]
            linf[resident] = st["linf_change"]
            assert st["rel_res"] <= inner_tol ** st["outer_iters"] * (1 + 1e-6)
            assert status == (L.OK if max_outer == 30 else L.E_NOCONV)
            assert st["converged"] == (max_outer == 30)
            assert st["outer_iters"] == max_outer or max_outer == 30
        assert abs(got[True] - got[False]) <= 1
        # the change that a capped solve reports is that of its last iteration
        assert max_outer == 30 or np.isclose(linf[True], linf[False], rtol=1e-2)


@pytest.mark.parametrize("level", [3, 5])
@pytest.mark.parametrize("count", [1, 2])
def test_relative_change_of_cells_at_zero(level, count):
    # a pulse in one cell of an empty box: the cells it has just reached count with their
    # absolute change, in the units of the energy
    p = config_uniform(level, kmode="const", seed=2)
    p.E = lambda l, c: np.where((np.asarray(c) == 3).all(axis=1), 1e3, 0.0)
    dt = 12.0 / 4 ** level
    o = oracle_from_problem(p, max_iter=count, abs_floor=0.0)
    h = o.solve_level(level, dt, ora.DIRICHLET, 0.0)
    e, cells, st = _solve(p, level, dt, 0.0, max_iter=count, abs_floor=0.0)
    assert st["iters"] == h["iters"] == count
    assert np.isclose(st["linf_change"], h["linf"], rtol=1e-10)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("level", [2, 4, 5])
@pytest.mark.parametrize("dt,tol", [(1e-9, 1e-10), (12.0, 0.0)])
def test_residuals_down_to_underflow(level, precision, dt, tol):
    # a pulse into an empty box in a tiny step, whose relative changes stay above tol until
    # the residual is zero, and solves to a residual of zero: they end, converged, with the
    # oracle's energies
    p = config_uniform(level, kmode="const", seed=2)
    if tol:
        p.E = lambda l, c: np.where((np.asarray(c) == 2).all(axis=1), 1e3, 0.0)
    kw = {} if tol else dict(abs_floor=0.0, linf_test=False)
    o = oracle_from_problem(p, **kw)
    o.solve_level(level, dt / 4 ** level, ora.DIRICHLET, 1e-13)
    e, cells, st = _solve(p, level, dt / 4 ** level, tol, precision=precision, **kw)
    if precision == 0:
        assert st["converged"] == 1 and st["status"] == 0
    else:
        assert st["status"] in ((0,) if tol else (0, -5))  # a true residual is never zero
    ref = align(level, o.cells(level), o.E[level], cells)
    assert np.linalg.norm(e - ref) <= 1e-11 * np.linalg.norm(ref)


def test_threads_whose_launches_need_other_amounts_of_lds():
    # the same kernel for shares with few and with many halo units, launched from threads at
    # the same time: no launch fails (it would be made in sweeps instead)
    import torch
    from paper_1401_1112_amd.solver import solver_from_problem
    ps = [_problem(k, seed=31 + k, compact=c) for k, c in ((700, True), (3000, False), (4096, True), (2000, False))]
    streams = [torch.cuda.Stream() for _ in ps]
    solvers = []
    for p, st in zip(ps, streams):
        with torch.cuda.stream(st):
            solvers.append(solver_from_problem(p, stream=st))
    torch.cuda.synchronize()
    forms = [[] for _ in ps]

    def work(k):
        with torch.cuda.stream(streams[k]):
            for _ in range(40):
                solvers[k].solve_level(5, 1e-3 / 32 ** 2, 0, 1e-6, raise_on_error=False)
                forms[k].append(solvers[k].stats()[0]["resident"])

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(ps))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for s in solvers:
        s.close()
    assert all(f == [1] * 40 for f in forms)


def test_contexts_side_by_side_are_the_same_bits():
    # eight contexts on threads of their own with levels of 8 to 96 shares: their launches
    # run side by side or in turn, in the form for company or alone, with the bits of the
    # context alone, and none gives up
    import torch
    from paper_1401_1112_amd.solver import solver_from_problem, to_numpy
    ps = [_problem(k, seed=50 + k) for k in (650, 900, 1400, 2000, 3000, 4000, 4096)] + \
        [config_uniform(5, kmode="lp", seed=4)]
    lv = [5] * len(ps)
    alone = [_solve(p, l, 12.0 / 32 ** 2, 1e-10)[0] for p, l in zip(ps, lv)]
    streams = [torch.cuda.Stream() for _ in ps]
    solvers = []
    for p, st in zip(ps, streams):
        with torch.cuda.stream(st):
            solvers.append(solver_from_problem(p, stream=st))
    torch.cuda.synchronize()
    out, forms = [[] for _ in ps], [[] for _ in ps]

    def work(k):
        p, s = ps[k], solvers[k]
        with torch.cuda.stream(streams[k]):
            for _ in range(12):
                for l in p.hierarchy.levels:
                    c = s.cells(l)
                    s.set_fields(l, p.rho(l, c), p.E(l, c), kmode=1)
                s.solve_level(lv[k], 12.0 / 32 ** 2, 0, 1e-10)
                forms[k].append(s.stats()[0]["resident"])
                out[k].append(s.E(lv[k]))
        streams[k].synchronize()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(ps))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k, s in enumerate(solvers):
        assert forms[k] == [1] * 12
        for e in out[k]:
            assert np.array_equal(to_numpy(e), alone[k]), k
        s.close()
