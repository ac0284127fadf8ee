"""The sweeps on levels and patches of the sizes that run resident by default: the tests
of parity, launch forms, formed coefficients, variants and refinement again, on solvers
whose resident form is switched off (amrfld_set_resident).  The sweeps still run every
larger level and patch and repeat a resident launch that did not end."""
import numpy as np
import pytest

from synth.configs import config_uniform, patch_batch

# fixtures and tests of the other modules, collected here a second time
from test_gpu_batch import (test_batch_fp64_parity_per_step, test_batch_matches_single_patch_calls,  # noqa: F401
                            test_batch_mixed_precision_reaches_tolerance,
                            test_batch_persistent_launch_equals_polled, test_batch_uneven_sizes_and_modes)
from test_gpu_checks import test_refinement_split_keeps_the_fp64_threshold  # noqa: F401
from test_gpu_coefs import (test_formed_equals_stored_batch, test_formed_equals_stored_levels,  # noqa: F401
                            test_formed_equals_stored_variants, test_mixed_formed_and_stored_both_meet_threshold)
from test_gpu_collapse import (test_collapse_fp64_parity, test_collapse_mixed_inner_plan_of_its_own,  # noqa: F401
                               test_collapse_mixed_reaches_tolerance, test_collapse_persistent_equals_polled)
from test_gpu_dirac import test_dirac_parity_reduced  # noqa: F401
from test_gpu_equilibrium import (test_equilibrium_flux_limited_parity, test_equilibrium_mixed_precision,  # noqa: F401
                                  test_equilibrium_parity_adaptive_reduced, test_equilibrium_parity_unique_reduced)
from test_gpu_fullsize import (fp64_step, gpu_solver, lognormal, oracle_step,  # noqa: F401
                               test_lognormal_formed_coefficients_equal_stored_bitwise,
                               test_lognormal_full_step_parity, test_lognormal_full_step_residuals,
                               test_lognormal_mixed_full_step, test_lognormal_persistent_equals_polled)
from test_gpu_graph import (test_graph_launch_shape_change_recaptures,  # noqa: F401
                            test_graph_mixed_replays_equal_eager, test_graph_recaptures_on_changes,
                            test_graph_replays_equal_eager, test_graph_theta_and_formed_coefficients)
from test_gpu_parity import (test_constant_state_zero_iterations, test_coupled_temperature_parity,  # noqa: F401
                             test_heat_gaussian_parity_every_step, test_mixed_precision_inner_iterations_track_fp64_cg,
                             test_mixed_precision_refinement_reaches_fp64_tolerance,
                             test_mixed_precision_uniform_closed_form, test_nan_density_is_nonfinite,
                             test_negative_energy_reported_like_oracle, test_noconv_returns_status_and_iterate,
                             test_own_schedule_with_restrict_equals_advance, test_persistent_level_solves_equal_polled,
                             test_tiny_amr_advance_parity, test_uniform_level_closed_form)
from test_gpu_unique import (test_unique_on_one_level_is_the_level_solve, test_unique_parity_coupled_collapse,  # noqa: F401
                             test_unique_parity_heat_gaussian, test_unique_parity_tiny)
from test_gpu_variants import (test_crank_nicolson_amr_parity, test_crank_nicolson_closed_form,  # noqa: F401
                               test_crank_nicolson_persistent_and_mixed, test_minerbo_amr_parity,
                               test_minerbo_batch_parity)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _sweeps_only():
    from paper_1401_1112_amd import solver as S
    with pytest.MonkeyPatch.context() as m:
        for cls in (S.HierarchySolver, S.BatchSolver):
            def init(self, *a, _was=cls.__init__, **kw):
                _was(self, *a, **kw)
                self.set_resident(False)
            m.setattr(cls, "__init__", init)
        yield


def test_the_switch_selects_the_form():
    # a level of 64 blocks, the composite of it alone and a batch, either way; the two
    # forms agree to rounding
    from paper_1401_1112_amd.solver import BatchSolver, solver_from_problem, to_numpy
    p = config_uniform(5, kmode="lp", seed=3)
    patches, alpha = patch_batch(4100, 3, n_min=8, n_max=20)
    out = {}
    for on in (False, True, False):
        s = solver_from_problem(p)
        s.set_resident(on)
        s.solve_level(5, 12.0 / 32 ** 2, 0, 1e-10)
        level = s.stats()[0]
        s.advance_unique(12.0 / 32 ** 2, 1e-10)
        comp = s.stats()[0]
        assert level["resident"] == comp["resident"] == int(on)
        b = BatchSolver(robin_alpha=alpha, time_sweeps=1)
        b.set_resident(on)
        res, _ = b.solve(patches, 2, 1e-10)
        # (sweeps are timed, resident patches are not)
        assert all(x["resident"] == int(on) and (x["n_timed"] == 0) == on for x in b.stats())
        out.setdefault(on, []).append([to_numpy(s.E(5))] + res)
        s.close()
        b.close()
    for a, c, d in zip(out[False][0], out[False][1], out[True][0]):
        assert np.array_equal(a, c)
        assert np.linalg.norm(a - d) <= 1e-9 * np.linalg.norm(a)


def test_set_resident_rejects_other_values():
    from paper_1401_1112_amd import _lib as L
    from paper_1401_1112_amd.solver import BatchSolver
    b = BatchSolver()
    for resident, wait in ((2, 0), (-1, 0), (1, -1)):
        assert L.amrfld_set_resident(b.ctx, resident, wait) == L.E_INVALID
        assert "set_resident" in b.last_error()
    b.close()
