"""The one-block-per-plane pass of 32^3 and 64^3 grids (schedule 0 of the y inverse, x pass and
y forward), the general column passes at the smallest lines, and the shell sums at the edges of
their range, against the CPU oracle.  Bars: 1e-12 relative L2 in FP64, 1e-5 in FP32, as for every
step kernel."""
import numpy as np
import pytest

import oracle as ora
from paper_2012_04838_amd import inputs
from tests.gpu_helpers import gpu_rhs, make_plan, poisoned_workspace, progress, rel_l2, set_params, to_numpy, torch_mod

pytestmark = pytest.mark.gpu

SC = (0.7, 1.0, 0.25, 4.0)
GRAD = ((0.0, 1.0, 0.0), (0.2, 1.0, -0.3), (0.5, 0.0, -0.25), (0.0, 0.0, 1.0))


def _prm(S, nu=0.01):
    return ora.Params(nu=nu, schmidt=SC[:S], mean_grad=GRAD[:S], power=0.1, k_force=2.0, forcing=True)


@pytest.mark.parametrize("N", [32, 64])
@pytest.mark.parametrize("S", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("prec", [32, 64])
def test_plane_rhs_matches_oracle_and_the_separate_passes(N, S, prec):
    torch_mod()
    tol = 1e-12 if prec == 64 else 1e-5
    x = inputs.random_spectral_state(N, 3 + S, 11 * N + S, ora.kmax_retained(N), 6.0)
    prm = _prm(S)
    ref = ora.rhs(x, prm)
    plan = make_plan(N, S, prec)
    set_params(plan, 0, prm)
    st, out = plan.new_state(), plan.new_state()
    plan.set_state(st, x, 0)
    got = {}
    # the plane pass, and the same schedule with one of its passes apart
    for sched in ([0, 0, 0, 0, 0], [0, 0, 1, 0, 0]):
        plan.set_pass_schedules(sched)
        out.zero_()
        plan.rhs(st, out, poisoned_workspace(plan))
        got[sched[2]] = to_numpy(plan.get_state(out, 0))
    progress(f"[plane] N={N} S={S} FP{prec} rhs rel L2 {rel_l2(got[0], ref):.2e} (separate passes {rel_l2(got[1], ref):.2e})")
    assert rel_l2(got[0], ref) < tol and rel_l2(got[1], ref) < tol
    assert rel_l2(got[0], got[1]) < 2 * tol


@pytest.mark.parametrize("N,S,prec", [(32, 1, 64), (64, 2, 64), (64, 1, 32)])
def test_plane_cfl_steps_in_a_batch(N, S, prec):
    """CFL steps (the grid maximum and the step record) of two slots around an inactive one."""
    torch_mod()
    prm = [_prm(S, 0.01), _prm(S, 0.02), _prm(S, 0.005)]
    y = [inputs.random_spectral_state(N, 3 + S, 5 + i, ora.kmax_retained(N), 4.0, 0.02 * (i + 1)) for i in range(3)]
    plan = make_plan(N, S, prec, batch=3)
    st, ws = plan.new_state(), poisoned_workspace(plan)
    for i in range(3):
        set_params(plan, i, prm[i], active=i != 1)
        plan.set_state(st, y[i], i)
    plan.step(st, ws, -0.5, 2)
    plan.step(st, ws, -0.25, 1)
    info = plan.read_step_info(ws)
    tol = 1e-12 if prec == 64 else 1e-5
    for i in (0, 2):
        ref, d = ora.step(y[i], prm[i], nsteps=2, cfl=0.5, return_dts=True)
        ref, e = ora.step(ref, prm[i], nsteps=1, cfl=0.25, return_dts=True)
        assert rel_l2(to_numpy(plan.get_state(st, i)), ref) < tol
        assert abs(info[i]["t"] - sum(d) - sum(e)) < max(tol, 1e-6 if prec == 32 else 0) * info[i]["t"]
        assert info[i]["steps"] == 3
    assert info[1]["steps"] == 0
    assert rel_l2(to_numpy(plan.get_state(st, 1)), y[1]) < (1e-15 if prec == 64 else 1e-6)


def test_plane_tuner_takes_the_three_passes_together():
    torch_mod()
    plan = make_plan(64, 1, 32)
    set_params(plan, 0, _prm(1))
    st, ws = plan.new_state(), plan.new_workspace()
    plan.init_field(st, ws, 0, 3, 4.0)
    best, _ = plan.tune_passes(st, ws, 2)
    three = best[1:4]
    assert three == [0, 0, 0] or 0 not in three


@pytest.mark.parametrize("N,S", [(10, 1), (12, 0), (14, 2), (18, 1), (22, 1), (26, 4), (98, 0)])
def test_general_columns_at_small_and_odd_lines(N, S):
    x = inputs.random_spectral_state(N, 3 + S, 70 + N, ora.kmax_retained(N), 3.0)
    prm = _prm(S)
    ref = ora.rhs(x, prm)
    assert rel_l2(gpu_rhs(x, prm, 64), ref) < 1e-12
    assert rel_l2(gpu_rhs(x, prm, 32), ref) < 1e-5


@pytest.mark.parametrize("N,S", [(8, 4), (24, 3), (200, 0)])
def test_shell_sums_at_the_edges(N, S):
    """Rows of three columns, four scalars, and rows longer than a wavefront (67 columns)."""
    torch_mod()
    prm = _prm(S)
    y = inputs.random_spectral_state(N, 3 + S, 2 + N, ora.kmax_retained(N), 0.3 * N, 0.1)
    plan = make_plan(N, S, 64)
    set_params(plan, 0, prm)
    st, ws = plan.new_state(), poisoned_workspace(plan)
    plan.set_state(st, y, 0)
    got = plan.spectra(st, ws)[0]
    ref = ora.spectra(y, prm)
    # sums of up to 1e5 positive FP64 terms in another order
    assert np.allclose(got["E"], ref["E"], rtol=1e-12, atol=1e-14 * ref["E"].max())
    for s in range(S):
        assert np.allclose(got["E_phi"][s], ref["E_phi"][s], rtol=1e-12, atol=1e-14 * ref["E_phi"][s].max())
    for k in ("K", "eps", "Re_lambda", "chi", "phi_var"):
        assert np.allclose(got[k], ref[k], rtol=1e-12)
