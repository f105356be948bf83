"""The general x pass at every way its lines share wavefronts (16, 32 and 64 lanes per line, lines past
the last of a grid, batches that change the choice), against the CPU oracle, and the shell sums of
the statistics in a batch and with more than 64 KB of LDS.  The plan's x_lines (lines per
256-thread block, 256 / lanes) says that the intended shape ran.  Bars: 1e-12 relative L2 in FP64,
1e-5 in FP32, as for every step kernel."""
import numpy as np
import pytest

import oracle as ora
from paper_2012_04838_amd import inputs, psdns
from tests.gpu_helpers import make_plan, poisoned_workspace, progress, rel_l2, set_params, to_numpy, torch_mod

pytestmark = pytest.mark.gpu

SC = (0.7, 1.0, 0.25, 4.0)
GRAD = ((0.0, 1.0, 0.0), (0.2, 1.0, -0.3), (0.5, 0.0, -0.25), (0.0, 0.0, 1.0))


def _prm(S, nu=0.01, dealias="cube"):
    return ora.Params(nu=nu, schmidt=SC[:S], mean_grad=GRAD[:S], power=0.1, k_force=2.0, forcing=True, dealias=dealias)


def _tol(prec):
    return 1e-12 if prec == 64 else 1e-5


# 98 and 90: 16 lanes, N^2 mod 16 = 4 lines past the last; 70: 32 lanes, 4 past the last; 84: 16 lanes,
# none; 40: a whole wavefront
@pytest.mark.parametrize("N,S,lines", [(98, 1, 16), (90, 3, 16), (84, 2, 16), (70, 2, 8), (40, 1, 4)])
def test_cfl_step_on_shared_wavefronts(N, S, lines):
    """One CFL step: the grid maximum (lanes past the last line add nothing to it) and the products."""
    torch_mod()
    prm = _prm(S)
    y = inputs.random_spectral_state(N, 3 + S, 31 + N, ora.kmax_retained(N), 6.0, 0.05)
    progress(f"[lines] N={N} S={S} oracle step")
    ref, dts = ora.step(y, prm, nsteps=1, cfl=0.5, return_dts=True)
    for prec in (64, 32):
        plan = make_plan(N, S, prec)
        assert plan.schedule_info(0)["x_lines"] == lines
        set_params(plan, 0, prm)
        st, ws = plan.new_state(), poisoned_workspace(plan)
        plan.set_state(st, y, 0)
        plan.step(st, ws, -0.5, 1)
        got, info = to_numpy(plan.get_state(st, 0)), plan.read_step_info(ws)[0]
        progress(f"[lines] N={N} S={S} FP{prec} rel L2 {rel_l2(got, ref):.2e}, dt {info['dt']:.15e} ({dts[0]:.15e})")
        assert rel_l2(got, ref) < _tol(prec)
        assert abs(info["dt"] - dts[0]) < _tol(prec) * dts[0]


@pytest.mark.parametrize("N,S,lines,alone", [(50, 1, 16, 4), (42, 3, 8, 4)])
@pytest.mark.parametrize("prec", [64, 32])
def test_batch_changes_the_shape_but_not_the_slots(N, S, lines, alone, prec):
    """Three slots, the middle one inactive, take more lines per wavefront than one slot does; each
    active slot matches the oracle and equals the same slot stepped alone."""
    torch_mod()
    prms = [_prm(S, nu) for nu in (0.01, 0.02, 0.005)]
    ys = [inputs.random_spectral_state(N, 3 + S, 7 * N + i, ora.kmax_retained(N), 4.0, 0.03 * (i + 1)) for i in range(3)]
    plan = make_plan(N, S, prec, batch=3)
    assert plan.schedule_info(0)["x_lines"] == lines
    st, ws = plan.new_state(), poisoned_workspace(plan)
    for i in range(3):
        set_params(plan, i, prms[i], active=i != 1)
        plan.set_state(st, ys[i], i)
    plan.step(st, ws, -0.5, 1)
    for i in (0, 2):
        got = to_numpy(plan.get_state(st, i))
        assert rel_l2(got, ora.step(ys[i], prms[i], nsteps=1, cfl=0.5)) < _tol(prec)
        one = make_plan(N, S, prec)
        assert one.schedule_info(0)["x_lines"] == alone
        set_params(one, 0, prms[i])
        s1, w1 = one.new_state(), poisoned_workspace(one)
        one.set_state(s1, ys[i], 0)
        one.step(s1, w1, -0.5, 1)
        diff = rel_l2(to_numpy(one.get_state(s1, 0)), got)
        progress(f"[lines] N={N} FP{prec} slot {i} in a batch and alone differ by {diff:.2e}")
        assert diff < _tol(prec)
    assert rel_l2(to_numpy(plan.get_state(st, 1)), ys[1]) < (1e-15 if prec == 64 else 1e-6)


@pytest.mark.parametrize("N,S,lines", [(84, 1, 16), (98, 1, 16), (70, 0, 8)])
def test_phase_shift_on_shared_wavefronts(N, S, lines):
    """The half-cell shift's factors where lines share a wavefront: right-hand side and one CFL step."""
    torch_mod()
    prm = _prm(S, dealias="phase")
    K = ora.kmax_retained(N, "phase")
    y = inputs.random_spectral_state(N, 3 + S, 5 + N, K, 6.0, 0.05)
    y = np.where(ora.retained_mask(N, "phase"), y, 0.0)
    progress(f"[lines] phase shift N={N} S={S} oracle")
    ref = ora.rhs(y, prm)
    step = ora.step(y, prm, nsteps=1, cfl=0.5)
    for prec in (64, 32):
        plan = make_plan(N, S, prec, dealias=psdns.DEALIAS_PHASE_SPHERE)
        assert plan.schedule_info(0)["x_lines"] == lines
        set_params(plan, 0, prm)
        st, out, ws = plan.new_state(), plan.new_state(), poisoned_workspace(plan)
        plan.set_state(st, y, 0)
        plan.rhs(st, out, ws)
        e_rhs = rel_l2(to_numpy(plan.get_state(out, 0)), ref)
        plan.step(st, ws, -0.5, 1)
        e_step = rel_l2(to_numpy(plan.get_state(st, 0)), step)
        progress(f"[lines] phase shift N={N} FP{prec} rhs {e_rhs:.2e}, step {e_step:.2e}")
        assert e_rhs < _tol(prec) and e_step < _tol(prec)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("N,S,positions", [(180, 1, 3), (250, 0, 4), (300, 0, 5)])
def test_fp32_lines_of_a_whole_wavefront(N, S, positions):
    """FP32 lines of 64 lanes with 3, 4 and 5 positions each."""
    torch_mod()
    prm = _prm(S)
    x = inputs.random_spectral_state(N, 3 + S, 70 + N, ora.kmax_retained(N), 8.0)
    progress(f"[lines] N={N} S={S} oracle right-hand side")
    ref = ora.rhs(x, prm)
    plan = make_plan(N, S, 32)
    assert plan.schedule_info(0)["x_lines"] == 4 and -(-N // 64) == positions
    set_params(plan, 0, prm)
    st, out = plan.new_state(), plan.new_state()
    plan.set_state(st, x, 0)
    plan.rhs(st, out, poisoned_workspace(plan))
    err = rel_l2(to_numpy(plan.get_state(out, 0)), ref)
    progress(f"[lines] N={N} S={S} FP32 rhs rel L2 {err:.2e}")
    assert err < 1e-5


@pytest.mark.parametrize("N,S,prec", [(24, 2, 64), (64, 1, 32), (128, 4, 32)])
def test_records_of_a_batch_are_those_of_single_slots(N, S, prec):
    """Every slot's record, shell sums and moments, is bitwise that of the slot on a plan of its own:
    the order of summation does not depend on the batch."""
    torch = torch_mod()
    prms = [_prm(S, nu) for nu in (0.01, 0.02, 0.005)]
    plan = make_plan(N, S, prec, batch=3)
    st, ws = plan.new_state(), poisoned_workspace(plan)
    ys = [inputs.random_spectral_state(N, 3 + S, N + i, ora.kmax_retained(N), 0.2 * N, 0.1) for i in range(3)]
    for i in range(3):
        set_params(plan, i, prms[i])
        plan.set_state(st, ys[i], i)
    for flags in (psdns.SPECTRA_SHELLS, psdns.SPECTRA_SHELLS | psdns.SPECTRA_MOMENTS):
        got = plan.spectra_raw(st, ws, flags).cpu().numpy()
        for i in range(3):
            one = make_plan(N, S, prec)
            set_params(one, 0, prms[i])
            s1, w1 = one.new_state(), poisoned_workspace(one)
            one.set_state(s1, ys[i], 0)
            ref = one.spectra_raw(s1, w1, flags).cpu().numpy()[0]
            assert np.array_equal(got[i], ref, equal_nan=True)
    torch.cuda.synchronize()


@pytest.mark.timeout(300)
def test_shell_table_beyond_64_kb():
    """1024^3 with four scalars: 592 shells of 14 sums, 66 304 bytes of LDS per wavefront.  The state is
    white noise (the sums need no symmetry), the reference an FP64 sum per shell with torch."""
    torch = torch_mod()
    N, S = 1024, 4
    plan = make_plan(N, S, 32)
    set_params(plan, 0, _prm(S, 3e-4))
    K, M, PX = plan.info.k_max, plan.info.m, plan.info.kx_pitch
    ns = int(plan.info.n_shells)
    assert ns * (2 + 3 * S) * 8 > 65536
    st, ws = plan.new_state(), plan.new_workspace()
    y = st.view(torch.float32).view(3 + S, M, M, PX, 2)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    for f in y:
        f.normal_(generator=gen)
    progress("[lines] 1024^3 S=4 shell sums")
    got = plan.spectra_raw(st, ws, psdns.SPECTRA_SHELLS)[0].cpu().numpy()
    k = torch.arange(M, device="cuda")
    k = torch.where(k <= K, k, k - M)
    kx = torch.arange(K + 1, device="cuda")
    w = torch.where(kx == 0, 1.0, 2.0).double()
    ref = torch.zeros((1 + S, ns), dtype=torch.float64, device="cuda")
    diss = torch.zeros((), dtype=torch.float64, device="cuda")
    # integer k^2 and FP64 roots: nint(|k|) is exact, |k| is never a half
    for z in range(M):
        k2 = k[z] ** 2 + k[:, None] ** 2 + kx[None, :] ** 2
        shell = torch.round(torch.sqrt(k2.double())).long().reshape(-1)
        e = y[:, z, :, :K + 1].double().square().sum(-1) * w  # field, ky, kx
        u = y[:3, z, :, :K + 1].double()
        ku = (kx[None, :, None] * u[0] + k[:, None, None] * u[1] + k[z] * u[2]).square().sum(-1) * w
        uu = e[:3].sum(0)
        diss += (k2 * uu + ku).sum()
        for q, f in enumerate([uu] + list(e[3:])):
            ref[q].index_add_(0, shell, 0.5 * f.reshape(-1))
    ref = (ref / float(N) ** 6).cpu().numpy()
    eps = 3e-4 * float(diss) / float(N) ** 6
    # positive FP64 terms, up to 4e6 in a shell and 1.6e8 in all, added in other orders
    assert np.allclose(got[:ns * (1 + S)].reshape(1 + S, ns), ref, rtol=1e-11)
    assert abs(got[ns * (1 + S) + 1] - eps) < 1e-11 * eps
    progress("[lines] 1024^3 S=4 shell sums agree")
