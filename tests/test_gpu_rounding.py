"""Rounding of a right-hand side: FP32 against the FP64 plan on the same (FP32-rounded) field, FP64
against an evaluation in extended precision on the CPU.  The bars are what the first kernels of
the library measured on these fields (products of every input by its twiddle, even radices first),
with 2% for the third digit and, in FP64, none: a faster form may not round more."""
import numpy as np
import pytest
import scipy.fft as sf

from paper_2012_04838_amd import inputs, psdns
from tests.gpu_helpers import make_plan, progress, torch_mod

pytestmark = pytest.mark.gpu


def _turbulence_like(torch, N, seed):
    """[4][N][N][N/2+1] in complex64: u solenoidal, E(k) ~ k^4 (k^2 + 9)^(-17/6) exp(-5 (k/K)^2), and a
    scalar of the same shape."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    K = (N - 1) // 3
    k = torch.arange(N, device="cuda")
    k = torch.where(k <= N // 2, k, k - N)
    kx = torch.arange(N // 2 + 1, device="cuda")
    kz, ky = k[:, None, None], k[None, :, None]
    k2 = (kz ** 2 + ky ** 2 + kx ** 2).float()
    amp = torch.sqrt(k2) * (k2 + 9) ** (-17 / 12) * torch.exp(-2.5 / K ** 2 * k2)
    f = torch.empty((4, N, N, N // 2 + 1), dtype=torch.complex64, device="cuda")
    flip = (-torch.arange(N, device="cuda")) % N
    for q in f:
        torch.view_as_real(q).normal_(generator=gen)
        q[:, :, 0] = (q[:, :, 0] + q[:, :, 0][flip][:, flip].conj()) / 2 ** 0.5
        q.mul_(amp)
    div = (f[0] * kx + f[1] * ky + f[2] * kz) / k2.clamp(min=1)
    for q, kk in zip(f, (kx, ky, kz)):
        q.sub_(div * kk)
    return f * float(N) ** 3


def _plan(N, prec, dealias=0):
    plan = make_plan(N, 1, prec, dealias=dealias)
    plan.set_slot(0, nu=1e-3, power=0.0, schmidt=[0.7], mean_grad=[[0, 1, 0]])
    return plan


def _fp32_error(N, dealias):
    torch = torch_mod()
    acc = []
    for seed in range(5 if N <= 64 else 3 if N <= 128 else 1):
        f, out = _turbulence_like(torch, N, seed), {}
        for prec in (64, 32):
            plan = _plan(N, prec, dealias)
            st, rhs = plan.new_state(), plan.new_state()
            plan.set_state(st, f, 0)
            plan.rhs(st, rhs, plan.new_workspace())
            out[prec] = rhs.view(torch.float32 if prec == 32 else torch.float64).double()
        acc.append(float((out[32] - out[64]).norm() / out[64].norm()))
    return float(np.sqrt(np.mean(np.square(acc))))


# mixed radix, 2/3 rule and phase shift (None: not measured)
@pytest.mark.parametrize("N,cube,sphere", [(24, 2.154e-7, 2.202e-7), (40, 2.906e-7, 2.665e-7), (56, 2.391e-7, 2.372e-7),
                                           (70, 2.695e-7, 2.448e-7), (98, 3.039e-7, 2.941e-7),
                                           (104, 2.917e-7, 2.673e-7), (150, 3.628e-7, 3.389e-7),
                                           (260, 4.549e-7, None), (520, 6.303e-7, None)])
def test_fp32_rounding_of_the_general_kernels(N, cube, sphere):
    for dealias, bar in ((psdns.DEALIAS_TWO_THIRDS, cube), (psdns.DEALIAS_PHASE_SPHERE, sphere)):
        if bar is None:
            continue
        err = _fp32_error(N, dealias)
        progress(f"[rounding] N={N} dealias={dealias} FP32 {err:.3e} (bar {bar:.3e})")
        assert err < 1.02 * bar


@pytest.mark.parametrize("N,cube,sphere", [(8, 8.732e-8, 1.138e-7), (16, 2.021e-7, 2.506e-7), (32, 2.537e-7, 2.704e-7),
                                           (64, 2.908e-7, 2.853e-7), (128, 3.555e-7, 3.415e-7),
                                           (256, 4.604e-7, 4.285e-7), (512, 6.550e-7, None)])
def test_fp32_rounding_of_the_tuned_kernels(N, cube, sphere):
    for dealias, bar in ((psdns.DEALIAS_TWO_THIRDS, cube), (psdns.DEALIAS_PHASE_SPHERE, sphere)):
        if bar is None:
            continue
        err = _fp32_error(N, dealias)
        progress(f"[rounding] N={N} dealias={dealias} FP32 {err:.3e} (bar {bar:.3e})")
        assert err < 1.02 * bar


def _rhs_extended(x, N, nu, sc):
    """dy/dt of Eqs. (7)-(8) without forcing, G = (0, 1, 0), in 80-bit floats."""
    L = np.longdouble
    K = (N - 1) // 3
    k = np.fft.fftfreq(N, 1 / N).astype(int)
    kx, ky, kz = np.arange(N // 2 + 1)[None, None, :].astype(L), k[None, :, None].astype(L), k[:, None, None].astype(L)
    kk = (kx, ky, kz)
    m = (abs(kx) <= K) & (abs(ky) <= K) & (abs(kz) <= K)
    y = [np.where(m, f, 0).astype(np.clongdouble) for f in x]

    def phys(f):
        return sf.irfftn(f, s=(N,) * 3)

    def spec(f):
        return np.where(m, sf.rfftn(f), 0)

    u = [phys(f) for f in y[:3]]
    om = [phys(1j * (kk[a] * y[b] - kk[b] * y[a])) for a, b in ((1, 2), (2, 0), (0, 1))]
    c = [spec(u[a] * om[b] - u[b] * om[a]) for a, b in ((1, 2), (2, 0), (0, 1))]
    adv = spec(sum(u[d] * phys(1j * kk[d] * y[3]) for d in range(3)) + u[1])
    k2 = kx * kx + ky * ky + kz * kz
    on = k2 > 0
    div = (kx * c[0] + ky * c[1] + kz * c[2]) / np.where(on, k2, 1)
    out = [np.where(on, c[d] - kk[d] * div, 0) - nu * k2 * y[d] for d in range(3)]
    return np.array(out + [np.where(on, -adv, 0) - nu / sc * k2 * y[3]])


@pytest.mark.parametrize("N,bar", [(16, 4.68e-16), (32, 5.46e-16), (64, 6.87e-16)])
def test_fp64_rounding_against_extended_precision(N, bar):
    torch_mod()
    x = inputs.random_spectral_state(N, 4, 11 * N, (N - 1) // 3, 6.0)
    plan = make_plan(N, 1, 64)
    plan.set_slot(0, nu=0.01, power=0.0, schmidt=[0.7], mean_grad=[[0, 1, 0]])
    st, out = plan.new_state(), plan.new_state()
    plan.set_state(st, x, 0)
    plan.rhs(st, out, plan.new_workspace())
    got = plan.get_state(out, 0).cpu().numpy().astype(np.clongdouble)
    # the slot's own FP64 parameters
    ref = _rhs_extended(x, N, np.longdouble(0.01), np.longdouble(0.7))
    err = float(np.sqrt((abs(got - ref) ** 2).sum() / (abs(ref) ** 2).sum()))
    progress(f"[rounding] N={N} FP64 {err:.3e} (bar {bar:.3e})")
    assert err < bar
