"""Rounding of the time step on smooth states, where the Taylor terms are small beside the state.

Reference: the same truncated series in long double (FP64) or FP64 (FP32-mixed).  Bar: two unit roundoffs u of the
state's precision in relative 2-norm.  A step is two exponentials; each may round the state three times
(column pass, plane pass, projector rows) with an rms of 0.42 u, which makes sqrt(6) 0.42 u = 1.0 u, and the
transforms' own noise, eps_FFT |z| E_max with eps_FFT = 0.4 u per stage, adds sqrt(2) 0.4 u 1.3 = 0.7 u at
|z| E_max = 1.3.  A form that rounds the state in each of K = 12 stages makes sqrt(6 12) 0.42 u = 3.6 u.
"""
import numpy as np
import pytest
import scipy.fft

pytestmark = pytest.mark.gpu

H = 0.42
EMAX = 1.5 * (np.pi / H) ** 2


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_21908_amd import nct
    return torch, nct


def smooth_inputs(n, S, seed):
    rs = np.random.default_rng(seed)
    g = [2 * np.pi * np.fft.fftfreq(v, d=H) for v in n]
    g2 = (g[0] ** 2)[:, None, None] + (g[1] ** 2)[None, :, None] + (g[2] ** 2)[None, None, :]
    filt = np.exp(-0.5 * g2)
    z = np.fft.ifftn(np.fft.fftn(rs.standard_normal((S, 2) + n) + 1j * rs.standard_normal((S, 2) + n),
                                 axes=(2, 3, 4)) * filt, axes=(2, 3, 4))
    z /= np.sqrt((np.abs(z) ** 2).sum(axis=(1, 2, 3, 4), keepdims=True) * H ** 3)
    F = np.fft.ifftn(np.fft.fftn(rs.standard_normal((4,) + n), axes=(1, 2, 3)) * filt, axes=(1, 2, 3)).real
    F *= np.array([2.0, 0.3, 0.3, 0.3])[:, None, None, None] / np.abs(F).max()
    return z, F


def frozen_step(psi, F, n, K, dt, real, cplx):
    """Two exponentials T_K(-i dt/2 H) in fixed fields, in the given precision."""
    pi = real("3.14159265358979323846264338327950288")
    g2 = 0
    for d in range(3):
        k = np.arange(n[d])
        k = np.where(k < (n[d] + 1) // 2, k, k - n[d]).astype(real)
        g2 = g2 + ((2 * pi * k / (real(H) * n[d])) ** 2).reshape([-1 if e == d else 1 for e in range(3)])
    v, bx, by, bz = F.astype(real)

    def apply(p):
        o = scipy.fft.ifftn(scipy.fft.fftn(p, axes=(2, 3, 4)) * (g2 / 2), axes=(2, 3, 4))
        u, d = p[:, 0], p[:, 1]
        o[:, 0] += (v + bz) * u + (bx - 1j * by) * d
        o[:, 1] += (bx + 1j * by) * u + (v - bz) * d
        return o

    p = psi.astype(cplx)
    for _ in range(2):
        term = out = p
        for k in range(1, K + 1):
            term = (cplx(-0.5j) * real(dt) / k) * apply(term)
            out = out + term
        p = out
    return p


def gpu_step(torch, nct, psi, F, n, K, dt, precision):
    s = nct.System(n, tuple(H * v for v in n), psi.shape[0], dt=dt, taylor_order=K, hartree=0, xc=0,
                   precision=precision)
    s.set_potentials(fields=torch.from_numpy(F).cuda())
    s.set_watchdog(0.0)
    x = torch.from_numpy(psi.astype(np.complex64 if precision == nct.NCT_FP32_MIXED else np.complex128)).cuda()
    s.step(x, 0.0, 1)
    out = x.cpu().numpy()
    s.close()
    return out


@pytest.mark.parametrize("K", [4, 8, 12])
def test_step_fp64_rounding_on_smooth_states(gpu, K):
    torch, nct = gpu
    n, dt = (16, 16, 16), 2 * 1.3 / EMAX
    print(f"[case] rounding FP64 K={K}", flush=True)
    psi, F = smooth_inputs(n, 2, 40)
    ref = frozen_step(psi, F, n, K, dt, np.longdouble, np.clongdouble)
    got = gpu_step(torch, nct, psi, F, n, K, dt, nct.NCT_FP64).astype(np.clongdouble)
    err = float(np.sqrt((np.abs(got - ref) ** 2).sum() / (np.abs(ref) ** 2).sum()))
    print(f"[case]   {err:.2e}", flush=True)
    assert err < 2 * 2.0 ** -53


@pytest.mark.parametrize("K", [4, 12])
def test_step_mixed_rounding_on_smooth_states(gpu, K):
    """Above 512 MiB of states, where FP32 steps take the real-space form."""
    torch, nct = gpu
    n, dt, S, C = (16, 16, 16), 2 * 1.3 / EMAX, 8208, 16
    print(f"[case] rounding mixed K={K}", flush=True)
    psi, F = smooth_inputs(n, C, 41)
    psi, F = psi.astype(np.complex64), F.astype(np.float32).astype(np.float64)
    ref = frozen_step(psi, F, n, K, dt, np.float64, np.complex128)
    got = gpu_step(torch, nct, np.tile(psi, (S // C, 1, 1, 1, 1)), F, n, K, dt, nct.NCT_FP32_MIXED)
    assert 2 * S * np.prod(n) * 8 > 512 * 2 ** 20
    err = float(np.sqrt((np.abs(got[-C:] - ref) ** 2).sum() / (np.abs(ref) ** 2).sum()))
    print(f"[case]   {err:.2e}", flush=True)
    assert err < 2 * 2.0 ** -24


def test_step_fp64_rounds_the_base_last(gpu):
    """Small |z| E_max: the Taylor base is added once per pass, after the small terms.  Two exponentials of two
    roundings each make sqrt(4) 0.42 u = 0.84 u, the transforms 0.28 u: 0.89 u in all (1.09 u with the base rounded
    twice in the column pass).  Bar: one unit roundoff."""
    torch, nct = gpu
    n, dt = (16, 16, 16), 2 * 0.5 / EMAX
    print("[case] rounding FP64, base last", flush=True)
    psi, F = smooth_inputs(n, 2, 42)
    ref = frozen_step(psi, F, n, 4, dt, np.longdouble, np.clongdouble)
    got = gpu_step(torch, nct, psi, F, n, 4, dt, nct.NCT_FP64).astype(np.clongdouble)
    err = float(np.sqrt((np.abs(got - ref) ** 2).sum() / (np.abs(ref) ** 2).sum()))
    print(f"[case]   {err:.2e}", flush=True)
    assert err < 2.0 ** -53


@pytest.mark.parametrize("K,ze", [(4, 2.2), (8, 2.6), (12, 3.0)])
def test_product_stages_round_the_base_twice(gpu, K, ze):
    """Product stages (|z| E_max beyond 2.05 + 0.1 (K - 4)) round w once with c (T_x + V) w and once with c T_yz w:
    sqrt(4 K) 0.39 u for two exponentials of K stages (0.39 u: the rms of a rounding in 2-norm over the spread
    of mantissas), the transforms' noise on smooth states well below.  Bar: a tenth more; a third rounding of
    w per stage makes sqrt(6 K) 0.39 u, 1.22 times."""
    torch, nct = gpu
    n, dt = (16, 16, 16), 2 * ze / EMAX
    print(f"[case] rounding FP64 product K={K}", flush=True)
    psi, F = smooth_inputs(n, 2, 43)
    ref = frozen_step(psi, F, n, K, dt, np.longdouble, np.clongdouble)
    got = gpu_step(torch, nct, psi, F, n, K, dt, nct.NCT_FP64).astype(np.clongdouble)
    err = float(np.sqrt((np.abs(got - ref) ** 2).sum() / (np.abs(ref) ** 2).sum()))
    print(f"[case]   {err:.2e}", flush=True)
    assert err < 1.1 * 0.39 * np.sqrt(4 * K) * 2.0 ** -53
