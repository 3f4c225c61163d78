"""Mixed-precision steps of large systems (more than 512 MiB of states, the real-space form): the states that a
step returns do not depend on what else it returns, the adjoint reverses them in the same form, and observables
and adjoints agree with FP64."""
import numpy as np
import pytest

from paper_2506_21908_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_21908_amd import nct
    return torch, nct


# |z| E_max = 42 dt: product stages at dt = 0.05 for K <= 4, Horner stages at 0.04 and for K = 6
CASES = [((32, 32, 32), 1027, 4, 0.05, "", 3), ((12, 24, 24), 4871, 4, 0.04, "velocity", 0),
         ((96, 8, 8), 5471, 3, 0.05, "length", 0), ((8, 96, 96), 457, 6, 0.05, "", 0),
         ((8, 64, 64), 1025, 4, 0.05, "velocity", 2), ((64, 48, 48), 229, 1, 0.05, "", 0)]


def _setup(torch, n, S, K, dt, laser, nk):
    w = I.make_system(n=n, L=tuple(0.42 * v for v in n), nstates=2, natoms=1, case=160, dt=dt, taylor_order=K,
                      bfield=I.BField(B0=(0.01, -0.02, 0.03), pulses=I.circular_pulses([0.1], [0.7], 0.05, 0.2)),
                      r_sphere=1.6, laser=[I.LaserPulse(A=0.02, omega=0.3, t0=0.0, tau=5.0)] if laser else None)
    if laser:
        w.laser_gauge = laser
    if nk:
        k = np.random.default_rng(8).uniform(-0.3, 0.3, (nk, 3))
        w.kvec = k[np.minimum(np.arange(S) * nk // (S - 5), nk - 1)]  # runs of unequal length
    w.nstates, w.occ = S, np.full(S, 2.0 / S)
    assert 2 * S * np.prod(n) * 8 > 512 * 2 ** 20
    psi = torch.randn((S, 2) + n, dtype=torch.complex64, generator=torch.Generator("cuda").manual_seed(9), device="cuda")
    psi /= torch.sqrt((psi.real ** 2 + psi.imag ** 2).sum(dim=(1, 2, 3, 4), keepdim=True) * 0.42 ** 3)
    psi[:, 1] *= 0.5  # a net moment
    return w, psi


@pytest.mark.parametrize("n,S,K,dt,laser,nk", CASES)
def test_states_do_not_depend_on_the_outputs(gpu, n, S, K, dt, laser, nk):
    """The same bits with and without observables and a tape; observables against the FP64 step."""
    torch, nct = gpu
    print(f"[case] outputs n={n} S={S} K={K} dt={dt} laser={laser!r} nk={nk}", flush=True)
    w, psi0 = _setup(torch, n, S, K, dt, laser, nk)
    s = nct.system_from_workload(w, precision=nct.NCT_FP32_MIXED, tape_steps=1)
    s.set_watchdog(0.0)
    got = []
    for obs, tape in ((False, False), (True, False), (False, True)):
        psi = psi0.clone()
        rows = s.step(psi, 0.3, 1, obs=obs, tape=tape)
        got.append((psi, rows))
    s.close()
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][0], got[2][0])
    d = nct.system_from_workload(w)
    d.set_watchdog(0.0)
    x = psi0.to(torch.complex128)
    ref = d.step(x, 0.3, 1, obs=True)
    d.close()
    # FP32 rounding of two exponentials, relative to the largest entry
    assert float((got[0][0] - x).abs().max() / x.abs().max()) < 1e-5
    # sums over all states of quantities that carry 1e-6 at most
    err = np.abs(got[1][1][0, 1:12] - ref[0, 1:12]) / np.maximum(np.abs(ref[0, 1:12]), 1e-3 * np.abs(ref[0, 1:12]).max())
    print(f"[case]   observables {err.max():.1e}", flush=True)
    assert err.max() < 1e-5


@pytest.mark.parametrize("n,S,K,dt,laser,nk,frozen",
                         [c + (False,) for c in CASES] + [c + (True,) for c in CASES if not c[4] and not c[5]])
def test_adjoint_in_the_form_of_the_step(gpu, n, S, K, dt, laser, nk, frozen):
    """Taped and recomputed adjoint steps give the same bits, and agree with FP64 (lambda to the FP32 rounding of
    the six exponentials, 2-norm bar 1e-5; dL/dB, sums of FP32 products, to 1e-4)."""
    torch, nct = gpu
    print(f"[case] adjoint n={n} S={S} K={K} dt={dt} laser={laser!r} nk={nk} frozen={frozen}", flush=True)
    w, psi0 = _setup(torch, n, S, K, dt, laser, nk)
    F = None
    if frozen:
        F = torch.rand((4,) + n, dtype=torch.float64, generator=torch.Generator("cuda").manual_seed(2), device="cuda") - 0.5
    out = []
    for prec in (nct.NCT_FP32_MIXED, nct.NCT_FP64):
        s = nct.system_from_workload(w, precision=prec, tape_steps=1 if prec == nct.NCT_FP32_MIXED else 0)
        s.set_watchdog(0.0)
        if frozen:
            s.set_potentials(fields=F)
        p0 = psi0 if prec == nct.NCT_FP32_MIXED else psi0.to(torch.complex128)
        lam1, lam = torch.empty_like(p0), torch.empty_like(p0)
        s.magnetization_seed(p0, (0.3, -0.5, 0.8), lam1)
        dB = s.backward_step(-1, p0, 0.3, lam1, lam)
        if prec == nct.NCT_FP32_MIXED:
            psi, lam2 = p0.clone(), torch.empty_like(p0)
            s.step(psi, 0.3, 1, tape=True)
            dB2 = s.backward_step(0, None, 0.3, lam1, lam2)
            assert torch.equal(lam, lam2) and np.array_equal(dB, dB2)
            del psi, lam2
        out.append((lam, dB))
        s.close()
    (a, da), (b, db) = out
    num = sum(float((a[i:i + 64].to(torch.complex128) - b[i:i + 64]).abs().square().sum()) for i in range(0, S, 64))
    den = sum(float(b[i:i + 64].abs().square().sum()) for i in range(0, S, 64))
    err, eb = (num / den) ** 0.5, 0.0 if frozen else np.abs(da - db).max() / np.abs(db).max()
    print(f"[case]   lambda {err:.1e} dB {eb:.1e}", flush=True)
    assert err < 1e-5 and eb < 1e-4
