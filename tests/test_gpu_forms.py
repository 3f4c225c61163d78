"""Schedules and exponential forms in combinations that small systems do not reach: state groups with a second
stream each, mixed-precision applications at k-points, and adjoints in product stages.

Product stages start at |z| E_max = 2.05 (+ 0.1 per order above 4); with h = 0.42 bohr E_max = 83.9, so a step of
0.05 has 2.10 and one of 0.048 has 2.01.  Bars are those of the same comparisons on small systems: bit for
bit, 1e-10 for the dot products, 1e-8 for gradients, 1e-5 for mixed applications."""
import numpy as np
import pytest

from oracle import nct_oracle as O
from paper_2506_21908_amd import inputs as I
from parity_metrics import max_rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_21908_amd import nct
    return torch, nct


# states above 32 MiB (FP64) and 64 MiB (mixed): the projector chain of each group has a stream of its own
@pytest.mark.parametrize("n,S,prec,laser,nk", [((32, 32, 32), 41, 0, "", 0), ((32, 32, 32), 41, 0, "", 3),
                                               ((32, 32, 32), 41, 0, "velocity", 0), ((24, 24, 24), 79, 0, "velocity", 4),
                                               ((32, 32, 32), 133, 1, "velocity", 3), ((32, 32, 32), 133, 1, "", 0),
                                               ((32, 32, 32), 1029, 1, "velocity", 3)])
def test_overlap_groups_with_streams_of_their_own_bitwise(gpu, n, S, prec, laser, nk):
    torch, nct = gpu
    print(f"[case] groups n={n} S={S} prec={prec} laser={laser!r} nk={nk}", flush=True)
    assert 2 * S * np.prod(n) * (8 if prec else 16) > (64 if prec else 32) * 2 ** 20
    w = I.make_system(n=n, L=tuple(0.42 * v for v in n), nstates=4, natoms=2, case=170, min_sep=3.0, r_sphere=2.4,
                      bfield=I.BField(pulses=I.circular_pulses([0.1], [0.5], 0.05, 0.1)),
                      laser=[I.LaserPulse(A=0.2, omega=0.3, t0=0.1, tau=1.0)] if laser else None)
    if laser:
        w.laser_gauge = laser
    psi0 = nct.states_to_device(w.psi0, prec)
    psi0 = psi0[torch.arange(S) % 4] * torch.exp(1j * torch.arange(S, device="cuda"))[:, None, None, None, None].to(psi0.dtype)
    w.nstates, w.occ = S, np.full(S, 4.0 / S)
    if nk:
        w.kvec = np.random.default_rng(2).uniform(-0.3, 0.3, (nk, 3))[np.minimum(np.arange(S) * nk // (S - 6), nk - 1)]
    out = []
    for ov in (False, True):
        s = nct.system_from_workload(w, precision=prec, overlap=ov)
        s.set_watchdog(0.0)
        psi = psi0.clone()
        obs = s.step(psi, 0.0, 2, obs=True)
        out.append((psi, obs))
        s.close()
    assert torch.equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1], out[1][1])
    assert bool(torch.isfinite(torch.view_as_real(out[0][0])).all())


@pytest.mark.parametrize("n,S,nk,prec", [((16, 12, 16), 7, 3, 1), ((12, 24, 24), 17, 4, 1), ((16, 12, 16), 7, 3, 0),
                                         ((8, 64, 64), 5, 2, 1), ((16, 48, 48), 3, 3, 1)])
def test_application_with_uneven_runs_of_vectors(gpu, n, S, nk, prec):
    """H_k psi in real space, both precisions, an odd number of states in runs of unequal length."""
    torch, nct = gpu
    print(f"[case] H_k n={n} S={S} nk={nk} prec={prec}", flush=True)
    L = tuple(0.5 * v for v in n)
    w = I.make_system(n=n, L=L, nstates=S, natoms=2, case=171, min_sep=2.0, r_sphere=0.45 * min(L))
    w.kvec = (np.random.default_rng(3).uniform(-1.0, 1.0, (nk, 3)) * np.pi / np.array(L))[
        np.minimum(np.arange(S) * nk // max(S - 2, 1), nk - 1)]
    F = np.random.default_rng(7).uniform(-0.4, 0.4, (4,) + n)
    sysd = O.system_from_workload(w)
    ref = (O.kinetic(w.psi0, sysd.grid, w.kvec) + O.apply_local(w.psi0, F[0], F[1:])
           + O.apply_nonlocal(w.psi0, sysd.projs, sysd.grid, w.kvec))
    s = nct.system_from_workload(w, precision=prec)
    s.set_potentials(fields=torch.from_numpy(F).cuda())
    psi = nct.states_to_device(w.psi0, prec)
    hpsi = torch.empty_like(psi)
    s.apply_hamiltonian(psi, hpsi, 0.0)
    assert max_rel(hpsi.cpu().numpy(), ref) < (1e-5 if prec else 1e-12)


def _system(K, dt, **kw):
    return I.make_system(n=(12, 12, 12), L=(5.04,) * 3, nstates=4, natoms=1, case=172, full_spinors=False, dt=dt,
                         taylor_order=K, r_sphere=2.0, **kw)


@pytest.mark.parametrize("K,dt,frozen", [(4, 0.05, False), (4, 0.05, True), (4, 0.048, False), (1, 0.05, False),
                                         (2, 0.05, False), (3, 0.05, False), (3, 0.05, True), (6, 0.056, False),
                                         (1, 0.05, True), (12, 0.07, False)])
def test_adjoint_dot_product_in_product_stages(gpu, K, dt, frozen):
    """Re<lam_n, dpsi_n> = Re<lam_{n+1}, J dpsi_n> and dL/dB against the oracle's tangent-linear step; taped and
    recomputed adjoints bit for bit."""
    torch, nct = gpu
    print(f"[case] adjoint K={K} dt={dt} frozen={frozen}", flush=True)
    w = _system(K, dt, bfield=I.BField(B0=(0.01, 0.0, 0.02), pulses=I.circular_pulses([0.1], [0.7], 0.05, 0.2)))
    sysd = O.system_from_workload(w)
    t_n = 0.1
    rng = np.random.default_rng(1)
    lam1, dpsi = (rng.standard_normal(w.psi0.shape) + 1j * rng.standard_normal(w.psi0.shape) for _ in range(2))
    s = nct.system_from_workload(w, tape_steps=1)
    s.set_watchdog(0.0)
    if frozen:
        F = rng.uniform(-0.3, 0.3, (4,) + w.n)
        s.set_potentials(fields=torch.from_numpy(F).cuda())
        H = lambda x: (O.kinetic(x, sysd.grid) + O.apply_local(x, F[0], F[1:])
                       + O.apply_nonlocal(x, sysd.projs, sysd.grid))
        Z = lambda x: np.zeros_like(x)
        phi, dphi = O._taylor_jvp(H, Z, w.psi0, dpsi, 0.5 * dt, K)
        _, dnext = O._taylor_jvp(H, Z, phi, dphi, 0.5 * dt, K)
    else:
        _, dnext = O.etrs_step_jvp(sysd, w.psi0, dpsi, t_n, np.zeros(3), np.zeros(3))
    psi = nct.states_to_device(w.psi0)
    lam_in = nct.states_to_device(lam1)
    lam_out = torch.empty_like(lam_in)
    dLdB = s.backward_step(-1, psi, t_n, lam_in, lam_out)
    lhs, rhs = (float(np.real(np.vdot(a, b))) for a, b in ((lam_out.cpu().numpy(), dpsi), (lam1, dnext)))
    assert abs(lhs - rhs) < 1e-10 * np.linalg.norm(lam1) * np.linalg.norm(dpsi)
    if not frozen:
        for j in range(6):
            e = np.zeros(3)
            e[j % 3] = 1.0
            _, dn2 = O.etrs_step_jvp(sysd, w.psi0, np.zeros_like(dpsi), t_n, *((e, np.zeros(3)) if j < 3 else (np.zeros(3), e)))
            ref = float(np.real(np.vdot(lam1, dn2)))
            assert abs(dLdB[j] - ref) < 1e-10 * max(abs(ref), 1e-3), (j, dLdB[j], ref)
    psi2 = nct.states_to_device(w.psi0)
    s.step(psi2, t_n, 1, tape=True)
    lam_out2 = torch.empty_like(lam_in)
    dLdB2 = s.backward_step(0, None, t_n, lam_in, lam_out2)
    assert torch.equal(lam_out, lam_out2)
    assert np.array_equal(dLdB, dLdB2)


@pytest.mark.parametrize("nk", [0, 2])
def test_gradient_schedules_in_product_stages(gpu, nk):
    """Taped and two-level recomputed pulse gradients against the oracle's forward mode, at Gamma and with
    k-points."""
    torch, nct = gpu
    print(f"[case] gradient nk={nk}", flush=True)
    pulses = I.circular_pulses([0.1, 0.25], [0.5, 1.0], 0.05, 0.15)
    w = _system(4, 0.05, bfield=I.BField(pulses=pulses))
    if nk:
        w.kvec = np.repeat(np.random.default_rng(5).uniform(-0.3, 0.3, (nk, 3)), 4 // nk, axis=0)
        w.occ = np.full(4, 0.5)
    nsteps = 9
    g_ref = O.mz_gradient_tangent_linear(O.system_from_workload(w), w.psi0, nsteps)
    grads = []
    for tape in (4, 0):
        s = nct.system_from_workload(w, tape_steps=tape)
        theta = torch.tensor([p.A for p in pulses] + [p.omega for p in pulses], dtype=torch.float64, requires_grad=True)
        L = nct.pulse_mz(theta, s, nct.states_to_device(w.psi0), pulses, nsteps, 4, checkpoint_on_host=(tape == 0),
                         sub_every=2)
        L.backward()
        grads.append(theta.grad.numpy())
        s.close()
    scale = np.max(np.abs(g_ref))
    assert np.allclose(grads[0], g_ref, rtol=1e-8, atol=1e-12 * scale)
    assert np.allclose(grads[1], g_ref, rtol=1e-8, atol=1e-12 * scale)
    assert np.allclose(grads[0], grads[1], rtol=1e-12, atol=1e-14 * scale)
