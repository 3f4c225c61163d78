"""FP64 real-space form of the H application and product form of the exponential against the oracle.

Bars: 1e-12 of the largest entry for one H application (the bar of the other single applications: a few
roundings per transform stage, times the spread of the kinetic factors), 1e-12 for one step.
"""
import numpy as np
import pytest

from oracle import nct_oracle as O
from paper_2506_21908_amd import inputs as I
from parity_metrics import max_rel

pytestmark = pytest.mark.gpu

PLANES = [(8, 8), (12, 12), (16, 16), (24, 24), (32, 32), (48, 48), (64, 64), (96, 96),
          (8, 16), (16, 8), (12, 16), (16, 12), (16, 24), (24, 16)]
LINES = [8, 12, 16, 24, 32, 48, 64, 96]


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_21908_amd import nct
    return torch, nct


@pytest.mark.parametrize("k", range(len(PLANES)))
def test_apply_every_plane_with_overlapping_spheres(gpu, k):
    """Every built plane pair (partial waves, partial work items) with another column length, an odd
    number of states and projector spheres that overlap (several rows at one grid point)."""
    torch, nct = gpu
    ny, nz = PLANES[k]
    n = (LINES[(3 * k + 1) % len(LINES)] if ny * nz < 2000 else 8, ny, nz)
    L = tuple(0.5 * v for v in n)
    print(f"[case] apply n={n}", flush=True)
    w = I.make_system(n=n, L=L, nstates=3, case=70 + k, natoms=3, min_sep=0.2 * min(L), r_sphere=0.45 * min(L))
    F = np.random.default_rng(k).uniform(-0.5, 0.5, (4,) + n)
    sysd = O.system_from_workload(w)
    ref = (O.kinetic(w.psi0, sysd.grid) + O.apply_local(w.psi0, F[0], F[1:])
           + O.apply_nonlocal(w.psi0, sysd.projs, sysd.grid))
    s = nct.system_from_workload(w)
    s.set_potentials(fields=torch.from_numpy(F).cuda())
    psi = nct.states_to_device(w.psi0)
    hpsi = torch.empty_like(psi)
    s.apply_hamiltonian(psi, hpsi, 0.0)
    assert max_rel(hpsi.cpu().numpy(), ref) < 1e-12


# the product form starts where |z| E_max = 1.25, z = dt / 2: at h = 0.42 (E_max = 83.9) dt = 0.0298
@pytest.mark.parametrize("K,dt", [(4, 0.029), (4, 0.031), (1, 0.031), (2, 0.031), (3, 0.031), (5, 0.04),
                                  (8, 0.05), (12, 0.05), (13, 0.05)])
def test_step_both_forms(gpu, K, dt):
    """One step on either side of the rule that chooses Horner or product stages, odd and even orders."""
    torch, nct = gpu
    print(f"[case] step K={K} dt={dt}", flush=True)
    w = I.make_system(n=(12, 12, 12), L=(5.04,) * 3, nstates=6, natoms=1, case=90, dt=dt, taylor_order=K,
                      full_spinors=False, bfield=I.BField(B0=(0.01, -0.02, 0.03)), r_sphere=2.0)
    psi_ref, _ = O.run(O.system_from_workload(w), w.psi0, 1)
    s = nct.system_from_workload(w)
    s.set_watchdog(0.0)  # low orders do not conserve the norm
    psi = nct.states_to_device(w.psi0)
    s.step(psi, 0.0, 1)
    assert max_rel(psi.cpu().numpy(), psi_ref) < 1e-12


@pytest.mark.parametrize("S,natoms,nch,prec", [(1, 1, 1, 0), (17, 2, 2, 0), (33, 3, 5, 0), (1025, 8, 5, 0),
                                               (17, 2, 2, 1), (1025, 8, 3, 1)])
def test_projector_chain_splits(gpu, S, natoms, nch, prec):
    """Contraction and scatter over few and many (atom, states) pairs (shares of the row tiles, chunk
    lengths), 16 and 32 padded projectors, ragged states: the nonlocal term alone, with the kinetic part
    taken off by a second application at zero projector energy.  Mixed: FP32 sums of 64 products."""
    torch, nct = gpu
    print(f"[case] chain S={S} natoms={natoms} channels={nch} prec={prec}", flush=True)
    n, L = (8, 8, 8), (6.0,) * 3
    w = I.make_system(n=n, L=L, nstates=min(S, 40), case=110, natoms=natoms, min_sep=1.0)
    w.channels = w.channels[:nch]
    w.nstates, w.occ = S, np.ones(S)
    w.psi0 = np.resize(w.psi0, (S,) + w.psi0.shape[1:]) * np.linspace(0.5, 1.5, S)[:, None, None, None, None]
    sysd = O.system_from_workload(w)
    ref = O.apply_nonlocal(w.psi0, sysd.projs, sysd.grid)
    psi = nct.states_to_device(w.psi0, prec)
    out = []
    for scale in (1.0, 0.0):
        for c in w.channels:
            c.energy = c.energy if scale else 0.0
        s = nct.system_from_workload(w, precision=prec)
        s.set_potentials(fields=torch.zeros((4,) + n, dtype=torch.float64, device="cuda"))
        hpsi = torch.empty_like(psi)
        s.apply_hamiltonian(psi, hpsi, 0.0)
        out.append(hpsi.cpu().numpy().astype(np.complex128))
        s.close()
    assert max_rel(out[0] - out[1], ref) < (2e-5 if prec else 1e-11)


# Mixed precision: FP32 unit roundoff 6e-8, some 16 roundings on a point's way through the transforms and
# the sum of the terms, times a spread of kinetic factors of up to 4 against their mean: 4e-6, bar 1e-5.
@pytest.mark.parametrize("k", range(len(PLANES)))
def test_mixed_apply_every_plane_with_overlapping_spheres(gpu, k):
    """The same in mixed precision, every plane with another column length than above."""
    torch, nct = gpu
    ny, nz = PLANES[k]
    n = (LINES[(5 * k + 2) % len(LINES)] if ny * nz < 2000 else 12, ny, nz)
    L = tuple(0.5 * v for v in n)
    print(f"[case] mixed apply n={n}", flush=True)
    w = I.make_system(n=n, L=L, nstates=3, case=130 + k, natoms=3, min_sep=0.2 * min(L), r_sphere=0.45 * min(L))
    F = np.random.default_rng(k).uniform(-0.5, 0.5, (4,) + n)
    sysd = O.system_from_workload(w)
    ref = (O.kinetic(w.psi0, sysd.grid) + O.apply_local(w.psi0, F[0], F[1:])
           + O.apply_nonlocal(w.psi0, sysd.projs, sysd.grid))
    s = nct.system_from_workload(w, precision=nct.NCT_FP32_MIXED)
    s.set_potentials(fields=torch.from_numpy(F).cuda())
    psi = nct.states_to_device(w.psi0, nct.NCT_FP32_MIXED)
    hpsi = torch.empty_like(psi)
    s.apply_hamiltonian(psi, hpsi, 0.0)
    assert max_rel(hpsi.cpu().numpy(), ref) < 1e-5


@pytest.mark.parametrize("n,S,K,dt,laser", [((12, 12, 12), 19440, 4, 0.029, ""), ((96, 8, 8), 5470, 4, 0.05, "velocity"),
                                            ((12, 24, 24), 4870, 13, 0.05, "length"), ((8, 96, 96), 456, 5, 0.04, "")])
def test_mixed_step_of_large_states(gpu, n, S, K, dt, laser):
    """One mixed-precision step just above 512 MiB of states, where FP32 takes the real-space form, against
    the FP64 step: both exponential forms, shifted kinetic factors, ragged groups of states."""
    torch, nct = gpu
    print(f"[case] mixed step n={n} S={S} K={K} dt={dt} laser={laser!r}", flush=True)
    assert 2 * S * np.prod(n) * 8 > 512 * 2 ** 20
    w = I.make_system(n=n, L=tuple(0.42 * v for v in n), nstates=2, natoms=1, case=95, dt=dt, taylor_order=K,
                      bfield=I.BField(B0=(0.01, -0.02, 0.03)), r_sphere=1.6,
                      laser=[I.LaserPulse(A=0.02, omega=0.3, t0=0.0, tau=5.0)] if laser else None)
    if laser:
        w.laser_gauge = laser
    w.nstates, w.occ = S, np.full(S, 2.0 / S)
    psi = torch.randn((S, 2) + n, dtype=torch.complex64, generator=torch.Generator("cuda").manual_seed(5), device="cuda")
    psi /= float(torch.linalg.vector_norm(psi[0]) * np.sqrt(0.42 ** 3))
    out = []
    for p in (nct.NCT_FP64, nct.NCT_FP32_MIXED):
        x = psi.to(torch.complex128) if p == nct.NCT_FP64 else psi.clone()
        s = nct.system_from_workload(w, precision=p)
        s.set_watchdog(0.0)
        s.step(x, 0.0, 1)
        s.close()
        out.append(x)
    assert float((out[1] - out[0]).abs().max() / out[0].abs().max()) < 1e-5


@pytest.mark.parametrize("S,natoms,nch,prec,nk", [(2051, 1, 1, 0, 0), (2051, 3, 5, 0, 3), (2061, 8, 2, 0, 2),
                                                  (8195, 1, 5, 1, 0), (8195, 5, 1, 1, 3), (8209, 2, 3, 1, 2),
                                                  (37, 3, 5, 0, 3), (37, 3, 2, 1, 3)])
def test_projector_chain_with_coefficients_made_first(gpu, S, natoms, nch, prec, nk):
    """The chain on its own stream (states above 32 MiB FP64, 64 MiB mixed; the last two below): coefficients
    summed once, row tiles in pairs, 16 and 32 padded projectors, ragged states, Bloch phases in runs of unequal
    length.  The nonlocal term alone, as above."""
    torch, nct = gpu
    print(f"[case] chain, own stream S={S} natoms={natoms} channels={nch} prec={prec} nk={nk}", flush=True)
    n, L = (8, 8, 8), (6.0,) * 3
    assert S < 100 or 2 * S * 512 * (8 if prec else 16) > (64 if prec else 32) * 2 ** 20
    w = I.make_system(n=n, L=L, nstates=32, case=111, natoms=natoms, min_sep=1.0)
    w.channels = w.channels[:nch]
    w.nstates, w.occ = S, np.ones(S)
    w.psi0 = np.resize(w.psi0, (S,) + w.psi0.shape[1:]) * np.linspace(0.5, 1.5, S)[:, None, None, None, None]
    if nk:
        w.kvec = np.random.default_rng(6).uniform(-0.4, 0.4, (nk, 3))[np.minimum(np.arange(S) * nk // (S - 9), nk - 1)]
    sysd = O.system_from_workload(w)
    ref = O.apply_nonlocal(w.psi0, sysd.projs, sysd.grid, w.kvec if nk else None)
    psi = nct.states_to_device(w.psi0, prec)
    out = []
    for scale in (1.0, 0.0):
        for c in w.channels:
            c.energy = c.energy if scale else 0.0
        s = nct.system_from_workload(w, precision=prec)
        s.set_potentials(fields=torch.zeros((4,) + n, dtype=torch.float64, device="cuda"))
        hpsi = torch.empty_like(psi)
        s.apply_hamiltonian(psi, hpsi, 0.0)
        out.append(hpsi.cpu().numpy().astype(np.complex128))
        s.close()
    assert max_rel(out[0] - out[1], ref) < (2e-5 if prec else 1e-11)
