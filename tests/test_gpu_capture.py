"""H applications under HIP graph capture and the Bloch phase tables behind them: a system's first application can
be recorded (nothing is allocated during a call), and a recorded application in the velocity gauge keeps its own
A(t), whatever eager calls at other times or in the other gauge run between its replays.  Results are compared bit
for bit with eager applications on a second system."""
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


def _workload(n, S, kpoints, gauge):
    laser = [I.LaserPulse(A=0.5, omega=0.4, t0=1.0, tau=1.5)] if gauge else None
    w = I.make_system(n=n, L=tuple(0.5 * v for v in n), nstates=4, natoms=2, case=150, min_sep=2.5, r_sphere=2.4,
                      laser=laser)
    w.psi0 = np.resize(w.psi0, (S,) + w.psi0.shape[1:])
    w.nstates, w.occ = S, np.ones(S)
    if gauge:
        w.laser_gauge = gauge
    if kpoints:
        w.kvec = np.repeat(np.random.default_rng(3).uniform(-0.3, 0.3, (3, 3)), (S + 2) // 3, axis=0)[:S]
    return w


# (12^3 x 5: one stream; 32^3 x 40 FP64, 40 MiB: the projector chain on a second stream)
@pytest.mark.parametrize("n,S,prec,kpoints,gauge",
                         [((12, 12, 12), 5, 0, True, ""), ((12, 12, 12), 5, 0, False, "velocity"),
                          ((12, 12, 12), 5, 1, True, "velocity"), ((32, 32, 32), 40, 0, True, "velocity")])
def test_first_application_recorded_and_replayed(gpu, n, S, prec, kpoints, gauge):
    torch, nct = gpu
    print(f"[case] capture n={n} S={S} prec={prec} kpoints={kpoints} gauge={gauge!r}", flush=True)
    w = _workload(n, S, kpoints, gauge)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        eager = nct.system_from_workload(w, precision=prec, stream=st)
        s = nct.system_from_workload(w, precision=prec, stream=st)
        psi = nct.states_to_device(w.psi0, prec)
        rho = torch.empty((4,) + n, dtype=torch.float64, device="cuda")
        for x in (eager, s):
            x.density_magnetization(psi, 0.0, rho_v=rho, update_fields=True)
        want, other, out = torch.empty_like(psi), torch.empty_like(psi), torch.zeros_like(psi)
        eager.apply_hamiltonian(psi, want, 0.5)
        eager.apply_hamiltonian(psi, other, 2.0)
        st.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            s.apply_hamiltonian(psi, out, 0.5)
        for k in range(4):
            out.zero_()
            g.replay()
            st.synchronize()
            assert torch.equal(out, want), k
            s.apply_hamiltonian(psi, out, 2.0)  # eager, another time
            st.synchronize()
            assert torch.equal(out, other), k
            if k == 1 and gauge and kpoints:  # and the other gauge
                s.set_laser_gauge("length")
                s.apply_hamiltonian(psi, out, 2.0)
                s.set_laser_gauge("velocity")
        del g
    eager.close()
    s.close()


def test_changed_vectors_reach_later_applications(gpu):
    """Bloch vectors set again, in more runs than before, with and without the velocity gauge, and taken off."""
    torch, nct = gpu
    print("[case] vectors set again", flush=True)
    n, S = (12, 12, 12), 6
    w = _workload(n, S, False, "velocity")
    psi = nct.states_to_device(w.psi0)
    s = nct.system_from_workload(w)
    s.density_magnetization(psi, 0.0, update_fields=True)
    rng = np.random.default_rng(4)
    ks = [np.repeat(rng.uniform(-0.3, 0.3, (r, 3)), S // r, axis=0) for r in (2, 6, 1)] + [None]
    for kv in ks:
        for g in ("length", "velocity"):
            fresh = nct.system_from_workload(w)
            fresh.density_magnetization(psi, 0.0, update_fields=True)
            for x in (s, fresh):
                x.set_laser_gauge(g)
                x.set_kpoints(kv)
            a, b = torch.empty_like(psi), torch.empty_like(psi)
            s.apply_hamiltonian(psi, a, 0.7)
            fresh.apply_hamiltonian(psi, b, 0.7)
            assert torch.equal(a, b)
            fresh.close()
    s.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("gauge", ["length", "velocity"])
def test_recorded_application_follows_vectors(gpu, prec, gauge):
    """A recorded application replayed after the Bloch vectors were set again, in more runs and in fewer."""
    torch, nct = gpu
    print(f"[case] recorded, then vectors set again prec={prec} gauge={gauge}", flush=True)
    n, S = (12, 12, 12), 6
    w = _workload(n, S, False, "velocity")
    rng = np.random.default_rng(5)
    ks = [np.repeat(rng.uniform(-0.3, 0.3, (r, 3)), S // r, axis=0) for r in (2, 6, 1, 3)]
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        s, eager = (nct.system_from_workload(w, precision=prec, stream=st) for _ in range(2))
        psi = nct.states_to_device(w.psi0, prec)
        out, want = torch.zeros_like(psi), torch.empty_like(psi)
        for x in (s, eager):
            x.density_magnetization(psi, 0.0, update_fields=True)
            x.set_laser_gauge(gauge)
            x.set_kpoints(ks[0])
        st.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            s.apply_hamiltonian(psi, out, 0.5)
        for kv in ks + ks[:2]:
            s.set_kpoints(kv)
            eager.set_kpoints(kv)
            eager.apply_hamiltonian(psi, want, 0.5)
            out.zero_()
            g.replay()
            st.synchronize()
            assert torch.equal(out, want), len(np.unique(kv, axis=0))
        del g
    eager.close()
    s.close()
