"""Overlap and triangular change of basis of the ground state at the edges of their tiles (16, 32 and 64
states), against numpy's Cholesky factor in FP64.

Bars: sums of 2N = 1536 products and a factor of condition below ten, 1e-12 in FP64; mixed precision
stores the states in FP32 (6e-8 of a value): 1e-6 of the largest.
"""
import numpy as np
import pytest

from paper_2506_21908_amd import inputs as I
from parity_metrics import max_rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("S,nk", [(1, 0), (15, 0), (17, 0), (32, 0), (33, 0), (65, 0), (130, 0), (51, 3)])
def test_orthonormalisation(S, nk, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_21908_amd import nct
    print(f"[case] orthonormalise S={S} nk={nk} prec={prec}", flush=True)
    n = (12, 8, 8)
    w = I.make_system(n=n, L=(6.0, 4.0, 4.0), nstates=2, case=150)
    w.nstates, w.occ = S, np.ones(S)
    if nk:
        w.kvec = np.repeat(np.linspace(-0.2, 0.3, 3 * nk).reshape(nk, 3), S // nk, axis=0)
    rng = np.random.default_rng(S)
    A = rng.standard_normal((S, 2 * 768)) + 1j * rng.standard_normal((S, 2 * 768))
    psi = nct.states_to_device(A.reshape((S, 2) + n), prec)
    A = psi.cpu().numpy().astype(np.complex128).reshape(S, -1)
    dV = 96.0 / 768
    ref = np.empty_like(A)
    run = S // max(nk, 1)
    for i in range(0, S, run):
        X = A[i:i + run]
        M = np.linalg.inv(np.linalg.cholesky(dV * X.conj() @ X.T)).conj().T
        ref[i:i + run] = M.T @ X
    s = nct.system_from_workload(w, precision=prec)
    s.ground_state(psi, 0, 0.01)
    assert max_rel(psi.cpu().numpy().reshape(S, -1), ref) < (1e-6 if prec else 1e-12)
