"""A state without a value (NaN) that no other state reads leaves the others'
solution alone: re-centring goes on, so they reach a tolerance far below the
FP32 resolution of V.  Rows of constant length: V in LDS, the band window.
(General CSR rows turn a policy's NaN into +inf, which ends re-centring.)"""
import numpy as np
import pytest
import torch

import oracle
from paper_2110_02901_amd import binding as mb
from paper_2110_02901_amd import inputs

from gpu_util import csr_case, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,band,window", [(8, None, -1), (8, 40, 0)])
def test_other_states_converge(k, band, window):
    n, m, gamma, tol = 700, 3, 0.95, 1e-10
    rp, col, val, c = inputs.csr_mdp(n, m, k, 1.0, 12, band=band)
    col = np.where(col == 0, 1, col).astype(np.int32)
    col[rp[0]:rp[m]] = 0  # state 0 leads to itself, no other state to it
    h, mdp = csr_case(rp, col, val, c, gamma)
    mb.mdp_set_tuning(h, band_window=window)
    V = torch.zeros(n, device=dev())
    V[0] = float("nan")
    V64 = torch.zeros(n, dtype=torch.float64, device=dev())
    pol = torch.zeros(n, dtype=torch.int32, device=dev())
    st = mb.mpi_solve(h, V, pol, 5, n // 5, 3, mb.workspace(h, n // 5), tol_dv=tol, max_outer=400,
                      V64_out=V64)
    assert st["converged"] and st["recentrings"] > 0
    Vs, mu, _ = oracle.policy_iteration(mdp)
    assert float(np.max(np.abs(V64.cpu().numpy()[1:] - Vs[1:]))) <= tol / (1 - gamma)
    assert np.array_equal(pol.cpu().numpy()[1:], mu[1:])
