"""The resident-value kernel of dense MDPs (V in every workgroup's LDS, the
batch's values exchanged as tagged words) against the oracle, at the edges of
its tiles and dispatch: rows of a few values to several steps, remainders of
the 16-byte loads, one workgroup and all of them, batches of fewer positions
than workgroups (a state's rows split into parts), a short last batch, more
sweeps than one draw of the order covers, re-centring after every sweep.

Tolerance: a sweep's FP32 dot products are allowed SWEEP_RTOL * max|V| against
FP64 (the single-sweep tests' bound); T sweeps, each a contraction, at most T
times that.
"""
import numpy as np
import pytest
import torch

import oracle
from oracle import quantize as qz
from paper_2110_02901_amd import binding as mb
from paper_2110_02901_amd import inputs

from gpu_util import SWEEP_RTOL, dense_case, dev, run_sweep, up

pytestmark = pytest.mark.gpu


def stored_case(n, m, dtype, gamma, seed):
    """(handle, oracle MDP) of a random dense MDP stored in `dtype`."""
    P, c = inputs.dense_mdp(n, m, 0.5, seed, dtype=np.float32)
    if dtype == "f32":
        return dense_case(P, c, gamma)
    rows = P.reshape(n * m, n)
    q, s = mb.mdp_quantize_rows(up(rows), dtype)
    h = mb.mdp_create_dense_q(q.reshape(-1), dtype, s, up(c), gamma)
    q_ref, s_ref = qz.quantize_rows(rows, dtype)
    return h, oracle.DenseMDP(qz.dequantized(q_ref, s_ref, dtype).reshape(n, m, n), c, gamma)


def check_sweeps(h, mdp, b, T, seed=11):
    """T sweeps of vi_solve (no stop) from a seeded V against the oracle's."""
    n = mdp.n
    V0 = inputs.values(n, 3, 0.0, 5.0).astype(np.float32)
    V, V64 = up(V0), torch.zeros(n, dtype=torch.float64, device=dev())
    st = mb.vi_solve(h, V, b, seed, mb.workspace(h, b), tol_dv=-1.0, max_sweeps=T, V64_out=V64)
    assert st["sweeps"] == T
    ref = V0.astype(np.float64)
    for t in range(T):
        ref, _, dv = oracle.mb_sweep(mdp, ref, b, oracle.sweep_permutation(n, seed, t))
    tol = T * SWEEP_RTOL * float(np.max(np.abs(V0)))
    assert float(np.max(np.abs(V64.cpu().numpy() - ref))) <= tol
    assert abs(st["final_dv_inf"] - dv) <= tol


# rows of one partial step, one step, two, several; every remainder mod 4;
# b: one position, a few, one short last batch, all
@pytest.mark.parametrize("n,m,b", [
    (4, 3, 2), (5, 1, 5), (6, 2, 1), (63, 9, 10), (64, 4, 16), (257, 5, 13), (500, 6, 100),
    (511, 6, 64), (512, 33, 300), (1022, 7, 1022), (1025, 3, 7), (2050, 2, 2049), (3073, 17, 40),
])
def test_fp32_sweeps(n, m, b):
    h, mdp = stored_case(n, m, "f32", 0.9, 40 + n)
    assert mb.mdp_engine(h, b) == "dense"
    check_sweeps(h, mdp, b, 3)


@pytest.mark.parametrize("dtype,n,m,b", [
    ("bf16", 8, 3, 3), ("bf16", 504, 6, 100), ("bf16", 1032, 5, 33), ("bf16", 4104, 2, 700),
    ("fp8", 16, 2, 16), ("fp8", 496, 6, 100), ("fp8", 1040, 5, 33), ("fp8", 8208, 1, 900),
])
def test_stored_sweeps(dtype, n, m, b):
    h, mdp = stored_case(n, m, dtype, 0.9, 60 + n)
    check_sweeps(h, mdp, b, 3)


def test_streamed_table_with_a_tail():
    # 201 MB: read with non-temporal loads; n % 4 = 3
    h, mdp = stored_case(4099, 3, "f32", 0.95, 5)
    check_sweeps(h, mdp, 512, 2)
    run_sweep(h, mdp, inputs.values(4099, 4, 0.0, 3.0), 512, 7, 1,
              policy=inputs.policy(4099, 3, 8))


@pytest.mark.parametrize("n,b", [(64, 16), (300, 30), (700, 100)])
def test_order_beyond_one_draw(n, b):
    h, mdp = stored_case(n, 3, "f32", 0.5, 7)
    check_sweeps(h, mdp, b, 40)


@pytest.mark.parametrize("dtype,n", [("f32", 250), ("f32", 1027), ("bf16", 520), ("fp8", 1040)])
def test_recentring_after_every_sweep(dtype, n):
    h, mdp = stored_case(n, 4, dtype, 0.9, 90 + n)
    mb.mdp_set_tuning(h, recentre_every=1, recentre_force=True)
    check_sweeps(h, mdp, n // 3, 6)


@pytest.mark.parametrize("dtype,n,m,b", [("f32", 70, 3, 9), ("f32", 514, 5, 60), ("f32", 2311, 3, 97),
                                         ("bf16", 1000, 4, 125), ("fp8", 1008, 4, 1008)])
def test_mpi_to_tolerance(dtype, n, m, b):
    gamma, tol = 0.9, 1e-9
    h, mdp = stored_case(n, m, dtype, gamma, 20 + n)
    V = torch.zeros(n, device=dev())
    V64 = torch.zeros(n, dtype=torch.float64, device=dev())
    pol = torch.zeros(n, dtype=torch.int32, device=dev())
    st = mb.mpi_solve(h, V, pol, 5, b, 3, mb.workspace(h, b), policy_is_init=False, tol_dv=tol,
                      max_outer=500, V64_out=V64)
    assert st["converged"] and st["policy_changes_last"] == 0
    Vs, mu, _ = oracle.policy_iteration(mdp)
    # residual <= tol bounds the distance by tol / (1 - gamma); the row scales
    # of the two quantisers may differ by an FP32 ulp
    slack = 0.0 if dtype == "f32" else 2.0 ** -23 * float(np.max(np.abs(Vs))) * gamma / (1 - gamma)
    assert float(np.max(np.abs(V64.cpu().numpy() - Vs))) <= tol / (1 - gamma) + slack
    if dtype == "f32":
        assert np.array_equal(pol.cpu().numpy(), mu)


def test_bad_policy_is_reported_by_one_workgroup_and_by_many():
    for n, b in ((40, 10), (1500, 300)):
        h, _ = stored_case(n, 3, "f32", 0.9, 9)
        pol = torch.zeros(n, dtype=torch.int32, device=dev())
        pol[n // 2] = 3
        ws = mb.workspace(h, b)
        with pytest.raises(mb.MbdpError):
            mb.mpi_solve(h, torch.zeros(n, device=dev()), pol, 2, b, 1, ws, tol_dv=1e-6)
        # the workspace serves the next call
        pol.zero_()
        assert mb.mpi_solve(h, torch.zeros(n, device=dev()), pol, 2, b, 1, ws, tol_dv=1e-6)["converged"]
