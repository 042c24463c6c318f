"""What a call with a bad entry in its explicit order or policy leaves behind:
the error, V as it was and a change of 0, for dense MDPs served by one
workgroup and by many, in the first batch and in a later one, and for sparse
MDPs (explicit orders); the workspace serves the next call."""
import numpy as np
import pytest
import torch

from paper_2110_02901_amd import binding as mb
from paper_2110_02901_amd import inputs

from gpu_util import csr_case, dense_case, dev, run_sweep, up

pytestmark = pytest.mark.gpu


def check_left_alone(h, n, b, policy=None, perm=None):
    ws = mb.workspace(h, b)
    ws.fill_(0xFF)  # as another call may have left it
    V0 = inputs.values(n, 5, 1.0, 4.0).astype(np.float32)
    V, dv = up(V0), torch.full((1,), 7.0, device=dev())
    mb.mb_sweep(h, V, b, 3, 0, ws, policy=policy, perm=perm, dv_out=dv)
    with pytest.raises(mb.MbdpError) as e:
        mb.mbdp_sync_status(ws)
    assert e.value.status == mb.MBDP_ERR_DEVICE
    assert np.array_equal(V.cpu().numpy(), V0)
    assert float(dv.item()) == 0.0
    mb.mb_sweep(h, V, b, 3, 0, ws, dv_out=dv)
    mb.mbdp_sync_status(ws)
    assert float(dv.item()) > 0.0


@pytest.mark.parametrize("n,b", [(40, 10), (40, 40), (1500, 300), (1500, 1500), (1500, 20)])
@pytest.mark.parametrize("at", [0, -1])
def test_dense(n, b, at):
    P, c = inputs.dense_mdp(n, 3, 0.5, 9, dtype=np.float32)
    h, mdp = dense_case(P, c, 0.9)
    perm = np.random.default_rng(n).permutation(n).astype(np.int32)
    for bad in (n, -1):
        wrong = perm.copy()
        wrong[at] = bad
        check_left_alone(h, n, b, perm=up(wrong))
    pol = np.zeros(n, np.int32)
    pol[at] = 3
    check_left_alone(h, n, b, policy=up(pol))
    # a solve from a bad policy: V and the policy stay
    V0 = inputs.values(n, 6, 1.0, 4.0).astype(np.float32)
    V, P0 = up(V0), up(pol)
    with pytest.raises(mb.MbdpError) as e:
        mb.mpi_solve(h, V, P0, 2, b, 1, mb.workspace(h, b), tol_dv=1e-6)
    assert e.value.status == mb.MBDP_ERR_DEVICE
    assert np.array_equal(V.cpu().numpy(), V0) and np.array_equal(P0.cpu().numpy(), pol)
    run_sweep(h, mdp, V0, b, 3, 0, perm=perm)


@pytest.mark.parametrize("k", [None, 8])
def test_sparse_order(k):
    n = 700
    if k:
        rp, col, val, c = inputs.csr_mdp(n, 3, k, 1.0, 4)
    else:
        rp, col, val, c = inputs.csr_ragged_mdp(n, 3, 1, 9, 1.0, 4)
    h, _ = csr_case(rp, col, val, c, 0.9)
    for b in (100, n):
        wrong = np.arange(n, dtype=np.int32)
        wrong[-1] = n
        check_left_alone(h, n, b, perm=up(wrong))


@pytest.mark.parametrize("n,b", [(40, 10), (1500, 300)])
def test_status_words_of_another_call(n, b):
    # a workspace of ones: an abort and an error that no call of ours raised
    P, c = inputs.dense_mdp(n, 3, 0.5, 9, dtype=np.float32)
    h, _ = dense_case(P, c, 0.9)
    ws = mb.workspace(h, b)
    V = torch.zeros(n, device=dev())
    for t in range(5):
        ws.fill_(0xFF)
        mb.mb_sweep(h, V, b, 3, t, ws)
        mb.mbdp_sync_status(ws)
    ws.fill_(0xFF)
    assert mb.vi_solve(h, V, b, 3, ws, tol_dv=1e-6)["converged"]
