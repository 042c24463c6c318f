"""Infinite values of V reach every row with a positive probability of them and
nothing else: lanes past a row's end or a segment's contribute no 0 * inf.
Rows of partial chunks in every value type, the value in the last column and
in the first, policy and minimum sweeps, the FP64 correction's rows and the
batched kernel."""
import numpy as np
import pytest
import torch

from paper_2110_02901_amd import binding as mb

from gpu_util import dev

pytestmark = pytest.mark.gpu


def positive_rows(n, m, ld=None):
    """P [n*m, ld]: rows whose n entries are all positive in every storage."""
    P = torch.zeros(n * m, ld or n, device=dev())
    w = 1.0 + (torch.arange(n * m * n, device=dev()) % 7).float().view(n * m, n) / 7
    P[:, :n] = w / w.sum(1, keepdim=True)
    return P


def handle(n, m, dtype):
    P, c = positive_rows(n, m), torch.rand(n, m, device=dev())
    if dtype == "f32":
        return mb.mdp_create_dense(P, c, 0.9)
    q, s = mb.mdp_quantize_rows(P, dtype)
    return mb.mdp_create_dense_q(q, dtype, s, c, 0.9)


@pytest.mark.parametrize("dtype,n,m", [("f32", 30, 3), ("f32", 500, 4), ("f32", 2311, 2),
                                       ("f32", 2312, 2), ("f32", 4099, 2), ("f32", 4100, 2), ("bf16", 504, 3), ("bf16", 2312, 2),
                                       ("fp8", 496, 3), ("fp8", 4112, 1)])
def test_sweeps(dtype, n, m):
    h = handle(n, m, dtype)
    pol = torch.zeros(n, dtype=torch.int32, device=dev())
    for b in (max(1, n // 5), n):
        ws = mb.workspace(h, b)
        for at in (0, n - 1):
            for policy, value in ((pol, float("inf")), (None, -float("inf"))):
                V = torch.ones(n, device=dev())
                V[at] = value
                mb.mb_sweep(h, V, b, 3, 0, ws, policy=policy)
                mb.mbdp_sync_status(ws)
                assert bool((V == value).all()), (b, at, value)


@pytest.mark.parametrize("n", [500, 2311, 4099])
def test_correction(n):
    h = handle(n, 2, "f32")
    ws = mb.workspace(h, n)
    for at in (0, n - 1):
        V = torch.ones(n, dtype=torch.float64, device=dev())
        V[at] = -float("inf")
        mb.mdp_refine(h, V, n, 3, ws, K=0, eps=1e-6, max_iters=1)
        assert bool((V == -float("inf")).all()), at


@pytest.mark.parametrize("dtype,n,ld,lanes", [("f32", 70, 80, 16), ("f32", 70, 80, 64),
                                              ("bf16", 100, 112, 32), ("fp8", 300, 304, 16)])
def test_batch(dtype, n, ld, lanes):
    P, c = positive_rows(n, 2, ld), torch.rand(n, 2, device=dev())
    it = {"n": n, "m": 2, "dtype": dtype, "ld": ld, "c": c, "gamma": 0.9, "b": n, "seed": 3,
          "lanes": lanes, "team": 1}
    if dtype == "f32":
        it["P"] = P
    else:
        it["P"], it["row_scale"] = mb.mdp_quantize_rows(P, dtype)
    for at in (0, n - 1):
        it["V"] = torch.ones(n, dtype=torch.float64, device=dev())
        it["V"][at] = -float("inf")
        ws = mb.batch_workspace(1)
        mb.mdp_batch_upload([it], ws)
        mb.mdp_batch_launch(1, 1e-6, 1, ws)
        mb.mdp_batch_read_stats(ws, 1)
        assert bool((it["V"] == -float("inf")).all()), at
