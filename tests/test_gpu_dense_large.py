"""Dense MDPs around the limits of the resident-value kernel (V in LDS, at most
16384 states and 8192 entries of a workgroup's list) and past them, where the
general dense engine runs (a workgroup per state, columns split over
workgroups for small batches, up to four states at once for large ones):
every value type, 16-byte and single loads, minimum and policy sweeps,
re-centring, both solvers.  The reference is plain FP64 on the GPU.

Tolerance: SWEEP_RTOL * max|V| a sweep, as for single sweeps; T sweeps at most
T times that.
"""
import functools

import numpy as np
import pytest
import torch

import oracle
from paper_2110_02901_amd import binding as mb
from paper_2110_02901_amd import inputs

from gpu_util import SWEEP_RTOL, dev, up

pytestmark = pytest.mark.gpu
GAMMA = 0.9


class Table:
    """A random dense MDP on the GPU, its handle and its FP64 backups."""

    def __init__(self, dtype, n, m, seed=5):
        g = torch.Generator(device=dev())
        g.manual_seed(seed + n)
        self.dtype, self.n, self.m = dtype, n, m
        self.c = torch.rand(n, m, generator=g, device=dev())
        P = torch.rand(n * m, n, generator=g, device=dev())
        for r in range(0, n * m, 4096):
            P[r:r + 4096] /= P[r:r + 4096].sum(1, keepdim=True)
        if dtype == "f32":
            self.P, self.scale = P, None
            self.h = mb.mdp_create_dense(P, self.c, GAMMA)
        else:
            self.P, self.scale = mb.mdp_quantize_rows(P, dtype)
            self.h = mb.mdp_create_dense_q(self.P, dtype, self.scale, self.c, GAMMA)

    def q(self, states, V):
        """Q(s, .) of `states` [len, m] at V (FP64)."""
        out = []
        for part in states.split(max(1, 2048 // self.m)):
            rows = (part[:, None] * self.m + torch.arange(self.m, device=dev())).reshape(-1)
            x = self.P.view(self.n * self.m, self.n)[rows]
            if self.dtype == "bf16":
                x = x.view(torch.bfloat16)
            elif self.dtype == "fp8":
                x = x.view(torch.float8_e4m3fn)
            d = x.to(torch.float64) @ V
            if self.scale is not None:
                d = d * self.scale[rows].double()
            out.append(self.c[part].double() + GAMMA * d.view(len(part), self.m))
        return torch.cat(out)

    def sweep(self, V, b, seed, t, policy=None):
        order = torch.from_numpy(oracle.sweep_permutation(self.n, seed, t).astype(np.int64)).to(dev())
        V = V.clone()
        for s in order.split(b):
            Q = self.q(s, V)
            V[s] = Q.min(1).values if policy is None else Q[torch.arange(len(s)), policy[s].long()]
        return V


@functools.lru_cache(maxsize=1)
def table(dtype, n, m):
    return Table(dtype, n, m)


def v0(n):
    return up(inputs.values(n, 4, 0.0, 5.0).astype(np.float32))


def check_sweep(t, b, policy=None):
    V = v0(t.n)
    ref = t.sweep(V.double(), b, 7, 2, policy)
    ws = mb.workspace(t.h, b)
    dv = torch.zeros(1, device=dev())
    W = V.clone()
    mb.mb_sweep(t.h, W, b, 7, 2, ws, policy=policy, dv_out=dv)
    mb.mbdp_sync_status(ws)
    tol = SWEEP_RTOL * float(V.abs().max())
    assert float((W.double() - ref).abs().max()) <= tol
    assert abs(float(dv) - float((ref - V.double()).abs().max())) <= tol


def check_solves(t, b, T=3):
    """T sweeps of value iteration, re-centred after every sweep, and MPI."""
    n = t.n
    V = v0(n)
    ref = V.double()
    for k in range(T):
        ref = t.sweep(ref, b, 11, k)
    tol = T * SWEEP_RTOL * float(V.abs().max())
    mb.mdp_set_tuning(t.h, recentre_every=1, recentre_force=True)
    V64 = torch.zeros(n, dtype=torch.float64, device=dev())
    W = V.clone()
    st = mb.vi_solve(t.h, W, b, 11, mb.workspace(t.h, b), tol_dv=-1.0, max_sweeps=T, V64_out=V64)
    assert st["sweeps"] == T and st["recentrings"] == T - 1
    assert float((V64 - ref).abs().max()) <= tol
    mb.mdp_set_tuning(t.h)
    pol = torch.zeros(n, dtype=torch.int32, device=dev())
    W = torch.zeros(n, device=dev())
    st = mb.mpi_solve(t.h, W, pol, 5, b, 3, mb.workspace(t.h, b), policy_is_init=False, tol_dv=1e-6,
                      V64_out=V64)
    assert st["converged"] and st["policy_changes_last"] == 0
    Q = t.q(torch.arange(n, device=dev()), V64)
    slack = SWEEP_RTOL * float(V64.abs().max())
    assert float((Q.min(1).values - V64).abs().max()) <= 1e-6 + slack
    assert bool((Q.gather(1, pol.long()[:, None])[:, 0] <= Q.min(1).values + slack).all())


# past 16384 states: b = n and large batches (several states a workgroup),
# fewer states than workgroups (split columns), a short last batch
GENERAL = [("f32", 16388, 2), ("f32", 16387, 1), ("bf16", 16400, 2), ("fp8", 16400, 2)]


@pytest.mark.parametrize("dtype,n,m", GENERAL)
def test_general_engine_sweeps(dtype, n, m):
    t = table(dtype, n, m)
    for b in (n, 5000, 700, 100, 9):
        check_sweep(t, b)
    pol = up(inputs.policy(n, m, 6).astype(np.int32))
    for b in (n, 3000, 50):
        check_sweep(t, b, pol)


@pytest.mark.parametrize("dtype,n,m", GENERAL)
def test_general_engine_solves(dtype, n, m):
    check_solves(table(dtype, n, m), 4000)


# the longest list of a workgroup (8192 batches), and one entry more; more
# actions than a tile of rows
@pytest.mark.parametrize("n", [8192, 8196])
def test_both_sides_of_the_list_limit(n):
    t = table("f32", n, 1)
    check_sweep(t, 1)
    check_sweep(t, 2, up(inputs.policy(n, 1, 6).astype(np.int32)))


def test_general_engine_many_actions_and_one_state_batches():
    t = table("fp8", 8208, 20)
    check_sweep(t, 1)


# V fills the LDS; R of a re-centring is read from memory (more than 8192 states)
@pytest.mark.parametrize("dtype,n,m", [("f32", 16384, 1), ("f32", 9001, 2), ("bf16", 16384, 2),
                                       ("fp8", 16384, 2)])
def test_resident_kernel_up_to_its_limit(dtype, n, m):
    t = table(dtype, n, m)
    for b in (n, 5000, 300):
        check_sweep(t, b)
    check_sweep(t, 1000, up(inputs.policy(n, m, 6).astype(np.int32)))
    check_solves(t, 3000)


# the FP64 correction past 8192 states (V in memory): FP64 on both sides,
# summed in different orders
@pytest.mark.parametrize("n", [8196, 9001])
@pytest.mark.parametrize("K,b", [(0, 3000), (0, 9), (3, 3000), (3, 8196)])
def test_correction_with_v_in_memory(n, K, b):
    t = table("f32", n, 2)
    ref = v0(n).double()
    every = torch.arange(n, device=dev())
    outer, sweeps = (0, 2) if K == 0 else (2, 2 * K)
    for k in range(sweeps):
        if K and k % K == 0:
            mu = t.q(every, ref).argmin(1)
        ref = t.sweep(ref, b, 13, k, mu if K else None)
    Q = t.q(every, ref)
    V = v0(n).double()
    pol = torch.zeros(n, dtype=torch.int32, device=dev())
    st = mb.mdp_refine(t.h, V, b, 13, mb.workspace(t.h, b), K=K, eps=0.0, max_iters=2,
                       policy_out=pol)
    assert st["sweeps"] == sweeps and st["outer_iters"] == outer
    assert float((V - ref).abs().max()) <= 1e-12 * float(ref.abs().max())
    assert abs(st["residual_out"] - float((Q.min(1).values - ref).abs().max())) <= 1e-11
    assert bool((Q.gather(1, pol.long()[:, None])[:, 0] <= Q.min(1).values + 1e-11).all())
