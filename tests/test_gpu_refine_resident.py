"""The FP64 correction with V in every workgroup's LDS (dense, n <= 8192) at
the edges of its dispatch: a lone workgroup and many, each row shape (rows of
at most two steps side by side, single rows of a table in the caches and past
them), rows shorter than a load (the engine with V in memory), rows that are
not whole 16-byte loads, fewer states than workgroups, parts of a state's rows
on several workgroups, one batch and short last batches; every output against
the oracle, from a perturbed J*."""
import numpy as np
import pytest

import oracle
from paper_2110_02901_amd import inputs

from gpu_util import dense_case
from test_gpu_refine import Case, compare

pytestmark = pytest.mark.gpu


# The correction runs whole where policy iteration gives J*; the largest
# sizes stop at a sweep limit from an arbitrary V.
@pytest.mark.parametrize("n,m,b", [
    (3, 2, 2), (4, 3, 2), (5, 2, 5), (64, 4, 64), (257, 5, 31), (300, 130, 300), (1021, 3, 1),
    (1024, 8, 16), (1100, 7, 1024),
])
@pytest.mark.parametrize("K", [0, 1, 4])
def test_correction_to_eps(n, m, b, K):
    P, c = inputs.dense_mdp(n, m, 0.5, 40 + n, dtype=np.float32)
    h, mdp = dense_case(P, c, 0.9)
    cs = Case(h, mdp)
    Vstar, _, _ = oracle.policy_iteration(mdp)
    V0 = Vstar + inputs.values(n, 6, -1e-3, 1e-3).astype(np.float64)
    compare(mdp, V0, K, b, 500 + b, 1e-8, Vstar=Vstar, first_sweep=2)
    compare(mdp, V0, K, b, 500 + b, 1e-6, Vstar=Vstar, V_ref=Vstar)
    del cs


@pytest.mark.parametrize("n,m,b", [(2050, 6, 1030), (4095, 3, 333), (8192, 1, 3000), (8190, 1, 8190)])
@pytest.mark.parametrize("K", [0, 2])
def test_sweep_limit(n, m, b, K):
    P, c = inputs.dense_mdp(n, m, 1.0, 41 + n, dtype=np.float32)
    h, mdp = dense_case(P, c, 0.9)
    cs = Case(h, mdp)
    compare(mdp, inputs.values(n, 7, 0.0, 10.0).astype(np.float64), K, b, 600, 0.0, max_iters=3)
    del cs
