"""The FP64 correction of sparse MDPs on both sides of its choice between
values stored through to memory and plain stores released at the barrier: one
unit per wavefront and several, in policy sweeps, improvement passes and both,
with a short last batch; every output against the oracle."""
import numpy as np
import pytest

from paper_2110_02901_amd import inputs

from gpu_util import csr_case
from test_gpu_refine import Case, compare

pytestmark = pytest.mark.gpu


# 4096 wavefronts: a policy unit is 8 states at k = 32, 32 at k = 8; an
# improvement unit is a state; general CSR switches above two states each
@pytest.mark.parametrize("kind,n,b", [
    ("k32", 4000, 700), ("k32", 4100, 1000), ("k32", 33000, 32768), ("k32", 70000, 32769),
    ("k8", 140000, 131073), ("ragged", 8192, 3000), ("ragged", 8200, 8193), ("ragged", 20000, 9000),
])
@pytest.mark.parametrize("K", [0, 3])
def test_sparse(kind, n, b, K):
    if kind == "ragged":
        rp, col, val, c = inputs.csr_ragged_mdp(n, 2, 1, 9, 1.0, 30)
    else:
        rp, col, val, c = inputs.csr_mdp(n, 2, int(kind[1:]), 1.0, 30)
    h, mdp = csr_case(rp, col, val, c, 0.9)
    cs = Case(h, mdp)
    compare(mdp, inputs.values(n, 7, 0.0, 10.0).astype(np.float64), K, b, 600, 0.0, max_iters=3)
    del cs
