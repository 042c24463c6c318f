"""The multi-vector product at the edges of its dispatch, against the oracle:
launches that fill the device (eight wavefronts per workgroup) and fewer, K
ranges of one short round, of whole rounds and with a short last one, row
tiles that end inside a workgroup.  Two sweeps, the second with W from the
first; tolerance of a sweep: 2^-16 of the largest change of V (two BF16 terms
of W in the products), twice."""
import numpy as np
import pytest

from oracle import multi as om

from test_gpu_multi import bf16_case, gpu_multi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,b,rs", [
    (32, 1, 5, (16, 64)), (96, 3, 96, (16, 32, 48, 64)), (288, 3, 100, (16, 32, 48, 64)),
    (1056, 16, 1056, (16, 32)), (2080, 8, 2080, (48, 64)),
])
def test_two_sweeps(n, m, b, rs):
    gamma = 0.9
    for r in rs:
        h, Pst, C = bf16_case(n, m, r, gamma, 60 + n)
        V0 = np.random.Generator(np.random.Philox(n + r)).uniform(0.0, 2.0, (n, r))
        Vg, _, st = gpu_multi(h, C, V0, b, 9, max_sweeps=2, policy=False)
        assert st["sweeps"] == 2
        ref, _, _, _ = om.multi_value_iteration(Pst, C.astype(np.float64), gamma, b, 9, V0=V0,
                                                tol_dv=-1, max_sweeps=2)
        err = float(np.max(np.abs(Vg - ref)))
        bound = 2 * 2.0 ** -16 * float(np.max(np.abs(ref - V0))) + 1e-12
        assert err <= bound, (r, err, bound)
