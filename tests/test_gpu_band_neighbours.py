"""The band engine's batches, ordered among the workgroups whose windows
overlap only: windows that reach no neighbour, one and many workgroups away,
and fewer states than workgroups; against the oracle, and bit for bit against
the general engine, which orders all workgroups (the sums are the same)."""
import numpy as np
import pytest

from paper_2110_02901_amd import binding as mb, inputs

from gpu_util import csr_case, run_sweep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,band,b", [
    (30000, 0, 700), (30000, 1, 30), (30000, 118, 311), (30000, 1200, 311), (150, 20, 7), (257, 3, 2),
])
def test_batches_ordered_among_neighbours(n, band, b):
    m, k = 3, 8
    rp, col, val, c = inputs.csr_mdp(n, m, k, 1.0, 80 + band, band=max(band, 8))
    if band < 8:  # narrower than the generator's rows: clamp the columns
        s = np.repeat(np.arange(n), m * k)
        col = np.clip(col, s - band, s + band).clip(0, n - 1).astype(np.int32)
    h, mdp = csr_case(rp, col, val, c, 0.95)
    assert mb.mdp_engine(h, b) == "ell-band"
    V0 = inputs.values(n, 5, 0.0, 9.0)
    Vb, _ = run_sweep(h, mdp, V0, b, 21, 1, check_arg=False)
    mb.mdp_set_tuning(h, band_window=-1)
    assert mb.mdp_engine(h, b) == "ell"
    Ve, _ = run_sweep(h, mdp, V0, b, 21, 1, check_arg=False)
    assert np.array_equal(Vb, Ve)
