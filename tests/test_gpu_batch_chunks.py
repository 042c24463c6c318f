"""The batched kernel's chunks at their edges, against the oracle: rows shorter
and longer than a step of a lane group, numbers of actions around the rows taken
together (8, FP8 4) and several passes of them, one batch per sweep and batches
of one state, fewer states than lane groups, alone and in teams.

FP64 arithmetic on exactly decoded rows: the batched tests' 1e-11 relative."""
import numpy as np
import pytest

import oracle
from paper_2110_02901_amd import binding as mb

from test_gpu_batch import make_item

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("team", [1, 3])
@pytest.mark.parametrize("lanes", [0, 16, 32, 64])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8"])
def test_chunk_edges(dtype, lanes, team):
    shapes = [(5, 9, 5), (17, 17, 1), (130, 7, 130), (129, 64, 20), (520, 3, 65), (16, 1, 7)]
    made = [make_item(n, m, dtype, 0.9, b, 70 + i, 30 + i, lanes)
            for i, (n, m, b) in enumerate(shapes)]
    items = [x[0] for x in made]
    for it in items:
        it["team"] = team
    ws = mb.batch_workspace(len(items))
    mb.mdp_batch_upload(items, ws)
    T = 5
    mb.mdp_batch_launch(len(items), -1.0, T, ws)
    stats = mb.mdp_batch_read_stats(ws, len(items))
    for (item, mdp, V0), st in zip(made, stats):
        assert st["sweeps"] == T and st["team"] == team
        ref, _, info = oracle.value_iteration(mdp, item["b"], item["seed"], V0=V0, tol_dv=-1,
                                              max_sweeps=T)
        Vg = item["V"].cpu().numpy()
        assert np.max(np.abs(Vg - ref)) <= 1e-11 * max(1.0, float(np.max(np.abs(ref))))
        Q = oracle.q_values(mdp, np.arange(mdp.n), Vg)
        chosen = Q[np.arange(mdp.n), item["policy"].cpu().numpy()]
        assert np.all(chosen <= Q.min(axis=1) + 1e-10)


def test_as_many_mdps_as_compute_units_share_them():
    # a heavy MDP among light ones is given workgroups of its own
    made = [make_item(n, 4, "bf16", g, max(1, n // 8), 9, 50 + n, with_oracle=False)
            for n, g in ((900, 0.98), (64, 0.9), (80, 0.9))]
    items = [x[0] for x in made]
    ws = mb.batch_workspace(len(items))
    mb.mdp_batch_upload(items, ws)
    mb.mdp_batch_launch(len(items), -1.0, 2, ws)
    teams = [s["team"] for s in mb.mdp_batch_read_stats(ws, len(items))]
    assert teams[0] > 1 and sum(teams) <= 256
