"""Many episodes, few beliefs: the levels at which the lanes of a wavefront send one
of them to a new belief, and the edge of the rule that says which levels those are
(512 episodes to each of the (|A| |O|)^(level + 1) beliefs a level may create).

Each plan is held to the serial oracle draw by draw (tests/drawcheck.py).
"""

import numpy as np
import pytest

from paper_2510_27191_amd import instances as I
from tests.drawcheck import (assert_tree_parity, check_draws, forced_parity, gpu_forced_plan,
                             oracle_plan)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_27191_amd import vopp
    vopp.lib()
    return vopp


# No level crowded, the first one, two, all of them.
@pytest.mark.parametrize("nA,nO,n_p,K,depth", [
    (2, 1, 1023, 3, 3), (2, 1, 1024, 3, 3), (2, 1, 2047, 3, 1), (2, 1, 2048, 3, 3),
    (1, 1, 511, 3, 3), (1, 1, 513, 3, 3), (2, 3, 3072, 3, 3), (3, 1, 4610, 3, 4),
    (16, 1, 8200, 2, 2), (40, 1, 20500, 2, 2), (2, 1, 33000, 3, 2)])
def test_crowded_levels(V, orc, nA, nO, n_p, K, depth):
    inst = I.tabular_dense(21, 7, nA, nO, with_heuristic=True)
    forced_parity(V, orc, inst, I.tabular_belief(inst), n_p, K, depth, seed=2)


# The navigation model with a grid of one cell, and of four.
@pytest.mark.parametrize("key_n,n_p", [(1, 2047), (1, 2049), (2, 8200)])
def test_crowded_levels_of_the_navigation_model(V, orc, key_n, n_p):
    inst = dict(I.nav2d(4, 6), key_n=key_n, key_lo=0, inv_bin=0.1 * key_n)
    forced_parity(V, orc, inst, I.nav_belief(5, 500), n_p, 3, 3, seed=4)


# Episodes that follow another's run while it grows: every iteration goes to the full
# depth, so that in the first one nearly all beliefs are new, and shared.  Draws and
# tree are compared.  The premise of forced_parity on the rows' relative error
# does not hold for every such plan (rows whose entries nearly cancel: 18.0 units for 64
# episodes of 2 actions to depth 8, in the same bits when episodes did not
# follow runs at all), and it is not asserted.
def parity(V, orc, inst, bel, n_p, K, depth, seed):
    o = oracle_plan(orc, inst, bel, n_p, K, depth, seed=seed, schedule=1)
    pom = V.Pomdp.from_instance(inst)
    ws = V.Workspace(pom, V.params(n_p, seed=seed, schedule=1), K, depth)
    try:
        b = V.belief_tensor(inst, bel)
        nb = b.numel() if inst["kind"] == "tabular" else b.numel() // 2
        res, tree, act, obs = gpu_forced_plan(V, pom, ws, inst, b, nb, n_p, K, depth, o,
                                              seed=seed, schedule=1)
    finally:
        ws.close()
        pom.close()
    check_draws(o, act, obs)
    assert_tree_parity(res, tree, o, int(inst["nA"]))


@pytest.mark.parametrize("nA,nO,n_p,K,depth", [
    (1, 1, 300, 2, 8), (2, 1, 64, 3, 8), (2, 1, 2500, 3, 8), (2, 1, 300, 2, 20),
    (4, 1, 1500, 3, 6), (16, 1, 1500, 2, 5), (40, 1, 900, 2, 5), (70, 1, 900, 2, 5),
    (130, 1, 3000, 2, 3)])
def test_runs_that_are_followed(V, orc, nA, nO, n_p, K, depth):
    inst = I.tabular_dense(21, 7, nA, nO, with_heuristic=True)
    parity(V, orc, inst, I.tabular_belief(inst), n_p, K, depth, seed=2)


@pytest.mark.parametrize("key_n", [1, 2])
def test_navigation_runs_that_are_followed(V, orc, key_n):
    # near the goal, so that runs end early too
    inst = dict(I.nav2d(4, 6, heuristic=1), key_n=key_n, key_lo=0, inv_bin=0.1 * key_n)
    parity(V, orc, inst, I.nav_belief(5, 500, 6.6, 8.6), 2500, 3, 6, seed=4)
