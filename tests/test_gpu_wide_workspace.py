"""Plans in a workspace that was made for more actions than the model has.

A workspace serves every plan that is not larger than the one it was made for, the
number of actions included.  The rows of the tree are then the model's, so
result and tree are those of a workspace made for the model, bit for bit.
"""

import numpy as np
import pytest

from paper_2510_27191_amd import instances as I
from tests.drawcheck import assert_tree_parity, check_draws, gpu_forced_plan, oracle_plan
from tests.test_gpu_failed_plans import same_plan
from tests.test_gpu_reroot import top_branch

pytestmark = pytest.mark.gpu

N_P, K, DEPTH = 1500, 4, 4


@pytest.fixture(scope="module")
def V():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_27191_amd import vopp
    vopp.lib()
    return vopp


def model(kind):
    if kind == "nav":
        return I.nav2d(4, 6, heuristic=1), I.nav_belief(5, 500)
    inst = I.tabular_dense(21, 7, kind, 3, with_heuristic=True)
    return inst, I.tabular_belief(inst)


def n_states(inst, b):
    return b.numel() if inst["kind"] == "tabular" else b.numel() // 2


def wide_workspace(V, nA):
    inst = I.tabular_dense(5, 4, nA, 2)
    pom = V.Pomdp.from_instance(inst)
    ws = V.Workspace(pom, V.params(N_P, schedule=1), K + 1, DEPTH + 1)
    pom.close()
    return ws


CASES = [("nav", 8), ("nav", 64), ("nav", 65), ("nav", 100), ("nav", 3025), (3, 5), (3, 130),
         (8, 64), (9, 100), (40, 100), (64, 68), (65, 130), (70, 3025)]


@pytest.mark.parametrize("kind,wide", CASES)
def test_plan_equals_one_in_its_own_workspace(V, kind, wide):
    inst, bel = model(kind)
    pom = V.Pomdp.from_instance(inst)
    prm = V.params(N_P, seed=4)
    b = V.belief_tensor(inst, bel)
    nb = n_states(inst, b)
    ws, own = wide_workspace(V, wide), V.Workspace(pom, prm, K, DEPTH)
    try:
        for _ in range(2):
            r = V.plan(pom, b, nb, K, DEPTH, prm, ws=ws)
            f = V.plan(pom, b, nb, K, DEPTH, prm, ws=own)
            same_plan(V, pom.nA, r, ws, f, own)
    finally:
        ws.close()
        own.close()
        pom.close()


@pytest.mark.parametrize("kind", ["nav", 3, 70])
def test_plan_matches_the_oracle(V, orc, kind):
    inst, bel = model(kind)
    o = oracle_plan(orc, inst, bel, N_P, K, DEPTH, seed=4)
    pom = V.Pomdp.from_instance(inst)
    b = V.belief_tensor(inst, bel)
    ws = wide_workspace(V, 100)
    try:
        res, tree, act, obs = gpu_forced_plan(V, pom, ws, inst, b, n_states(inst, b), N_P, K,
                                              DEPTH, o, seed=4)
    finally:
        ws.close()
        pom.close()
    check_draws(o, act, obs)
    assert_tree_parity(res, tree, o, int(inst["nA"]))


# Each of the two workspaces of a re-rooting made for more actions, or both.
@pytest.mark.parametrize("kind", ["nav", 3, 70])
@pytest.mark.parametrize("src_wide,dst_wide", [(True, False), (False, True), (True, True)])
def test_reroot_between_workspaces(V, kind, src_wide, dst_wide):
    inst, bel = model(kind)
    pom = V.Pomdp.from_instance(inst)
    b = V.belief_tensor(inst, bel)
    nb = n_states(inst, b)
    p1, p2 = V.params(N_P, seed=4), V.params(N_P, seed=11)
    own = [V.Workspace(pom, p1, K, DEPTH) for _ in range(2)]
    ws = [wide_workspace(V, 130) if w else V.Workspace(pom, p1, K, DEPTH)
          for w in (src_wide, dst_wide)]
    try:
        r = V.plan(pom, b, nb, K, DEPTH, p1, ws=ws[0])
        f = V.plan(pom, b, nb, K, DEPTH, p1, ws=own[0])
        same_plan(V, pom.nA, r, ws[0], f, own[0])
        o = top_branch(V.tree_dump(own[0], pom.nA, f.n_beliefs, f.n_actions), f.action)
        kept = [V.reroot(pom, w[0], f.action, o, p2, 3, DEPTH, w[1]) for w in (ws, own)]
        assert kept[0] == kept[1] > 1
        r = V.plan(pom, b, nb, 3, DEPTH, p2, ws=ws[1])
        f = V.plan(pom, b, nb, 3, DEPTH, p2, ws=own[1])
        same_plan(V, pom.nA, r, ws[1], f, own[1])
    finally:
        for w in ws + own:
            w.close()
        pom.close()
