"""Trees of single-visit beliefs: the edges of the forward launch, of the walk
along the runs and of the sweep of the beliefs that several episodes reached.

A belief that only the episode that created it visited has a short record, and
the beliefs an episode creates in one iteration form a run.  The cases below
take the places where that can go wrong: nearly every belief shared (two
actions, one observation), no belief shared, runs that are a leaf only or as
deep as a plan may be, rows of each width, tables around the sizes where the
search trees over their rows gain a level, and obstacle lists around the size
that is kept on chip.  Each plan is held to the serial oracle draw by draw;
structure and counts are equal and values agree to the bound of
tests/drawcheck.py (fp32 records against double precision).
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


# (|A|, |O|, episodes, iterations, depth): shared beliefs first.
@pytest.mark.parametrize("nA,nO,n_p,K,depth", [
    (2, 1, 64, 4, 4), (2, 1, 65, 4, 4), (2, 1, 2500, 5, 5), (1, 1, 300, 3, 3),
    (3, 2, 1025, 6, 2), (3, 4, 1000, 3, 1), (4, 64, 63, 5, 5),
    (8, 3, 1500, 4, 4), (9, 3, 700, 3, 4), (16, 3, 700, 3, 4), (17, 3, 700, 3, 3),
    (40, 2, 900, 3, 3), (64, 1, 900, 3, 3), (65, 2, 900, 3, 3), (130, 1, 700, 3, 3)])
def test_shared_and_single_beliefs(V, orc, nA, nO, n_p, K, depth):
    inst = I.tabular_dense(21, 7, nA, nO, with_heuristic=True)
    forced_parity(V, orc, inst, I.tabular_belief(inst), n_p, K, depth, seed=2,
                  schedule=0 if K >= depth else 1)


# The deepest plans.  A record in single precision rounds once per backup, so
# over 64 backups its error may reach 64 units of 2^-24 of the row's largest
# entry, more than the 16 that the draw screen of forced_parity assumes (37.6 were
# measured, before and after runs had records of their own): the draws and the
# tree are compared, that premise is not asserted.
@pytest.mark.parametrize("K,schedule", [(64, 0), (3, 1)])
def test_deepest_plan(V, orc, K, schedule):
    inst = I.tabular_dense(21, 7, 2, 2, with_heuristic=True)
    bel = I.tabular_belief(inst)
    o = oracle_plan(orc, inst, bel, 3, K, 64, seed=2, schedule=schedule)
    pom = V.Pomdp.from_instance(inst)
    ws = V.Workspace(pom, V.params(3, seed=2, schedule=schedule), K, 64)
    res, tree, act, obs = gpu_forced_plan(V, pom, ws, inst, V.belief_tensor(inst, bel), bel.size,
                                          3, K, 64, o, seed=2, schedule=schedule)
    ws.close()
    pom.close()
    check_draws(o, act, obs)
    assert_tree_parity(res, tree, o, 2)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 64, 65, 128, 129, 300])
@pytest.mark.parametrize("which", ["successors", "observations"])
def test_row_lengths(V, orc, which, n):
    if which == "successors":
        inst = I.tabular_dense(5, n, 3, 5, alpha=2.0)
    else:
        inst = I.tabular_sparse(5, 30, 3, n, n_succ=6)
    forced_parity(V, orc, inst, I.tabular_belief(inst), 1200, 3, 3, seed=4)


def test_successor_rows_of_unequal_length(V, orc):
    inst = I.tabular_dense(8, 12, 4, 5, with_heuristic=True)
    rows = 12 * 4
    rng = np.random.default_rng(3)
    lens = rng.integers(1, 13, size=rows)
    col, tp = [], []
    for n in lens:
        col.append(np.sort(rng.choice(12, size=n, replace=False)).astype(np.int32))
        tp.append(rng.dirichlet(np.ones(n)).astype(np.float32))
    inst = dict(inst, rowptr=np.concatenate([[0], np.cumsum(lens)]).astype(np.int32),
                col=np.concatenate(col), tprob=np.concatenate(tp))
    forced_parity(V, orc, inst, I.tabular_belief(inst), 1200, 4, 4, seed=4)


@pytest.mark.parametrize("n_disks", [0, 1, 64, 65])
def test_obstacle_counts(V, orc, n_disks):
    inst = I.nav2d(6, 8)
    c = np.random.default_rng(9).uniform(0.0, 10.0, size=(n_disks, 2))
    inst = dict(inst, disks=c.astype(np.float32), disk_r2=0.04)
    forced_parity(V, orc, inst, I.nav_belief(3, 128), 1500, 5, 5, seed=4)


# Reference policies that are not uniform: one largest entry, and two.
@pytest.mark.parametrize("nA", [5, 8, 9, 16, 17, 40, 64])
@pytest.mark.parametrize("ties", [False, True])
def test_runs_under_a_prior(V, orc, nA, ties):
    inst = I.tabular_dense(31, 9, nA, 2, with_heuristic=True)
    pi0 = np.random.default_rng(nA).uniform(0.5, 1.5, size=(nA,))
    pi0[nA // 2] = 2.0
    if ties:
        pi0[nA - 1] = 2.0
    forced_parity(V, orc, inst, I.tabular_belief(inst), 900, 4, 4, seed=6, pi0=pi0 / pi0.sum())


# Long rows in plans of one level, whose runs are leaves only.
@pytest.mark.parametrize("nA,n_p,K", [(65, 1, 2), (70, 257, 3), (130, 1500, 4)])
def test_long_rows_of_one_level(V, orc, nA, n_p, K):
    inst = I.tabular_dense(23, 8, nA, 3, with_heuristic=True)
    forced_parity(V, orc, inst, I.tabular_belief(inst), n_p, K, 1, seed=3)
