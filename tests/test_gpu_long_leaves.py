"""Leaves of long action rows (more than 64 actions): plans of one level, whose beliefs
are full from the start, leaves at a deeper plan's full depth, which get no row,
and leaves of the iterations before, which do.  A leaf without a row is dumped and
re-rooted with the initial one.

Plans and chains of plans are held to the serial oracle draw by draw
(tests/drawcheck.py, tests/test_gpu_reroot.py).
"""

import pytest

from paper_2510_27191_amd import instances as I
from tests.drawcheck import forced_parity
from tests.test_gpu_failed_plans import same_plan
from tests.test_gpu_reroot import forced_chain

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_27191_amd import vopp
    vopp.lib()
    return vopp


def model(nA, nO):
    inst = I.tabular_dense(23, 8, nA, nO, with_heuristic=True)
    return inst, I.tabular_belief(inst)


# Episodes around a block of the claim pass (32 or 256 leaves), few and many leaves.
@pytest.mark.parametrize("nA,nO,n_p", [(65, 1, 1), (65, 1, 31), (68, 2, 33), (130, 1, 255),
                                       (130, 3, 257), (1030, 2, 700), (4096, 1, 300)])
@pytest.mark.parametrize("K,depth", [(3, 1), (3, 2), (4, 3)])
def test_plans(V, orc, nA, nO, n_p, K, depth):
    # (the share of draws near a boundary grows with the boundaries: as in
    # tests/test_gpu_wide.py)
    inst, bel = model(nA, nO)
    forced_parity(V, orc, inst, bel, n_p, K, depth, seed=3, max_flag_frac=0.2)


@pytest.mark.parametrize("nA", [65, 130])
@pytest.mark.parametrize("plans", [
    [(700, 3, 2), (700, 3, 1), (700, 2, 2)],      # to one level and back
    [(700, 3, 1), (700, 3, 1)],
    [(700, 3, 3), (500, 3, 3), (500, 3, 2)]])
@pytest.mark.parametrize("schedule", [0, 1])
def test_chains(V, orc, nA, plans, schedule):
    inst, bel = model(nA, 2)
    forced_chain(V, orc, inst, bel, plans, nA, schedule=schedule)


# The same tree whatever the order in which episodes reach their leaves, and after
# another plan in the workspace.
def test_anytime_and_repeated_plans_of_one_level(V):
    inst, bel = model(130, 2)
    pom = V.Pomdp.from_instance(inst)
    b = V.belief_tensor(inst, bel)
    prm = V.params(900, seed=5)
    ws, ref = V.Workspace(pom, prm, 4, 3), V.Workspace(pom, prm, 4, 1)
    try:
        f = V.plan(pom, b, b.numel(), 4, 1, prm, ws=ref)
        for _ in range(2):
            V.plan(pom, b, b.numel(), 4, 3, prm, ws=ws)
            r = V.plan(pom, b, b.numel(), 4, 1, prm, ws=ws)
            same_plan(V, 130, r, ws, f, ref)
        r, k = V.plan_anytime(pom, b, b.numel(), 4, 1, 1e6, prm, ws=ws)
        assert k == 4
        same_plan(V, 130, r, ws, f, ref)
    finally:
        ws.close()
        ref.close()
        pom.close()
