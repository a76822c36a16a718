"""Plans of one level with rows of up to 64 actions: beliefs are full leaves from the
start, found by table slot or id, and the leaf sweep goes by the run words (tests of
longer rows: tests/test_gpu_long_leaves.py).

Plans and chains of plans are held to the serial oracle draw by draw
(tests/drawcheck.py, tests/test_gpu_reroot.py); batched and served plans, which take the
general way, give the same results.
"""

import numpy as np
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


# Episodes around a block, a crowded level, and more runs than one to a thread of the
# sweep's largest launch (131,072).
@pytest.mark.parametrize("nA,nO,n_p,K", [
    (1, 1, 1, 1), (1, 1, 600, 3), (2, 1, 255, 3), (2, 3, 257, 4), (4, 8, 1000, 5),
    (3, 4, 33000, 4), (8, 2, 5000, 3), (16, 3, 900, 3), (17, 2, 900, 3), (40, 2, 900, 3),
    (64, 1, 900, 3)])
def test_tabular(V, orc, nA, nO, n_p, K):
    inst, bel = model(nA, nO)
    forced_parity(V, orc, inst, bel, n_p, K, 1, seed=3)


@pytest.mark.parametrize("nA", [5, 40])
def test_prior(V, orc, nA):
    inst, bel = model(nA, 3)
    pi0 = np.random.default_rng(nA).uniform(0.5, 1.5, size=(nA,))
    forced_parity(V, orc, inst, bel, 900, 4, 1, seed=6, pi0=pi0 / pi0.sum())


@pytest.mark.parametrize("lo,hi", [(0.5, 1.5), (7.9, 8.9)])      # the second: terminals
def test_navigation(V, orc, lo, hi):
    inst = I.nav2d(4, 6, heuristic=1)
    forced_parity(V, orc, inst, I.nav_belief(5, 500, lo, hi), 1500, 4, 1, seed=4)


@pytest.mark.parametrize("plans", [
    [(700, 3, 3), (700, 3, 1), (700, 2, 3)],
    [(700, 3, 1), (700, 3, 1)],
    [(700, 3, 2), (300, 4, 1)]])
@pytest.mark.parametrize("nA", [3, 16, 40])
def test_chains(V, orc, nA, plans):
    inst, bel = model(nA, 2)
    forced_chain(V, orc, inst, bel, plans, nA)


def test_every_entry_point(V):
    inst, bel = model(5, 4)
    pom = V.Pomdp.from_instance(inst)
    b = V.belief_tensor(inst, bel)
    prm = V.params(900, seed=5)
    ws, ref = V.Workspace(pom, prm, 4, 3), V.Workspace(pom, prm, 4, 1)
    try:
        f = V.plan(pom, b, b.numel(), 4, 1, prm, ws=ref)
        for _ in range(2):
            V.plan(pom, b, b.numel(), 4, 3, prm, ws=ws)
            r = V.plan(pom, b, b.numel(), 4, 1, prm, ws=ws)
            same_plan(V, 5, r, ws, f, ref)
        r, k = V.plan_anytime(pom, b, b.numel(), 4, 1, 1e6, prm, ws=ws)
        assert k == 4
        same_plan(V, 5, r, ws, f, ref)
        from tests.test_zz_no_alloc import noalloc, same
        same(f, noalloc(V, pom, b, b.numel(), 4, 1, prm), 5)
        batch = V.Batch([(pom, b, b.numel(), 4, 1, prm)] * 2)
        for mode in (V.BATCH_EAGER, V.BATCH_GRAPH, V.BATCH_PERSISTENT):
            for q in batch.run(mode=mode)[0]:
                assert q.action == f.action and q.v_root == f.v_root
                assert np.array_equal(q.values, f.values)
                assert (q.particle_steps, q.n_beliefs, q.n_actions) == \
                    (f.particle_steps, f.n_beliefs, f.n_actions)
        batch.close()
    finally:
        ws.close()
        ref.close()
        pom.close()
