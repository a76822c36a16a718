"""What a plan that failed leaves behind.

A plan is refused before it starts (arguments, sizes), or it starts and then
fails, for instance because a belief particle holds a state outside [0, nS).
The first kind leaves its workspace as it was; after the second kind the
workspace holds neither a tree nor a kept subtree, and the next plan in it is
one from a fresh root.
"""

import numpy as np
import pytest

from paper_2510_27191_amd import instances as I
from tests.test_gpu_reroot import top_branch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_27191_amd import vopp
    vopp.lib()
    return vopp


def same_plan(V, nA, r, ws, f, ws_f):
    """Both results and trees, bit for bit."""
    assert r.action == f.action and r.v_root == f.v_root
    assert np.array_equal(r.values, f.values)
    assert (r.particle_steps, r.n_beliefs, r.n_actions) == \
        (f.particle_steps, f.n_beliefs, f.n_actions)
    tr = V.tree_dump(ws, nA, r.n_beliefs, r.n_actions)
    tf = V.tree_dump(ws_f, nA, f.n_beliefs, f.n_actions)
    for k in tf:
        assert np.array_equal(tr[k], tf[k]), k


def models(nA):
    inst = I.tabular_dense(21, 7, nA, 3, with_heuristic=True)
    return inst, I.tabular_belief(inst)


def with_bad_state(inst, b):
    bad = b.clone()
    bad[-1] = inst["nS"]
    return bad


# A kept subtree is planned from once.  (The same draws as before, under the same
# parameters, would meet the beliefs that the failed plan created.)
@pytest.mark.parametrize("schedule", [0, 1])
@pytest.mark.parametrize("nA", [3, 16, 70])
@pytest.mark.parametrize("anytime", [False, True])
def test_failed_plan_uses_up_the_kept_subtree(V, nA, schedule, anytime):
    inst, bel = models(nA)
    pom = V.Pomdp.from_instance(inst)
    b = V.belief_tensor(inst, bel)
    bad = with_bad_state(inst, b)
    p1, p2 = V.params(700, seed=2), V.params(700, seed=9, schedule=schedule)
    src, dst, ref = (V.Workspace(pom, p, 4, 4) for p in (p1, p2, p2))
    try:
        r1 = V.plan(pom, b, b.numel(), 4, 4, p1, ws=src)
        o = top_branch(V.tree_dump(src, nA, r1.n_beliefs, r1.n_actions), r1.action)
        assert V.reroot(pom, src, r1.action, o, p2, 4, 4, dst) > 1
        with pytest.raises(V.VoppError) as e:      # refused before it starts
            V.plan(pom, b, b.numel(), 5, 4, p2, ws=dst)
        assert e.value.status == V.VOPP_E_INVALID
        with pytest.raises(V.VoppError) as e:
            if anytime:
                V.plan_anytime(pom, bad, b.numel(), 4, 4, 1e6, p2, ws=dst)
            else:
                V.plan(pom, bad, b.numel(), 4, 4, p2, ws=dst)
        assert e.value.status == V.VOPP_E_INVALID and "nS" in str(e.value)
        r = V.plan(pom, b, b.numel(), 4, 4, p2, ws=dst)
        f = V.plan(pom, b, b.numel(), 4, 4, p2, ws=ref)
        same_plan(V, nA, r, dst, f, ref)
    finally:
        for w in (src, dst, ref):
            w.close()
        pom.close()


# ... and a call that was refused before it started has not used it up.
def test_refused_call_leaves_the_kept_subtree(V):
    inst, bel = models(3)
    pom = V.Pomdp.from_instance(inst)
    b = V.belief_tensor(inst, bel)
    p1, p2 = V.params(700, seed=2), V.params(700, seed=9)
    src, one, two = (V.Workspace(pom, p, 4, 4) for p in (p1, p2, p2))
    try:
        r1 = V.plan(pom, b, b.numel(), 4, 4, p1, ws=src)
        o = top_branch(V.tree_dump(src, 3, r1.n_beliefs, r1.n_actions), r1.action)
        for w in (one, two):
            assert V.reroot(pom, src, r1.action, o, p2, 4, 4, w) > 1
        with pytest.raises(V.VoppError):
            V.plan(pom, b, b.numel(), 5, 4, p2, ws=one)
        with pytest.raises(V.VoppError):
            V.plan(pom, b, 0, 4, 4, p2, ws=one)
        x = V.plan(pom, b, b.numel(), 4, 4, p2, ws=one)
        y = V.plan(pom, b, b.numel(), 4, 4, p2, ws=two)
        same_plan(V, 3, x, one, y, two)
    finally:
        for w in (src, one, two):
            w.close()
        pom.close()


# A failed plan of another size than the one before it leaves no tree.
@pytest.mark.parametrize("nA", [3, 70])
def test_failed_plan_leaves_no_tree(V, nA):
    inst, bel = models(nA)
    pom = V.Pomdp.from_instance(inst)
    b = V.belief_tensor(inst, bel)
    p1, p2 = V.params(700, seed=2), V.params(300, seed=5)
    ws, dst = V.Workspace(pom, p1, 4, 4), V.Workspace(pom, p1, 4, 4)
    try:
        r1 = V.plan(pom, b, b.numel(), 4, 4, p1, ws=ws)
        o = top_branch(V.tree_dump(ws, nA, r1.n_beliefs, r1.n_actions), r1.action)
        with pytest.raises(V.VoppError):
            V.plan(pom, with_bad_state(inst, b), b.numel(), 3, 3, p2, ws=ws)
        for use in (lambda: V.level_counts(ws),
                    lambda: V.tree_dump(ws, nA, r1.n_beliefs, r1.n_actions),
                    lambda: V.reroot(pom, ws, r1.action, o, p1, 4, 4, dst)):
            with pytest.raises(V.VoppError) as e:
                use()
            assert e.value.status == V.VOPP_E_INVALID and "no plan" in str(e.value)
        r = V.plan(pom, b, b.numel(), 4, 4, p1, ws=ws)
        f = V.plan(pom, b, b.numel(), 4, 4, p1, ws=dst)
        same_plan(V, nA, r, ws, f, dst)
    finally:
        ws.close()
        dst.close()
        pom.close()


# A kept subtree's beliefs are named by keys whose split into action and
# observation is the model's.
@pytest.mark.parametrize("nA,other", [(70, 300), (300, 70), (3, 8)])
def test_kept_subtree_of_another_model_is_refused(V, nA, other):
    inst, bel = models(nA)
    inst2, bel2 = models(other)
    pom, pom2 = V.Pomdp.from_instance(inst), V.Pomdp.from_instance(inst2)
    b, b2 = V.belief_tensor(inst, bel), V.belief_tensor(inst2, bel2)
    p1, p2 = V.params(300, seed=2), V.params(300, seed=9)
    big = pom if nA > other else pom2
    src = V.Workspace(pom, p1, 3, 3)
    dst, two = (V.Workspace(big, p2, 6, 6) for _ in range(2))
    try:
        r1 = V.plan(pom, b, b.numel(), 3, 3, p1, ws=src)
        o = top_branch(V.tree_dump(src, nA, r1.n_beliefs, r1.n_actions), r1.action)
        for w in (dst, two):
            assert V.reroot(pom, src, r1.action, o, p2, 3, 3, w) > 1
        with pytest.raises(V.VoppError) as e:
            V.plan(pom2, b2, b2.numel(), 3, 3, p2, ws=dst)
        assert e.value.status == V.VOPP_E_INVALID and "kept subtree" in str(e.value)
        x = V.plan(pom, b, b.numel(), 3, 3, p2, ws=dst)
        y = V.plan(pom, b, b.numel(), 3, 3, p2, ws=two)
        same_plan(V, nA, x, dst, y, two)
    finally:
        for w in (src, dst, two):
            w.close()
        pom.close()
        pom2.close()


# Waits inside a launch are bounded: with a bound of no turns at all, a plan in which
# episodes share new beliefs ends with an error, and so do its launches.
@pytest.mark.parametrize("nA,n_p", [(2, 64), (2, 2500), (16, 1500), (64, 900), (70, 900)])
@pytest.mark.parametrize("schedule", [0, 1])
def test_waits_are_bounded(V, nA, n_p, schedule):
    inst = I.tabular_dense(21, 7, nA, 1, with_heuristic=True)
    bel = I.tabular_belief(inst)
    pom = V.Pomdp.from_instance(inst)
    b = V.belief_tensor(inst, bel)
    prm = V.params(n_p, seed=2, schedule=schedule)
    ws, ref = V.Workspace(pom, prm, 5, 5), V.Workspace(pom, prm, 5, 5)
    try:
        ws.wait_limit(0)
        with pytest.raises(V.VoppError) as e:
            V.plan(pom, b, b.numel(), 5, 5, prm, ws=ws)
        assert e.value.status == V.VOPP_E_INTERNAL and "wait" in str(e.value)
        with pytest.raises(V.VoppError):
            V.level_counts(ws)
        ws.wait_limit(-1)
        r = V.plan(pom, b, b.numel(), 5, 5, prm, ws=ws)
        f = V.plan(pom, b, b.numel(), 5, 5, prm, ws=ref)
        same_plan(V, nA, r, ws, f, ref)
    finally:
        ws.close()
        ref.close()
        pom.close()
