"""The end of an anytime plan, decided in a launch whose blocks still start.

The root backup decides that the plan is over, in the same launch as the sweep
of the full beliefs (or as its block's other wavefronts, for long rows).  Blocks
that start after that decision still belong to the plan's last iteration.
A plan wide enough to fill that launch, beside other work that holds up its
blocks, has to give the plain plan's tree every time.
"""

import pytest

from paper_2510_27191_amd import instances as I
from tests.test_gpu_failed_plans import same_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_27191_amd import vopp
    vopp.lib()
    return vopp


# (The sums' resolution is the finest for these sizes, whatever the iterations,
# so plain and anytime plans agree bit for bit.)
@pytest.mark.parametrize("nA,nO,n_p,K,depth", [(3, 64, 20000, 4, 3), (16, 8, 20000, 3, 3),
                                               (70, 3, 4000, 3, 2), (64, 1, 300, 5, 1)])
def test_plan_beside_other_work(V, nA, nO, n_p, K, depth):
    import torch
    inst = I.tabular_dense(21, 16, nA, nO)
    bel = I.tabular_belief(inst)
    pom = V.Pomdp.from_instance(inst)
    b = V.belief_tensor(inst, bel)
    prm = V.params(n_p, seed=4)
    ws, ref = V.Workspace(pom, prm, K, depth), V.Workspace(pom, prm, K, depth)
    side = torch.cuda.Stream()
    x = torch.zeros(1 << 22, device="cuda")
    try:
        f = V.plan(pom, b, b.numel(), K, depth, prm, ws=ref)
        for _ in range(6):
            with torch.cuda.stream(side):
                for _ in range(40):
                    x.add_(1.0)
            r, k = V.plan_anytime(pom, b, b.numel(), K, depth, 1e6, prm, ws=ws)
            assert k == K
            same_plan(V, nA, r, ws, f, ref)
        # ... and one that stops after its first iteration.
        f1 = V.plan(pom, b, b.numel(), 1, depth, prm, ws=ref)
        for _ in range(3):
            with torch.cuda.stream(side):
                for _ in range(40):
                    x.add_(1.0)
            r, k = V.plan_anytime(pom, b, b.numel(), K, depth, 1e-6, prm, ws=ws)
            assert k == 1
            same_plan(V, nA, r, ws, f1, ref)
    finally:
        torch.cuda.synchronize()
        ws.close()
        ref.close()
        pom.close()
