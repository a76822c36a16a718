"""Many episodes, few beliefs: the levels at which the lanes of a wavefront send one
of them to a new belief, and the edge of the rule that says which levels those are
(512 episodes to each of the (|A| |O|)^(level + 1) beliefs a level may create).

Each plan is held to the serial oracle draw by draw (tests/drawcheck.py).
"""

import numpy as np
import pytest

from paper_2510_27191_amd import instances as I
from tests.drawcheck import forced_parity

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
