"""The learned call against the opening-angle call with the same lists."""
import numpy as np
import pytest

from paper_1005_5384_amd import learned as L
from paper_1005_5384_amd import octgrav as og
from paper_1005_5384_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,same_waves", [(230000, True), (70000, False), (3000, False)])
def test_same_lists_same_forces(n, same_waves):
    """From 11000 work items up both calls walk with one wave per item: the same bits.  Below that the
    opening-angle call's waves add up their own parts of the lists: equal to rounding."""
    pos, m = W.plummer(n, 13)
    T = og.Tree(pos, m, 16, 64)
    assert (T.stats["n_work"] > 11000) == same_waves
    T.set_mac(og.Mlp(L.init_params(1)), 0.45, 1.0, 0.0, float("inf"))  # every band cell opened
    acc, pot = T.forces(0.6, 0.01)
    g = T.group_counts()
    T.set_mac(None)
    a2, p2 = T.forces(0.45, 0.01)
    assert np.array_equal(g[:, :3], T.group_counts()[:, :3])
    if same_waves:
        assert (acc == a2).all() and (pot == p2).all()
    else:
        # compensated sums of the same terms, rounded to FP32: within an ulp of the vector's largest component
        ulp = 2.0 ** -23
        assert ((acc - a2).abs().amax(1) <= ulp * a2.abs().amax(1)).all()
        assert ((pot - p2).abs() <= ulp * p2.abs()).all()
