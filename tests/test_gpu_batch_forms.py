"""Batches of graphs that have a second message buffer of their own without
pairwise fused iterations (OR/AND graphs, dense three-way graphs): fused
iterations are refused, autotune works and stays two-phase, and runs give each
graph's lone results bitwise.
"""
import numpy as np
import pytest

from paper_2202_04110_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbp():
    from paper_2202_04110_amd import lbp as mod

    return mod


@pytest.fixture(scope="module")
def ctx(lbp):
    c = lbp.Context(0)
    yield c
    c.close()


BATCHES = {
    "deconv": lambda: [W.deconv(seed=4, K=2, tw=4, sd=12, img=13), W.deconv(seed=5, K=3, tw=5, sd=18, img=20)],
    "deconv_potts": lambda: [W.potts_grid(12, 3, 1), W.deconv(seed=4, K=2, tw=4, sd=12, img=13)],
    # both in one graph: pairwise and logical launches
    "union": lambda: [W.disjoint_union([W.ising_grid(9, 2), W.deconv(seed=4, K=2, tw=4, sd=12, img=13)])],
    "triplets": lambda: [W.triplet_grid(20, 3, 6), W.triplet_grid(11, 2, 7)],
    "triplet_potts": lambda: [W.triplet_grid(20, 3, 6), W.potts_grid(12, 3, 1)],
}


@pytest.mark.parametrize("name", list(BATCHES))
def test_batch_without_pairwise_fused_iterations(lbp, ctx, name):
    specs = BATCHES[name]()
    gs = [lbp.Graph(ctx, s) for s in specs]
    b = lbp.Batch(ctx, gs)
    with pytest.raises(lbp.LBPError) as ei:
        b.use_fused(True)
    assert ei.value.code == lbp.LBP_E_INVALID
    for T in (0.0, 0.7):
        assert b.autotune(0.5, T, reps=2) is False
        for iters in (1, 2, 5, 8):
            for g in gs:
                g.reset_messages()
            b.run_bp(iters, 0.5, T)
            for s, g in zip(specs, gs):
                lone = lbp.Graph(ctx, s)
                lone.run_bp(iters, 0.5, T)
                np.testing.assert_array_equal(g.get_messages(), lone.get_messages())
                np.testing.assert_array_equal(g.get_beliefs(), lone.get_beliefs())
                lone.free()
    b.free()
    for g in gs:
        g.free()
