"""Fused iterations with two wavefronts a tile against two-phase ones (a batch
of one graph), bitwise, around the sizes where the rule for them turns and with
ragged and idle lanes.
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


SPECS = {
    # two states: 512 tiles at 126 x 126; others at T > 0: 384 tiles
    "n2": lambda: W.ising_grid(70, 1), "n2_at": lambda: W.ising_grid(126, 2),
    "n2_past": lambda: W.ising_grid(130, 3), "n3": lambda: W.potts_grid(64, 3, 4),
    "n4": lambda: W.potts_grid(71, 4, 5), "n5_at": lambda: W.potts_grid(108, 5, 6),
    "n5_past": lambda: W.potts_grid(112, 5, 7), "n6": lambda: W.potts_grid(50, 6, 8),
    "n7": lambda: W.potts_grid(37, 7, 9), "n8": lambda: W.potts_grid(45, 8, 10),
    # slots that are not consecutive variables; two classes in one graph
    "chain": lambda: W.chain(11, 3000, 3), "scattered": lambda: W.random_pairwise(12, 3000, 4000, 5, max_degree=4),
    "both": lambda: W.disjoint_union([W.potts_grid(40, 3, 13), W.potts_grid(30, 5, 14)]),
}


@pytest.mark.parametrize("T", [0.0, 0.7])
@pytest.mark.parametrize("name", list(SPECS))
def test_half_tiles_match_two_phase(lbp, ctx, name, T):
    spec = SPECS[name]()
    g, ref = lbp.Graph(ctx, spec), lbp.Graph(ctx, spec)
    g.use_fused(True)
    batch = lbp.Batch(ctx, [ref])
    m0 = np.random.default_rng(1).normal(0, 1, g.ES).astype(np.float32)
    for iters, d in ((2, 0.5), (5, 0.3), (12, 0.0)):
        for x in (g, ref):
            x.set_messages(m0)
        g.run_bp(iters, d, T)
        batch.run_bp(iters, d, T)
        np.testing.assert_array_equal(g.get_messages(), ref.get_messages())
    batch.free()
    g.free()
    ref.free()
