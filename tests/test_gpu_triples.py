"""Fused iterations of three-way graphs against two-phase ones (a batch of one
graph), bitwise: both form every belief and update with the same additions in
the same order.
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


def scattered(seed, V, F, n):
    """Triples of any three variables, up to sixteen a variable, so tiles mix
    offsets and gathers take more than one round."""
    rng = np.random.default_rng(seed)
    deg = np.zeros(V, int)
    recs = []
    while len(recs) < F:
        vs = rng.choice(V, 3, replace=False)
        if (deg[vs] < 16).all():
            deg[vs] += 1
            recs.append({"kind": W.ENUM, "vars": [int(v) for v in vs], "logpot": rng.normal(0, 1, n ** 3)})
    return W._general_graph(np.full(V, n, np.int32), rng.normal(0, 1, V * n).astype(np.float32), recs, "triples")


SPECS = {
    "one": lambda: W.triplet_grid(3, 2, 1), "g9x3": lambda: W.triplet_grid(9, 3, 2),
    "g64x2": lambda: W.triplet_grid(64, 2, 3), "g65x3": lambda: W.triplet_grid(65, 3, 4),
    "g50x4": lambda: W.triplet_grid(50, 4, 5), "s2": lambda: scattered(6, 100, 400, 2),
    "s3": lambda: scattered(7, 90, 450, 3), "s4": lambda: scattered(8, 40, 130, 4),
    # both state counts in one graph: two launches an iteration
    "both": lambda: W.disjoint_union([W.triplet_grid(12, 3, 9), W.triplet_grid(11, 2, 10)]),
}


@pytest.mark.parametrize("T", [0.0, 0.7])
@pytest.mark.parametrize("name", list(SPECS))
def test_fused_triples_match_two_phase(lbp, ctx, name, T):
    spec = SPECS[name]()
    g, ref = lbp.Graph(ctx, spec), lbp.Graph(ctx, spec)
    batch = lbp.Batch(ctx, [ref])
    rng = np.random.default_rng(1)
    for iters, d in ((2, 0.5), (5, 0.3), (8, 0.0), (8, 0.0)):
        m0 = rng.normal(0, 1, g.ES).astype(np.float32)
        lp = rng.normal(0, 1, g.Tn).astype(np.float32)
        for x in (g, ref):
            x.set_log_potentials(lp)
            x.set_messages(m0)
        g.run_bp(iters, d, T)
        batch.run_bp(iters, d, T)
        np.testing.assert_array_equal(g.get_messages(), ref.get_messages())
        np.testing.assert_array_equal(g.get_beliefs(), ref.get_beliefs())
    batch.free()
    g.free()
    ref.free()
