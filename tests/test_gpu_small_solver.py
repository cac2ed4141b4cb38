"""The one-workgroup solver of small pairwise graphs against launched
iterations (a batch of one graph), bitwise.

The two repeat the same additions and updates in the same order, so the
comparison is exact; the launched path itself is held to the oracle elsewhere.
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


def _isolated(spec):
    """Two variables in no factor, one of another state count, at the end."""
    spec = spec.copy()
    n = int(spec.var_num_states[0])
    return W._pairwise_graph(np.concatenate([spec.var_num_states, [n, n + 3]]).astype(np.int32),
                             np.concatenate([spec.evidence, np.ones(2 * n + 3, np.float32)]),
                             spec.edge_var.reshape(-1, 2), spec.log_potentials, "isolated")


SPECS = {
    # one factor; one tile and a bit; two variable tiles per wavefront
    "pair": lambda: W.chain(1, 2, 2), "chain65": lambda: W.chain(2, 66, 3), "chain2000": lambda: W.chain(3, 2000, 2),
    # grids of every state count, ragged tiles; the largest that fit and one that does not
    "g2": lambda: W.ising_grid(32, 4), "g2max": lambda: W.ising_grid(45, 5), "g2over": lambda: W.ising_grid(46, 5),
    "g3": lambda: W.potts_grid(33, 3, 6), "g4": lambda: W.potts_grid(23, 4, 7), "g5": lambda: W.potts_grid(17, 5, 8),
    "g6": lambda: W.potts_grid(13, 6, 9), "g7": lambda: W.potts_grid(11, 7, 10), "g8": lambda: W.potts_grid(22, 8, 11),
    # degrees above four and above sixteen, both in one graph
    "deg12": lambda: W.random_pairwise(12, 300, 900, 4),
    "deg40": lambda: W.random_pairwise(13, 40, 500, 2, max_degree=40),
    "rbm15": lambda: W.rbm(15, 15, seed=14), "rbm17x16": lambda: W.rbm(17, 16, seed=15),
    "rbm64": lambda: W.rbm(64, 64, seed=16), "rbm65x64": lambda: W.rbm(65, 64, seed=17),
    "isolated": lambda: _isolated(W.potts_grid(9, 3, 18)),
}


@pytest.mark.parametrize("T", [0.0, 0.7])
@pytest.mark.parametrize("name", list(SPECS))
def test_small_solver_matches_launched(lbp, ctx, name, T):
    spec = SPECS[name]()
    g, ref = lbp.Graph(ctx, spec), lbp.Graph(ctx, spec)
    batch = lbp.Batch(ctx, [ref])
    rng = np.random.default_rng(1)
    for iters, d in ((2, 0.5), (7, 0.3), (20, 0.0)):
        m0 = rng.normal(0, 1, g.ES).astype(np.float32)
        ev = rng.normal(0, 1, g.VS).astype(np.float32)
        lp = rng.normal(0, 1, g.Tn).astype(np.float32)
        for x in (g, ref):
            x.set_evidence(ev)
            x.set_log_potentials(lp)
            x.set_messages(m0)
        g.run_bp(iters, d, T)
        batch.run_bp(iters, d, T)
        np.testing.assert_array_equal(g.get_messages(), ref.get_messages())
        np.testing.assert_array_equal(g.get_beliefs(), ref.get_beliefs())
    batch.free()
    g.free()
    ref.free()
