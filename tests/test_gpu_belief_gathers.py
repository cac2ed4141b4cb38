"""Belief sums of every variable path at the edges of its gather: beliefs from
given messages against the FP64 sum.

Tolerance: a sum of k + 1 numbers in any order rounds by at most k times half
an ulp of the sum of their magnitudes: k * 2^-24 * (|theta| + sum |m|) per
entry.
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


def hubs(degrees, states, extra=()):
    """One hub per degree with that many leaves (hub and leaves of the hub's
    state count), then variables of `extra` state counts in no factor."""
    nst, pairs, tabs = [], [], []
    for d, n in zip(degrees, states):
        h = len(nst)
        nst += [n] * (d + 1)
        for j in range(d):
            pairs.append((h, h + 1 + j))
            tabs.append(n)
    nst += list(extra)
    rng = np.random.default_rng(3)
    recs = [{"kind": W.ENUM, "vars": list(p), "logpot": rng.normal(0, 1, n * n)} for p, n in zip(pairs, tabs)]
    ev = rng.normal(0, 1, int(np.sum(nst)))
    return W._general_graph(np.array(nst, np.int32), ev.astype(np.float32), recs, "hubs")


DEGREES = [1, 2, 3, 4, 5, 8, 9, 16, 17, 63, 64, 65, 257, 300, 1025]
CASES = {
    "two": (DEGREES, [2] * 15, [2]), "three": (DEGREES, [3] * 15, [3]), "five": (DEGREES, [5] * 15, [5]),
    "eight": (DEGREES, [8] * 15, [8]), "nine": (DEGREES[:12], [9] * 12, [9]),
    "seventeen": ([1, 3, 20, 70], [17] * 4, []),
    # tiles of several state counts; many states and no edge
    "mixed": ([3, 1, 5, 2, 17, 70, 4], [2, 7, 3, 2, 5, 2, 8], [20, 2, 64]), "lone": ([], [], [20, 2, 64, 3]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_beliefs_match_the_sums(lbp, ctx, name):
    spec = hubs(*CASES[name])
    g = lbp.Graph(ctx, spec)
    off = spec.var_state_off()
    eo = spec.edge_state_off()
    m = np.random.default_rng(4).normal(0, 2, g.ES).astype(np.float32)
    for e in range(spec.num_edges):  # normalised rows, as every iteration leaves them
        m[eo[e]:eo[e + 1]] -= m[eo[e]:eo[e + 1]].max()
    g.set_messages(m)
    b = g.get_beliefs(normalized=False).astype(np.float64)
    want = spec.evidence.astype(np.float64).copy()
    mag = np.abs(want)
    deg = np.zeros(spec.num_vars)
    for e in range(spec.num_edges):
        v = spec.edge_var[e]
        want[off[v]:off[v + 1]] += m[eo[e]:eo[e + 1]]
        mag[off[v]:off[v + 1]] += np.abs(m[eo[e]:eo[e + 1]])
        deg[v] += 1
    tol = np.repeat(deg, spec.var_num_states) * 2.0 ** -24 * mag
    assert (np.abs(b - want) <= tol).all(), float((np.abs(b - want) - tol).max())
    g.free()


@pytest.mark.parametrize("nv", [8192, 8193, 8198])
def test_one_or_four_variables_a_wavefront(lbp, ctx, nv):
    """A wavefront each up to 8192 variables of 17 to 64 edges, four to a
    wavefront (the last one short) above."""
    spec = W.rbm(nv, 17, seed=5)
    g = lbp.Graph(ctx, spec)
    m = np.random.default_rng(4).normal(0, 2, (spec.num_edges, 2)).astype(np.float32)
    m -= m.max(1, keepdims=True)
    g.set_messages(m.reshape(-1))
    b = g.get_beliefs(normalized=False).astype(np.float64).reshape(-1, 2)
    want = spec.evidence.astype(np.float64).reshape(-1, 2).copy()
    mag = np.abs(want)
    np.add.at(want, spec.edge_var, m.astype(np.float64))
    np.add.at(mag, spec.edge_var, np.abs(m.astype(np.float64)))
    tol = np.bincount(spec.edge_var, minlength=spec.num_vars)[:, None] * 2.0 ** -24 * mag
    assert (np.abs(b - want) <= tol).all(), float((np.abs(b - want) - tol).max())
    g.free()
