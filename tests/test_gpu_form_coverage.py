"""Every variant of the iteration forms against two-phase iterations (a batch
of one graph), bitwise, with the form asserted: fused launches of every state
count, launch shape and variant; the one-workgroup solver with one, two, four
and eight factor tiles a wavefront; early exit in one workgroup; relay
iterations with both edge orders, narrow and wide factors and other factors
beside them.
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


def grid(L, n):
    return W.ising_grid(L, 1) if n == 2 else W.potts_grid(L, n, 1)


def match(lbp, ctx, spec, T, form, prepare=lambda g: None, iters=((2, 0.5), (7, 0.3), (12, 0.0)), seed=1):
    g, ref = lbp.Graph(ctx, spec), lbp.Graph(ctx, spec)
    batch = lbp.Batch(ctx, [ref])
    try:
        prepare(g)
        assert g.form(8, T)[0] == form
        rng = np.random.default_rng(seed)
        for n, d in iters:
            m0 = rng.normal(0, 1, g.ES).astype(np.float32)
            ev = rng.normal(0, 1, g.VS).astype(np.float32)
            for x in (g, ref):
                x.set_evidence(ev)
                x.set_messages(m0)
            g.run_bp(n, d, T)
            batch.run_bp(n, d, T)
            np.testing.assert_array_equal(g.get_messages(), ref.get_messages())
            np.testing.assert_array_equal(g.get_beliefs(), ref.get_beliefs())
    finally:
        batch.free()
        g.free()
        ref.free()


@pytest.mark.parametrize("T", [0.0, 0.7])
@pytest.mark.parametrize("n", range(2, 9))
def test_fused_launches_of_every_variant(lbp, ctx, n, T):
    """Grids and scattered slots, one wavefront a tile, all twelve shapes."""
    for spec in (grid(41, n), W.random_pairwise(7, 500, 1300, n, max_degree=9)):
        for w in (1, 2, 4):
            for v in range(4):
                def shaped(g):
                    g.use_fused(True)
                    g.use_automatic(False)
                    i = [ln["phase"] for ln in g.launches()].index(1)
                    g.set_fused_launch(i, w, v)
                    assert g.form(8, T)[1] == set()
                match(lbp, ctx, spec, T, "fused", shaped, iters=((5, 0.3),), seed=10 * w + v)


SMALL = {
    # name: spec, temperatures at which the rule takes it
    "n2_one": (lambda: grid(16, 2), (0.0, 0.7)), "n2_two": (lambda: grid(32, 2), (0.0, 0.7)),
    "n2_four": (lambda: grid(45, 2), (0.0, 0.7)),
    "n2_eight": (lambda: W.random_pairwise(13, 200, 5000, 2, max_degree=64), (0.0,)),
    "n3_one": (lambda: grid(20, 3), (0.0, 0.7)), "n3_two": (lambda: grid(30, 3), (0.0, 0.7)),
    "n3_four": (lambda: grid(40, 3), (0.0, 0.7)), "n4_one": (lambda: grid(21, 4), (0.0, 0.7)),
    "n4_two": (lambda: grid(31, 4), (0.0, 0.7)), "n5_one": (lambda: grid(16, 5), (0.0, 0.7)),
    "n5_two": (lambda: grid(26, 5), (0.0, 0.7)), "n6": (lambda: grid(22, 6), (0.0, 0.7)),
    "n7": (lambda: grid(19, 7), (0.0, 0.7)), "n8": (lambda: grid(17, 8), (0.0, 0.7)),
    "layer": (lambda: W.rbm(50, 43, seed=9), (0.0, 0.7)),
}


@pytest.mark.parametrize("name,T", [(k, T) for k, (_, Ts) in SMALL.items() for T in Ts])
def test_one_workgroup(lbp, ctx, name, T):
    match(lbp, ctx, SMALL[name][0](), T, "workgroup")


@pytest.mark.parametrize("T", [0.0, 1.0])
@pytest.mark.parametrize("check", [1, 2, 5, 10])
def test_early_exit_in_one_workgroup(lbp, ctx, check, T):
    spec = grid(9, 3)
    for tol, most in ((1e-3, 60), (0.0, 7), (0.0, 1)):
        g, ref = lbp.Graph(ctx, spec), lbp.Graph(ctx, spec)
        assert g.form(8, T)[0] == "workgroup"
        for _ in range(2):  # again from where the first stopped
            assert g.run_bp_until(most, 0.5, T, tol, check) == ref.run_bp_until_noalloc(most, 0.5, T, tol, check)
            np.testing.assert_array_equal(g.get_messages(), ref.get_messages())
        g.free()
        ref.free()


def products(seed, inputs, outputs, fan, ands_first, extra=None):
    """OR factors over `fan` products each, every product the child of one AND
    of two inputs and a parent of one OR (its first edge when ands_first is
    false); products, then outputs, after the inputs.  extra: dense factors
    among the inputs, pairwise of 2 x 2 or three-way."""
    rng = np.random.default_rng(seed)
    first = inputs + 64 - inputs % 64
    n = first + outputs * (fan + 1)
    ands, ors = [], []
    for o in range(outputs):
        prods = first + o * fan + np.arange(fan)
        for p in prods:
            a, b = rng.choice(inputs, 2, replace=False)
            ands.append({"kind": W.AND, "vars": [int(a), int(b), int(p)]})
        ors.append({"kind": W.OR, "vars": [int(p) for p in prods] + [first + outputs * fan + o]})
    recs = ands + ors if ands_first else ors + ands
    for i in range(0, inputs - 2, 3) if extra else ():
        recs.append({"kind": W.ENUM, "vars": [i, i + 1, i + 2][:extra], "logpot": rng.normal(0, 1, 2 ** extra)})
    return W._general_graph(np.full(n, 2, np.int32), rng.normal(0, 1, 2 * n).astype(np.float32), recs, "products")


RELAY = {
    "ands_first": lambda: products(2, 40, 12, 40, True), "ors_first": lambda: products(3, 40, 12, 40, False),
    "narrow": lambda: products(4, 20, 120, 6, True), "narrow_ors_first": lambda: products(5, 20, 120, 3, False),
    "wide": lambda: products(6, 60, 3, 700, True), "wide_ors_first": lambda: products(7, 60, 3, 257, False),
    "pairs": lambda: products(8, 50, 10, 70, True, extra=2), "triples": lambda: products(9, 50, 10, 70, False, extra=3),
    "beside_potts": lambda: W.disjoint_union([W.potts_grid(7, 3, 1), products(10, 30, 20, 40, False)]),
}


@pytest.mark.parametrize("T", [0.0, 0.5])
@pytest.mark.parametrize("name", list(RELAY))
def test_relay(lbp, ctx, name, T):
    match(lbp, ctx, RELAY[name](), T, "relay", iters=((2, 0.5), (5, 0.3), (8, 0.0), (1, 0.5)))
