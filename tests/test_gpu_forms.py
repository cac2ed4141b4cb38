"""Which form lbp_run_bp takes: the rules from upload, and every explicit choice
(use_fused, use_resident, set_fused_launch, use_automatic) honoured as it
stands; all forms of a graph give the same bits.
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
    # spec, T, form from upload, has pairwise fused iterations, fits the resident solver
    "ising33": (lambda: W.ising_grid(33, 102), 0.0, "workgroup", True, None),
    "potts9x3": (lambda: W.potts_grid(9, 3, 4), 1.0, "workgroup", True, None),
    "rbm20": (lambda: W.rbm(20, 20, 406), 0.05, "workgroup", False, True),
    "potts60x5": (lambda: W.potts_grid(60, 5, 1), 1.0, "two_phase", True, None),
    "potts112x8": (lambda: W.potts_grid(112, 8, 2), 1.0, "two_phase", True, False),
    "triplet30x3": (lambda: W.triplet_grid(30, 3, 3), 0.7, "fused", False, False),
    "deconv13": (lambda: W.deconv(seed=4, K=2, tw=4, sd=12, img=13), 0.0, "relay", False, None),
    "rbm90x30": (lambda: W.rbm(90, 30, seed=5), 1.0, "two_phase", False, None),
}


def run(g, T):
    g.reset_messages()
    g.run_bp(7, 0.5, T)
    m = g.get_messages()
    g.reset_messages()
    until = g.run_bp_until(9, 0.5, T, 0.0, 4)
    return m, g.get_beliefs(), until, g.get_messages()


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("name", list(SPECS))
def test_choices_hold_and_change_no_bits(lbp, ctx, name):
    make, T, auto, fused, resident = SPECS[name]
    spec = make()
    g = lbp.Graph(ctx, spec)
    assert g.fused == fused and g.form(8, T)[0] == auto
    assert g.form(1, T)[0] == "two_phase"
    first = run(g, T)
    ref = lbp.Graph(ctx, spec)  # whatever the graph: two-phase between and at checks
    ref.run_bp_until_noalloc(9, 0.5, T, 0.0, 4)
    np.testing.assert_array_equal(first[3], ref.get_messages())
    ref.free()
    if resident is not None:
        assert g.resident_state[0] == resident
    g.use_fused(False)
    assert g.form(8, T)[0] == "two_phase"
    assert same(run(g, T), first)
    g.use_automatic(True)
    assert g.form(8, T)[0] == auto
    if fused:
        g.use_fused(True)
        assert g.form(8, T)[0] == "fused"
        assert same(run(g, T), first)
    if g.resident_state[0]:
        g.use_resident(True)
        assert g.form(8, T)[0] == "resident"
        assert same(run(g, T), first)
        g.use_resident(False)
        assert g.form(8, T)[0] == ("fused" if fused else "two_phase")
        assert same(run(g, T), first)
    g.use_automatic(True)  # the choice of fused iterations stays for runs no rule takes
    assert g.form(8, T)[0] == ("fused" if auto == "two_phase" and fused else auto)
    assert same(run(g, T), first)
    g.use_automatic(False)
    assert g.form(8, T)[0] == ("fused" if fused else "two_phase")
    assert same(run(g, T), first)
    with pytest.raises(lbp.LBPError):
        g.form(-1, T)
    g.free()


def test_fused_shapes_that_were_set_are_run(lbp, ctx):
    """Two wavefronts a tile below the size line, one once a shape was set."""
    spec = W.disjoint_union([W.potts_grid(40, 3, 13), W.potts_grid(30, 5, 14)])
    g = lbp.Graph(ctx, spec)
    g.use_fused(True)
    assert g.form(4, 1.0) == ("fused", {0, 1})
    assert g.form(4, 0.0) == ("fused", {0})  # max-product of five states: one wavefront a tile
    g.run_bp(6, 0.5, 1.0)
    want = g.get_messages()
    nv = sum(l["phase"] == 0 for l in g.launches())
    g.set_fused_launch(nv + 1, 2, 1)
    assert g.form(4, 1.0) == ("fused", {0})
    g.reset_messages()
    g.run_bp(6, 0.5, 1.0)
    np.testing.assert_array_equal(g.get_messages(), want)
    g.use_automatic(True)
    assert g.form(4, 1.0) == ("fused", {0, 1})
    g.use_automatic(False)
    assert g.form(4, 1.0) == ("fused", set())
    g.free()
    for spec, half in ((W.potts_grid(108, 5, 6), {0}), (W.potts_grid(112, 5, 7), set()),
                       (W.random_pairwise(12, 300, 900, 4), set())):
        g = lbp.Graph(ctx, spec)
        assert g.form(4, 1.0)[1] == half  # 384 tiles at T > 0; at most four edges a variable
        g.free()


@pytest.mark.parametrize("name", ["ising33", "potts60x5", "triplet30x3", "deconv13"])
def test_applied_tables_keep_the_rules(lbp, ctx, name, tmp_path):
    """Applying shapes from a table is no explicit choice of a form."""
    from paper_2202_04110_amd import tune

    make, T, auto, fused, _ = SPECS[name]
    path = str(tmp_path / "tune.json")
    got = []
    for source in ("tuned", "cache"):
        g = lbp.Graph(ctx, make())
        assert tune.apply_or_tune(g, 0.5, T, reps=3, path=path, packaged=False)["source"] == source
        got.append((g.form(8, T), g.fused_in_use))
        g.free()
    assert got[0] == got[1]
