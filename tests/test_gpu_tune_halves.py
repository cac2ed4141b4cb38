"""The autotuner and its cache on fused launches that run two wavefronts a
tile: such launches take no shape, so none is searched, and none is recorded
for the other graphs of their size bucket.
"""
import json

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


def test_no_search_of_shapes_that_are_not_taken(lbp, ctx):
    g = lbp.Graph(ctx, W.potts_grid(60, 5, 1))
    i = next(i for i, ln in enumerate(g.launches()) if ln["phase"] == 1)
    g.set_fused_launch(i, 1, 3)
    g.use_automatic(True)
    assert g.form(2, 1.0)[1] == {0}
    for _ in range(3):  # twelve candidates at 2 iterations each: noise would pick another
        g.autotune(0.5, 1.0, reps=2)
        ln = g.launches()[i]
        assert (ln["fused_wpb"], ln["fused_variant"]) == (1, 3)
    g.free()


def test_cache_records_no_shape_for_them(lbp, ctx, tmp_path):
    from paper_2202_04110_amd import tune

    path = str(tmp_path / "tune.json")

    def apply(L):
        g = lbp.Graph(ctx, W.potts_grid(L, 5, 1))
        r = tune.apply_or_tune(g, 0.5, 1.0, reps=3, path=path, packaged=False)
        ln = [x for x in g.launches() if x["phase"] == 1][0]
        out = r["source"], g.form(2, 1.0)[1], (ln["fused_wpb"], ln["fused_variant"]), r["shapes"]
        g.free()
        return out

    def recorded():
        return [e for k, e in json.load(open(path)).items() if "|p1|" in k]

    # either side of the size line, in one bucket of every key
    src, halves, _, shapes = apply(98)
    assert src == "tuned" and halves == {0} and len(recorded()) == 1 and "fused_wpb" not in recorded()[0]
    assert all("fused_wpb" in s and "fused_variant" in s for s in shapes)
    src, halves, shape, _ = apply(112)
    assert src == "tuned" and halves == set()
    assert len(recorded()) == 1 and (recorded()[0]["fused_wpb"], recorded()[0]["fused_variant"]) == shape
    src, halves, _, _ = apply(98)
    assert src == "cache" and halves == {0}
    assert apply(112)[:3] == ("cache", set(), shape)
