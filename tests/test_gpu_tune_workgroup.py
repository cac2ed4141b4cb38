"""The autotuner chooses between the one-workgroup solver and launched
iterations by time, for the kind of temperature it was called with; the other
kind keeps the rule.  Whatever it chose, the bits are the same, and what it
chose is not slower than the other form by more than a fifth (timed here over
200 iterations, best of nine in turn).
"""
import time

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
    "ising33": lambda: W.ising_grid(33, 102), "potts20x6": lambda: W.potts_grid(20, 6, 1),
    "potts30x5": lambda: W.potts_grid(30, 5, 2), "rbm64": lambda: W.rbm(64, 64, seed=16),
}


@pytest.mark.parametrize("T", [0.0, 0.7])
@pytest.mark.parametrize("name", list(SPECS))
def test_autotune_times_the_workgroup(lbp, ctx, name, T):
    import torch

    spec = SPECS[name]()
    g = lbp.Graph(ctx, spec)
    other = 0.7 if T == 0.0 else 0.0
    g.run_bp(20, 0.5, T)
    want = g.get_messages()
    g.reset_messages()
    g.autotune(0.5, T, reps=20)
    assert not g.get_messages().any()
    chosen = g.form(8, T)[0]
    assert chosen in ("workgroup", "fused", "two_phase", "resident")
    rule = lbp.Graph(ctx, spec)  # with the same choice of fused iterations
    if g.fused:
        rule.use_fused(g.fused_in_use)
        rule.use_automatic(True)
    if g.form(8, other)[0] != "resident":  # (that choice holds at every temperature)
        assert g.form(8, other)[0] == rule.form(8, other)[0]
    rule.free()
    g.run_bp(20, 0.5, T)
    np.testing.assert_array_equal(g.get_messages(), want)
    # launched iterations of the same graph
    ref = lbp.Graph(ctx, spec)
    ref.use_fused(g.fused_in_use) if g.fused else ref.use_automatic(False)
    best = {}
    for _ in range(9):
        for k, x in (("chosen", g), ("launched", ref)):
            x.reset_messages()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            x.run_bp(200, 0.5, T)
            torch.cuda.synchronize()
            best[k] = min(best.get(k, 1.0), time.perf_counter() - t0)
    print("%s T=%g: %s, %.2f us an iteration, launched %.2f" % (name, T, chosen, best["chosen"] * 5e3,
                                                               best["launched"] * 5e3))
    assert best["chosen"] <= 1.2 * best["launched"]
    g.free()
    ref.free()
