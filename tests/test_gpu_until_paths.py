"""lbp_run_bp_until on the paths its checks take (fused pairs, the odd fused
iteration, three-way views, one workgroup, two-phase): iterations, residual and
messages bitwise those of lbp_run_bp_until_noalloc, which checks after
two-phase iterations whatever the graph.
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
    "potts50": (lambda: W.potts_grid(50, 5, 1), True), "potts50_plain": (lambda: W.potts_grid(50, 5, 1), False),
    "ising100": (lambda: W.ising_grid(100, 2), True), "triplet30": (lambda: W.triplet_grid(30, 3, 3), False),
    "small": (lambda: W.potts_grid(9, 3, 4), True), "rbm": (lambda: W.rbm(90, 30, seed=5), False),
}


@pytest.mark.parametrize("check", [1, 2, 5, 10])
@pytest.mark.parametrize("name", list(SPECS))
def test_until_matches_noalloc(lbp, ctx, name, check):
    make, fused = SPECS[name]
    spec = make()
    for tol, most in ((1e-3, 60), (0.0, 7), (0.0, 1)):
        out = []
        for noalloc in (False, True):
            g = lbp.Graph(ctx, spec)
            if fused and not noalloc:
                g.use_fused(True)
            for T in (1.0, 0.0):
                g.reset_messages()
                run = g.run_bp_until_noalloc if noalloc else g.run_bp_until
                done, r = run(most, 0.5, T, tol, check)
                out.append((noalloc, done, r, g.get_messages(), g.get_beliefs()))
                again = run(most, 0.5, T, tol, check)  # from where the first stopped
                out.append((noalloc, *again, g.get_messages(), g.get_beliefs()))
            g.free()
        half = len(out) // 2
        for a, b in zip(out[:half], out[half:]):
            assert a[1] == b[1] and a[2] == b[2], (name, check, tol, a[1:3], b[1:3])
            np.testing.assert_array_equal(a[3], b[3])
            np.testing.assert_array_equal(a[4], b[4])
