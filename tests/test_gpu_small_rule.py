"""The rule for the one-workgroup solver compares with the launched iterations
the graph would run instead: two-phase ones as uploaded, fused ones where those
are in use.  Grids on both sides of either line at T = 1; max-product always.
"""
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


# side, states: in one workgroup as uploaded, and with fused iterations in use
GRIDS = [(38, 2, True, True), (42, 2, True, True), (45, 2, True, False), (32, 3, True, True),
         (36, 3, True, False), (23, 4, True, True), (26, 4, True, False), (20, 5, True, True),
         (28, 5, False, False), (18, 6, True, True), (20, 6, True, False), (22, 6, True, False),
         (16, 7, True, True), (18, 7, True, False), (16, 8, True, True), (18, 8, True, False),
         (22, 8, False, False)]


@pytest.mark.parametrize("L,n,plain,fused", GRIDS)
def test_rule_compares_with_what_would_run(lbp, ctx, L, n, plain, fused):
    g = lbp.Graph(ctx, W.potts_grid(L, n, 1) if n > 2 else W.ising_grid(L, 1))
    assert g.form(50, 1.0)[0] == ("workgroup" if plain else "two_phase")
    assert g.form(50, 0.0)[0] == "workgroup"
    g.use_fused(True)
    g.use_automatic(True)
    assert g.form(50, 1.0)[0] == ("workgroup" if fused else "fused")
    assert g.form(50, 0.0)[0] == "workgroup"
    g.free()


@pytest.mark.parametrize("length,fused", [(500, True), (700, False)])
def test_rule_on_chains(lbp, ctx, length, fused):
    g = lbp.Graph(ctx, W.chain(3, length, 6))
    assert g.form(50, 1.0)[0] == "workgroup"
    g.use_fused(True)
    g.use_automatic(True)
    assert g.form(50, 1.0)[0] == ("workgroup" if fused else "fused")
    g.free()
