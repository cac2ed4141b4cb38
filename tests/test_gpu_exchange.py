"""Flat-order exchange of rows longer and shorter than the eight values the
kernels keep in flight: what goes in comes out, bitwise, and the read-out
agrees with FP64 on wide variables.

Read-out tolerance: q = B - max or B - LSE, differences of values below 16 in
magnitude: 4 half-ulps of 16 (4 * 16 * 2^-24) for the subtractions and the
FP32 exponentials' sum (relative 64 * 2^-23 over at most 64 states).
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


@pytest.mark.parametrize("states", [[2, 2], [3, 8], [8, 9], [7, 17], [16, 33], [2, 62]])
def test_rows_round_trip(lbp, ctx, states):
    import torch

    spec = W.single_enum(5, states)
    g = lbp.Graph(ctx, spec)
    rng = np.random.default_rng(6)
    ev, lp, m = (rng.normal(0, 1, k).astype(np.float32) for k in (g.VS, g.Tn, g.ES))
    m[: states[0]] -= m[: states[0]].max()
    m[states[0]:] -= m[states[0]:].max()
    g.set_evidence(torch.from_numpy(ev).cuda())
    g.set_messages(m)
    np.testing.assert_array_equal(g.get_messages(), m)
    np.testing.assert_array_equal(g.get_beliefs(normalized=False), ev + m)  # one edge each: one FP32 addition
    for T in (0.0, 1.0):
        g.set_log_potentials(torch.from_numpy(lp).cuda())
        g.run_bp(0, 0.5, T)  # only the temperature of the read-out
        q, mp = g.get_beliefs().astype(np.float64), g.decode_map()
        b = (ev + m).astype(np.float64)
        for v, off in ((0, 0), (1, states[0])):
            x = b[off:off + states[v]]
            z = x.max() if T == 0 else x.max() + np.log(np.exp(x - x.max()).sum())
            assert np.abs(q[off:off + states[v]] - (x - z)).max() <= 4 * 16 * 2.0 ** -24 + 64 * 2.0 ** -23
            assert mp[v] == x.argmax()
    # the tables: one max-product step from zero messages at no damping is
    # max over the other slot of (table + its evidence), normalised
    g.reset_messages()
    g.set_evidence(np.zeros(g.VS, np.float32))
    g.run_bp(1, 0.0, 0.0)
    t = lp.reshape(states).astype(np.float32)
    u = np.concatenate([t.max(1) - t.max(), t.max(0) - t.max()])
    np.testing.assert_allclose(g.get_messages(), u, rtol=0, atol=4 * 16 * 2.0 ** -24)
    g.free()
