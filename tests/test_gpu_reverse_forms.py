"""The one-launch reverse step of pairwise graphs against the four-launch one,
bitwise: the same graph beside a factor of unequal slots takes the latter.
Also against the FP64 oracle for eight states on both sides of the size where
the one-launch step ends; tolerance as in test_gpu_adjoint (2e-4 of the largest
gradient).
"""
import numpy as np
import pytest

from oracle import OracleGraph
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


def gradients(lbp, ctx, spec, gq, iters, d, T, k):
    import torch

    g = lbp.Graph(ctx, spec)
    out = []
    for _ in range(2):  # a record, and a second one into the same workspace
        g.reset_messages()
        g.run_bp_record(iters, d, T, k)
        for _ in range(2):  # the record stays valid
            gphi, gth = torch.zeros(g.Tn, device="cuda"), torch.zeros(g.VS, device="cuda")
            g.backward(torch.from_numpy(gq.astype(np.float32)).cuda(), gphi, gth)
            out.append((gphi.cpu().numpy(), gth.cpu().numpy()))
    g.free()
    for a, b in out[1:]:
        np.testing.assert_array_equal(a, out[0][0])
        np.testing.assert_array_equal(b, out[0][1])
    return out[0]


SPECS = {
    "n2": lambda: W.ising_grid(33, 1), "n3": lambda: W.potts_grid(21, 3, 2), "n4": lambda: W.potts_grid(40, 4, 3),
    "n5": lambda: W.potts_grid(23, 5, 4), "n6": lambda: W.potts_grid(17, 6, 5), "n7": lambda: W.potts_grid(13, 7, 6),
    "n8": lambda: W.potts_grid(40, 8, 7),
    # scattered slots; more than four and more than eight edges a variable
    "scattered": lambda: W.random_pairwise(8, 700, 1100, 5, max_degree=4),
    "many": lambda: W.random_pairwise(9, 300, 900, 4), "dense": lambda: W.random_pairwise(10, 60, 440, 3, max_degree=16),
    "dense8": lambda: W.random_pairwise(11, 150, 600, 8, max_degree=12),
    "both": lambda: W.disjoint_union([W.potts_grid(20, 3, 12), W.potts_grid(15, 6, 13)]),
}


@pytest.mark.parametrize("iters,k", [(15, 4), (6, 1), (9, 20)])
@pytest.mark.parametrize("name", list(SPECS))
def test_one_launch_steps_match_four(lbp, ctx, name, iters, k):
    spec = SPECS[name]()
    beside = W.disjoint_union([spec, W.single_enum(3, [2, 3])])  # no fused form for the whole
    g = lbp.Graph(ctx, spec)
    assert g.fused and max(ln["items"] for ln in g.launches()) <= 256  # (eight states: up to 256 tiles)
    g.free()
    g = lbp.Graph(ctx, beside)
    assert not g.fused
    g.free()
    gq = np.random.default_rng(5).normal(0, 1, beside.num_var_states)
    VS, Tn = spec.num_var_states, spec.num_logpots
    gphi, gth = gradients(lbp, ctx, spec, gq[:VS], iters, 0.4, 0.8, k)
    wphi, wth = gradients(lbp, ctx, beside, gq, iters, 0.4, 0.8, k)
    np.testing.assert_array_equal(gphi, wphi[:Tn])
    np.testing.assert_array_equal(gth, wth[:VS])


@pytest.mark.parametrize("L", [88, 92])
def test_eight_states_on_both_sides_of_the_line(lbp, ctx, L):
    spec = W.potts_grid(L, 8, 1)
    g = lbp.Graph(ctx, spec)
    tiles = max(ln["items"] for ln in g.launches())
    assert (tiles <= 256) == (L == 88)
    g.free()
    og = OracleGraph(spec)
    gq = np.random.default_rng(6).normal(0, 1, og.VS)
    ophi, oth, _ = og.backward(8, 0.5, 1.0, gq)
    gphi, gth = gradients(lbp, ctx, spec, gq, 8, 0.5, 1.0, 3)
    scale = max(1.0, float(np.abs(ophi).max()), float(np.abs(oth).max()))
    assert np.abs(gphi - ophi).max() <= 2e-4 * scale and np.abs(gth - oth).max() <= 2e-4 * scale
