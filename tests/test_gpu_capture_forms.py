"""Runs captured into a caller's HIP graph (a context without captured loops of
its own, on the capturing stream): each form's launches replay with the eager
bits, with other work and synchronisations between the replays.
"""
import numpy as np
import pytest

from paper_2202_04110_amd import workloads as W

pytestmark = pytest.mark.gpu

SPECS = {
    "workgroup": (lambda: W.ising_grid(20, 1), 0.0, "workgroup"),
    "halves": (lambda: W.potts_grid(60, 5, 2), 1.0, "fused"),
    "triples": (lambda: W.triplet_grid(30, 3, 3), 0.7, "fused"),
    "relay": (lambda: W.deconv(seed=4, K=2, tw=4, sd=12, img=13), 0.0, "relay"),
    "two_phase": (lambda: W.rbm(90, 30, seed=5), 1.0, "two_phase"),
}


@pytest.mark.parametrize("name", list(SPECS))
def test_captured_runs_replay(name):
    import torch

    from paper_2202_04110_amd import lbp

    make, T, form = SPECS[name]
    spec = make()
    ctx = lbp.Context(0)
    ctx.use_graphs(False)
    g = lbp.Graph(ctx, spec)
    if g.fused and form == "fused":
        g.use_fused(True)
        g.use_automatic(True)
    assert g.form(6, T)[0] == form
    want = []
    g.reset_messages()
    for _ in range(4):
        g.run_bp(6, 0.5, T)
        want.append(g.get_messages())
    g.reset_messages()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        ctx.set_stream(side)
        g.run_bp(6, 0.5, T)
    ctx.set_stream(torch.cuda.current_stream())
    assert not g.get_messages().any()  # captured, not run
    for w in want:
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(g.get_messages(), w)
        torch.zeros(1000, device="cuda").normal_()
        g.get_beliefs()
        torch.cuda.synchronize()
    del graph
    g.free()
    ctx.close()
