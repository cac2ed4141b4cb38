"""Small graphs of one kernel but different LDS sizes, run by threads at once on
streams of their own: the results are the lone ones and every graph keeps its
one-workgroup form.
"""
import threading

import numpy as np
import pytest

from paper_2202_04110_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_threads_with_different_lds_sizes():
    import torch

    from paper_2202_04110_amd import lbp

    specs = [W.ising_grid(8, 1), W.ising_grid(32, 2), W.rbm(30, 30, seed=3), W.chain(4, 900, 2)]
    jobs, errors = [], []
    for s in specs:
        stream = torch.cuda.Stream()
        ctx = lbp.Context(0, stream)
        g = lbp.Graph(ctx, s)
        assert g.form(8, 0.0)[0] == "workgroup"
        g.run_bp(50, 0.5, 0.0)
        jobs.append((ctx, g, g.get_messages()))

    def work(g, want):
        try:
            for _ in range(100):
                g.reset_messages()
                for _ in range(5):
                    g.run_bp(10, 0.5, 0.0)
            np.testing.assert_array_equal(g.get_messages(), want)
            assert g.form(8, 0.0)[0] == "workgroup"
        except Exception as e:  # reported in the test's own thread
            errors.append(e)

    ts = [threading.Thread(target=work, args=(g, want)) for _, g, want in jobs]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for ctx, g, _ in jobs:
        g.free()
        ctx.close()
    assert not errors, errors
