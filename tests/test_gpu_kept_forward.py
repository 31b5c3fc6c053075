"""The proposal network's activations, shared by single forward passes and the graph of a proposal batch: a batch that
runs again after the activations moved to larger buffers, and a backward pass after a batch that ran again."""
import os

import numpy as np
import pytest
import scenegen.netgen as ng
from test_gpu_halfpass import amh, scene  # noqa: F401
from test_gpu_parity import make_ctx, say

from oracle import nn_oracle as nn

pytestmark = pytest.mark.gpu

WEIGHTS = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1805_07920_amd", "weights",
                       "proposal.bin")
JOBS = [dict(ref=0, srcs=[1, 2, 3, 4], iters=1), dict(ref=2, srcs=[1, 3], iters=1)]


def forward_inputs(n, h, w):
    import torch

    x = torch.from_numpy(ng.random_features(7, n, h, w)).cuda().to(torch.bfloat16)
    return x, torch.from_numpy(ng.random_q_ref(8, n, h, w)).cuda()


def test_batch_again_after_a_larger_forward(amh):  # noqa: F811
    say("case proposal batch, larger forward, the batch again")
    sc = scene(131, 77, 4)
    with make_ctx(amh, sc, refine=1, seed=3) as ctx:
        ctx.nn_load(WEIGHTS)
        ctx.run_batch_proposal(JOBS)
        first = [ctx.get_job_result(j) for j in range(2)]
        x, q = forward_inputs(1, 80, 88)  # 7040 cells, the batch's jobs have 960
        ctx.nn_forward(x, q)
        assert all(np.array_equal(a, b) for a, b in zip(first[0], ctx.get_job_result(0)))  # the results stay
        for _ in range(2):  # built anew, then its graph once more
            ctx.run_batch_proposal(JOBS)
            for j in range(2):
                for a, b in zip(first[j], ctx.get_job_result(j)):
                    assert np.array_equal(a, b)


def test_backward_after_a_batch_that_ran_again(amh):  # noqa: F811
    import torch

    say("case proposal batch again, then a backward pass")
    sc = scene(131, 77, 4)
    h, w = 24, 40  # the cells of 131 x 77
    t = torch.from_numpy(ng.random_targets(9, 1, h, w)).cuda()
    grads = []
    for small in (False, True):
        with make_ctx(amh, sc, refine=1, seed=3) as ctx:
            ctx.nn_set_params(ng.random_params(10, nn.LAYERS))
            ctx.run_batch_proposal(JOBS)
            if small:  # another pass is kept in between
                ctx.nn_forward(*forward_inputs(1, 8, 16))
                ctx.run_batch_proposal(JOBS)
            loss = ctx.nn_backward(t)
            grads.append((loss, ctx.nn_get_grads()))
    assert grads[0][0] == grads[1][0]
    assert np.array_equal(grads[0][1], grads[1][1])
