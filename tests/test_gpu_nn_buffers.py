"""Buffers of the proposal network's forward pass: predictions written over the sweep's inverse depths, wherever those lie
in them, and features that start at any element -- bit for bit what separate, aligned buffers give, gradient included."""
import pytest
import scenegen.netgen as ng
from test_gpu_halfpass import amh  # noqa: F401
from test_gpu_nn import dev, say

from oracle import nn_oracle as nn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 8, 8), (2, 24, 40), (1, 320, 480)])
@pytest.mark.parametrize("over", ["start", "middle", "end", "beside"])
def test_predictions_over_the_inverse_depths(amh, shape, over):  # noqa: F811
    import torch

    say("case nn out over q_ref", shape, over)
    n, h, w = shape
    P = n * h * w
    x = dev(ng.random_features(1, n, h, w), torch.bfloat16)
    q = dev(ng.random_q_ref(2, n, h, w), torch.float32)
    t = dev(ng.random_targets(3, n, h, w), torch.float32)
    at = {"start": 0, "middle": 2 * P + 3, "end": 4 * P, "beside": 5 * P}[over]
    with amh.Context() as ctx:
        ctx.nn_set_params(ng.random_params(4, nn.LAYERS))
        want = ctx.nn_forward(x, q).clone()
        loss, grads = ctx.nn_backward(t), ctx.nn_get_grads()
        for _ in range(3):
            buf = torch.zeros(6 * P, device="cuda")
            buf[at:at + P] = q.ravel()
            got = ctx.nn_forward(x, buf[at:at + P].view(n, h, w), out=buf[:5 * P].view(n, h, w, 5))
            assert torch.equal(got, want)
            assert ctx.nn_backward(t) == loss and (ctx.nn_get_grads() == grads).all()


@pytest.mark.parametrize("offset", [1, 3, 7, 8])
def test_features_at_any_element(amh, offset):  # noqa: F811
    import torch

    say("case nn features at", offset)
    n, h, w = 2, 24, 40
    x = dev(ng.random_features(1, n, h, w), torch.bfloat16)
    q = dev(ng.random_q_ref(2, n, h, w), torch.float32)
    t = dev(ng.random_targets(3, n, h, w), torch.float32)
    buf = torch.zeros(x.numel() + 8, dtype=torch.bfloat16, device="cuda")
    y = buf[offset:offset + x.numel()].view(x.shape)
    y.copy_(x)
    assert (y.data_ptr() % 16 == 0) == (offset == 8)
    with amh.Context() as ctx:
        ctx.nn_set_params(ng.random_params(4, nn.LAYERS))
        want = ctx.nn_forward(x, q).clone()
        loss, grads = ctx.nn_backward(t), ctx.nn_get_grads()
        assert torch.equal(ctx.nn_forward(y, q), want)
        assert ctx.nn_backward(t) == loss and (ctx.nn_get_grads() == grads).all()
