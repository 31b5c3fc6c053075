"""The proposal network at the edges of its kernels' tiles: grids narrower than a tile, ragged in both directions, one
cell at the lowest level, splits of one partial block and of more than one block.  Forward and gradients against the
bf16-storage evaluation of the oracle (bars of test_gpu_nn; the gradient as one vector), and a batch against its
images one at a time, bit for bit."""
import numpy as np
import pytest
from test_gpu_nn import compare_predictions, dev, emulated, say

from oracle import nn_oracle as nn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amh():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1805_07920_amd as amh

    amh.lib()
    return amh


def inputs(shape):
    import scenegen.netgen as ng

    n, h, w = shape
    return (ng.random_params(50 + h, nn.LAYERS), ng.random_features(51 + w, n, h, w), ng.random_targets(52 + n, n, h, w),
            ng.random_q_ref(53, n, h, w))


# 34 816 cells: 64 splits of 544, a block of 512 and one of 32.  There only the loss and the gradient, which read every
# activation: compare_predictions bounds the largest angle over the cells, a bar for some hundreds of them.
@pytest.mark.parametrize("shape,cells", [((1, 8, 8), 1), ((3, 24, 40), 1), ((1, 136, 16), 1), ((1, 8, 152), 1),
                                         ((2, 128, 136), 0)])
def test_forward_and_gradient(amh, shape, cells):
    import torch

    say(f"case nn tiles {shape}")
    theta, x, t, q = inputs(shape)
    with amh.Context() as ctx:
        ctx.nn_set_params(theta)
        out = ctx.nn_forward(dev(x, torch.bfloat16), dev(q, torch.float32)).cpu().numpy().astype(np.float64)
        loss = ctx.nn_backward(dev(t, torch.float32))
        g = ctx.nn_get_grads().astype(np.float64)
    f64 = lambda a: a.astype(np.float64)
    z, Le, ge = emulated(f64(theta), f64(x), f64(q), f64(t))
    if cells:
        compare_predictions(out, z, f64(q), 1e-2, 1.0)
    rel = np.linalg.norm(g - ge) / np.linalg.norm(ge)
    say(f"  loss {loss:.6f} / {Le:.6f}, gradient {rel:.2e}")
    assert loss == pytest.approx(Le, rel=1e-4)
    assert rel <= 3e-2


@pytest.mark.parametrize("shape", [(3, 24, 40), (2, 16, 136)])
def test_batch_equals_its_images(amh, shape):
    import torch

    say(f"case nn batch {shape}")
    theta, x, _, q = inputs(shape)
    xd, qd = dev(x, torch.bfloat16), dev(q, torch.float32)
    with amh.Context() as ctx:
        ctx.nn_set_params(theta)
        both = ctx.nn_forward(xd, qd).clone()
        for i in range(shape[0]):
            one = ctx.nn_forward(xd[i:i + 1].contiguous(), qd[i:i + 1].contiguous())
            assert torch.equal(one[0], both[i])
