"""Weight and bias gradients of every layer where a split of its pixels spans several staged blocks, the last of them
partial: the gradient of a batch is the mean of its images' gradients, which take one block each (a kernel that
test_gpu_nn and test_gpu_nn_tiles hold against the oracle).

For 2^k images of equal size it is so up to the order of the fp32 sums: the loss divides by the number of cells, 2^k times
an image's, so every stored gradient of the batch is the image's times 2^-k, rounded to the same bf16 mantissa.  A sum of m
terms of random sign carries a relative error of about 2^-24 sqrt(m), 6e-5 for the 1.1 M cells here; one step of 32
pixels left out of a split of 17 472 would show as sqrt(32 / 17472) = 4e-2.  The bar is 1e-3, per layer and part."""
import numpy as np
import pytest
import scenegen.netgen as ng
from test_gpu_halfpass import amh  # noqa: F401
from test_gpu_nn import dev, say

from oracle import nn_oracle as nn

pytestmark = pytest.mark.gpu

MAX_SPLITS, LEVEL = 64, dict(enc0=0, enc1=1, enc2=2, enc3=3, dec2=2, dec1=1, dec0=0, head=0)


def blocks(name, co, cells):
    """Staged blocks of a split of layer `name` over `cells` cells of level 0, and the pixels of its last one."""
    P = cells >> (2 * LEVEL[name[:4]])
    B = 1024 if name == "head" else 512 if co <= 32 else 256
    n = max(1, min(MAX_SPLITS, (P + 255) // 256))
    chunk = -(-(-(-P // n)) // 32) * 32
    return -(-chunk // B), chunk % B


@pytest.mark.parametrize("shape,levels", [((16, 120, 160), 3), ((64, 104, 168), 4)])
def test_batch_gradient_is_the_mean_of_its_images(amh, shape, levels):  # noqa: F811
    import torch

    say("case nn splits", shape)
    n, h, w = shape
    for name, _, co, _ in nn.LAYERS:
        assert blocks(name, co, h * w)[0] == 1  # an image: one block
        if LEVEL[name[:4]] < levels:
            many, last = blocks(name, co, n * h * w)
            assert many > 1 and last > 0, name
    x = dev(ng.random_features(1, n, h, w), torch.bfloat16)
    q = dev(ng.random_q_ref(2, n, h, w), torch.float32)
    t = dev(ng.random_targets(3, n, h, w), torch.float32)
    with amh.Context() as ctx:
        ctx.nn_set_params(ng.random_params(4, nn.LAYERS))
        ctx.nn_forward(x, q)
        loss, got = ctx.nn_backward(t), ctx.nn_get_grads().astype(np.float64)
        want, mean = np.zeros_like(got), 0.0
        for i in range(n):
            ctx.nn_forward(x[i:i + 1], q[i:i + 1])
            mean += ctx.nn_backward(t[i:i + 1]) / n
            want += ctx.nn_get_grads().astype(np.float64) / n
    assert loss == pytest.approx(mean, rel=1e-5)
    o = 0
    for name, ci, co, k in nn.LAYERS:
        for part, size in (("W", co * k * k * ci), ("b", co)):
            a, b = got[o:o + size], want[o:o + size]
            rel = np.linalg.norm(a - b) / np.linalg.norm(b)
            say(f"  {name}.{part}: {rel:.1e}")
            assert rel <= 1e-3, (name, part)
            o += size
