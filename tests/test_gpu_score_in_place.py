"""Fixed hypotheses in host memory whose costs go over the planes: every query is read before a cost is written, at each
call of a context and at any size, and the costs are those of separate buffers, bit for bit."""
import ctypes as C

import numpy as np
import pytest
from test_gpu_halfpass import amh, scene  # noqa: F401
from test_gpu_parity import make_ctx, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Q", [1, 2000, 70000])
@pytest.mark.parametrize("n", [2, 9])  # costs of a query shorter and longer than its plane
def test_costs_over_planes(amh, Q, n):  # noqa: F811
    say("case score in place", Q, n)
    sc = scene(131, 77, 9)
    rng = np.random.default_rng(Q + n)
    pix = np.stack([rng.integers(0, 131, Q), rng.integers(0, 77, Q)], 1).astype(np.int32)
    planes = np.concatenate([rng.normal(0, 0.2, (Q, 2)), -np.ones((Q, 1)), rng.uniform(3.0, 6.0, (Q, 1))], 1)
    planes = planes.astype(np.float32)
    with make_ctx(amh, sc) as ctx:
        ctx.begin(0, list(range(1, n + 1)))
        want = ctx.score_fixed(planes, pix)
        for _ in range(3):
            buf = np.zeros(Q * max(n, 4), np.float32)
            buf[:4 * Q] = planes.ravel()
            p = buf.ctypes.data_as(C.c_void_p)
            ctx._check(ctx.L.amh_score_fixed(ctx.h, p, pix.ctypes.data_as(C.c_void_p), Q, p, 0), "amh_score_fixed")
            assert np.array_equal(buf[:Q * n].view(np.uint32), want.ravel().view(np.uint32))
