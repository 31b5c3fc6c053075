"""Fixed hypotheses from host memory are scored, from a context's second call on, in parts that fit its staging memory
(1 MiB halves, 24 + 4 n bytes a query): at the sizes around one, two and three parts the costs of the first, second and
third call are those of the device-memory call, bit for bit."""
import numpy as np
import pytest
from test_gpu_halfpass import amh, scene  # noqa: F401
from test_gpu_parity import make_ctx, say

pytestmark = pytest.mark.gpu

HALF = 1 << 20


@pytest.mark.parametrize("n", [1, 4])
@pytest.mark.parametrize("extra", [(0, 1), (1, 0), (1, 1), (2, 1), (3, -1), (3, 5)])
def test_host_parts_match_device_call(amh, n, extra):  # noqa: F811
    import torch

    most = HALF // (24 + 4 * n)
    Q = extra[0] * most + extra[1]
    say("case score parts", n, Q)
    sc = scene(131, 77, 4)
    rng = np.random.default_rng(Q)
    pix = np.stack([rng.integers(0, 131, Q), rng.integers(0, 77, Q)], 1).astype(np.int32)
    planes = np.concatenate([rng.normal(0, 0.2, (Q, 2)), -np.ones((Q, 1)), rng.uniform(3.0, 6.0, (Q, 1))], 1)
    planes = planes.astype(np.float32)
    with make_ctx(amh, sc) as ctx:
        ctx.begin(0, list(range(1, n + 1)))
        got = [ctx.score_fixed(planes, pix) for _ in range(3)]
        dp, dx = torch.from_numpy(planes).cuda(), torch.from_numpy(pix).cuda()
        out = torch.full((Q, n), -1.0, device="cuda")
        torch.cuda.synchronize()
        ctx._check(ctx.L.amh_score_fixed(ctx.h, dp.data_ptr(), dx.data_ptr(), Q, out.data_ptr(), 1), "amh_score_fixed")
        torch.cuda.synchronize()
        want = out.cpu().numpy()
    assert (want >= 0).all()
    for g in got:
        assert np.array_equal(g.view(np.uint32), want.view(np.uint32))
