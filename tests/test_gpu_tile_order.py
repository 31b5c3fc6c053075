"""A reference whose sources exceed the last-level cache (256 MB) takes hardware tile order by itself: the results are
those of the configured orders, bit for bit."""
import numpy as np
import pytest
import scenegen
from test_gpu_halfpass import amh  # noqa: F401
from test_gpu_parity import make_ctx, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [13, 14])  # 13 sources of 1920x1280: 255.6 MB, below 2^28 bytes; 14: above
def test_order_by_source_bytes(amh, n):  # noqa: F811
    say("case tile order", n)
    sc = scenegen.make_scene(1920, 1280, n, 30.0, 4, seed=n, src_dtype="f32", supersample=1)
    got = []
    for config in (None, 2, 3):
        with make_ctx(amh, sc, seed=4) as ctx:
            if config is not None:
                ctx.set_launch_config(config)
            ctx.run_checkerboard(0, list(range(1, n + 1)), 1)
            got.append(ctx.get_state())
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
