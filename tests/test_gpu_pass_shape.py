"""The tile shape and order of single references' half-passes: two-row tiles are taken where they are configured, at the
small sizes that take one-row tiles otherwise too, and the results do not depend on the shape."""
import ctypes as C

import numpy as np
import pytest
from test_gpu_halfpass import amh, scene  # noqa: F401
from test_gpu_parity import make_ctx, say

pytestmark = pytest.mark.gpu


# at most 256 4-row tiles of 16 columns take one row: 128 x 128 is the largest square of them
@pytest.mark.parametrize("w,h,n,rows", [(17, 9, 1, 1), (128, 128, 4, 1), (129, 128, 4, 4), (203, 165, 13, 3)])
def test_configured_rows(amh, w, h, n, rows):  # noqa: F811
    say("case pass shape", w, h, n)
    sc, got = scene(w, h, n), []
    with make_ctx(amh, sc, refine=1, seed=2) as ctx:
        with pytest.raises(amh.AmhError):
            ctx.get_pass_shape()  # no reference
        for config in (None, 0, 1, 4, 5):
            if config is not None:
                ctx.set_launch_config(config)
            ctx.run_checkerboard(0, list(range(1, n + 1)), 1)
            assert ctx.get_pass_shape() == dict(rows=2 if (config or 0) & 4 else rows, order=(config or 0) & 1)
            got.append(ctx.get_state())
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


def test_arguments(amh):  # noqa: F811
    rows, order = C.c_int(), C.c_int()
    assert amh.lib().amh_get_pass_shape(None, C.byref(rows), C.byref(order)) == amh.AMH_E_INVALID_ARG
    with make_ctx(amh, scene(17, 9, 1)) as ctx:
        ctx.begin(0, [1])
        assert ctx.L.amh_get_pass_shape(ctx.h, None, C.byref(order)) == amh.AMH_E_INVALID_ARG
        assert ctx.L.amh_get_pass_shape(ctx.h, C.byref(rows), None) == amh.AMH_E_INVALID_ARG
