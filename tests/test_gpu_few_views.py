"""Few source views: a workgroup scores the refinement candidates' pairs on all views together where they are few, and
otherwise drops candidates by their most important view first.  Which it does follows from the tile shape, the number of
views and the iteration; results and counters do not."""
import numpy as np
import pytest

import scenegen
from test_gpu_halfpass import amh  # noqa: F401
from test_gpu_parity import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("size", [(1, 1), (17, 9), (131, 77), (201, 165)])  # one-row tiles, the last four-row
def test_same_results_in_every_tile_shape(size, n, dtype, amh):  # noqa: F811
    w, h = size
    sc = scenegen.make_scene(w, h, n, 35.0, 6, seed=w + n, src_dtype=dtype, supersample=1)
    srcs = list(range(1, n + 1))
    got = {}
    for k in (1, 4):
        with amh.Context(seed=7, refine=1, k=k) as ctx:
            ctx.init_views([np.ascontiguousarray(i) for i in sc.images], sc.cams,
                           store_as=amh.AMH_F16 if dtype == "f16" else amh.AMH_F32)
            for cfg in (0, 4):  # by default; two-row tiles
                ctx.set_launch_config(cfg)
                ctx.run_checkerboard(0, srcs, 5)  # from the fourth iteration on 6 candidates, 3 before
                st = {a: b for a, b in ctx.get_stats().items() if a.startswith("evals")}
                got[cfg] = ctx.get_state(), st
                say(f"{w}x{h}, {n} views {dtype}, k {k}, tiles {ctx.get_pass_shape()}: {st}")
        for a, b in zip(got[0][0], got[4][0]):
            assert np.array_equal(a, b, equal_nan=True)
        assert got[0][1] == got[4][1]
