"""The evaluation counters are the method's, whatever the half-pass shares or leaves out: refinement candidates on every
view that carries weight.  What was computed is counted by itself."""
import copy
import ctypes as C

import numpy as np
import pytest
from test_gpu_halfpass import amh, scene  # noqa: F401
from test_gpu_parity import make_ctx, say

pytestmark = pytest.mark.gpu


def colour_mask(w, h, colour):
    return (np.add.outer(np.arange(h), np.arange(w)) % 2) == colour


@pytest.mark.parametrize("w,h,n,t,dtype", [(131, 77, 3, 0, "f32"), (131, 77, 6, 3, "f32"), (203, 165, 6, 1, "f32"),
                                           (203, 165, 14, 3, "f16"), (203, 165, 32, 0, "f32")])
def test_refinement_is_counted_on_every_weighted_view(amh, w, h, n, t, dtype):  # noqa: F811
    """With k = 32 every view of S_t carries weight, and those of S_{t-1} that left it; all views where there is none."""
    say("case refinement counter", w, h, n, t, dtype)
    sc = scene(w, h, n, dtype)
    with make_ctx(amh, sc, refine=1, seed=6, k=32) as ctx:
        ctx.begin(0, list(range(1, n + 1)))
        ctx.init_hypotheses()
        for i in range(2):
            ctx.pass_(i, 0)
            ctx.pass_(i, 1)
        S0, s0, c0 = ctx.get_state()[2], ctx.get_stats(), ctx.get_scored_evals()
        ctx.pass_(t, 0)
        S1, s1, c1 = ctx.get_state()[2], ctx.get_stats(), ctx.get_scored_evals()
    act = (S0 | S1).astype(np.uint64)
    act[act == 0] = (1 << n) - 1
    views = np.array([bin(int(a)).count("1") for a in act[colour_mask(w, h, 0)]])
    assert s1["evals_refine"] - s0["evals_refine"] == (6 if t >= 3 else 3) * int(views.sum())
    counted = sum(s1[k] - s0[k] for k in ("evals_propagation", "evals_refine"))
    assert 0 < c1 - c0 < counted


@pytest.mark.parametrize("w,h", [(131, 77), (203, 165)])
def test_dropped_candidates_count_and_are_not_scored(amh, w, h):  # noqa: F811
    """The second source looks away, so that every evaluation on it is short, and carries weight by S_{t-1}: from true
    planes most candidates are out of the running after the first source, and count on the second all the same."""
    say("case dropped candidates", w, h)
    sc = scene(w, h, 2)
    cams = [copy.deepcopy(c) for c in sc.cams]
    cams[2].R = np.diag([-1.0, 1.0, -1.0])
    cams[2].t = np.zeros(3)
    rays = np.stack([*np.meshgrid(np.arange(w), np.arange(h)), np.ones((h, w))], -1) @ np.linalg.inv(cams[0].K).T
    nrm, d = sc.normal_gt.astype(np.float64), sc.depth_gt.astype(np.float64)
    planes = np.concatenate([nrm, -(d * (nrm * rays).sum(-1))[..., None]], -1).astype(np.float32)
    with amh.Context(refine=1, seed=6) as ctx:
        ctx.init_views([np.ascontiguousarray(i) for i in sc.images], cams)
        ctx.begin(0, [1, 2])
        ctx.set_state(planes, np.full((h, w), 0.5, np.float32), np.full((h, w), 3, np.uint32), np.zeros((h, w), np.int32))
        ctx.pass_(0, 0)
        st, scored = ctx.get_stats(), ctx.get_scored_evals()
    n_pix = int(colour_mask(w, h, 0).sum())
    counted = st["evals_propagation"] + st["evals_refine"]
    say(f"  short {st['evals_short']}, counted {counted}, scored {scored}")
    assert st["evals_refine"] == 2 * 3 * n_pix
    assert st["evals_propagation"] // 2 <= st["evals_short"] < counted
    assert scored < counted - n_pix  # at least a candidate a pixel was dropped


def test_one_plane_is_scored_once(amh):  # noqa: F811
    w, h, n = 131, 77, 6
    say("case scored evaluations, one plane")
    sc = scene(w, h, n)
    args = (np.tile(np.array([0.05, -0.1, -0.99, 4.1], np.float32), (h, w, 1)), np.full((h, w), 0.5, np.float32),
            np.full((h, w), 1, np.uint32), np.zeros((h, w), np.int32))
    with make_ctx(amh, sc, refine=0, seed=4) as ctx:
        ctx.begin(0, list(range(1, n + 1)))
        ctx.set_state(*args)
        ctx.pass_(1, 0)
        assert ctx.get_scored_evals() == n * int(colour_mask(w, h, 0).sum())
        assert ctx.L.amh_get_scored_evals(ctx.h, None) == amh.AMH_E_INVALID_ARG
    assert amh.lib().amh_get_scored_evals(None, C.byref(C.c_uint64())) == amh.AMH_E_INVALID_ARG


def test_ablation_build_scores_what_it_counts(amh):  # noqa: F811
    say("case scored evaluations, ablation build")
    with make_ctx(amh, scene(131, 77, 3), refine=1, seed=4, sym_prop=1) as ctx:
        ctx.run_checkerboard(0, [1, 2, 3], 1)
        st = ctx.get_stats()
        assert ctx.get_scored_evals() == st["evals_propagation"] + st["evals_refine"] > 0


def test_zero_before_the_first_reference(amh):  # noqa: F811
    say("case counters of a new context")
    with make_ctx(amh, scene(131, 77, 3), refine=1, seed=4) as ctx:
        ctx.run_checkerboard(0, [1, 2, 3], 1)  # leaves counts in memory that a new context may get
    with make_ctx(amh, scene(131, 77, 3)) as ctx:
        st = ctx.get_stats()
        assert all(st[k] == 0 for k in st if k.startswith("evals") or k == "fallback_pixels")
        assert ctx.get_scored_evals() == 0
