"""The half-pass at the edges of its work split: view counts around the rule that scores the own planes with the
propagated ones, tiles of 1, 2, 3 and 4 rows, hypotheses that are all the same plane (one evaluation serves every row)
or all different, six candidates, no own row -- against the CPU oracle (the bars of test_gpu_parity) and, across tile
shapes, bit for bit."""
import numpy as np
import pytest
import scenegen
from short_predicate import short_mask
from test_gpu_parity import _pass_parity, make_ctx, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amh():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1805_07920_amd as amh

    amh.lib()
    return amh


_scenes = {}


def scene(w, h, n, dtype="f32"):
    key = (w, h, n, dtype)
    if key not in _scenes:
        _scenes[key] = scenegen.make_scene(w, h, n, 30.0, 4, seed=w + n, src_dtype=dtype, supersample=2)
    return _scenes[key]


# below and above the size that takes one-row tiles (at most 256 4-row tiles of 16 columns)
@pytest.mark.parametrize("w,h,n,t,colour,refine,own", [
    (131, 77, 1, 1, 0, 1, 1), (131, 77, 2, 1, 1, 1, 0), (131, 77, 4, 3, 0, 1, 1), (131, 77, 5, 3, 1, 1, 1),
    (203, 165, 3, 1, 0, 1, 1), (203, 165, 4, 3, 1, 1, 0), (203, 165, 5, 1, 1, 1, 1), (203, 165, 9, 3, 0, 1, 1),
    (203, 165, 5, 1, 0, 0, 0), (203, 165, 13, 3, 1, 1, 1), (203, 163, 32, 1, 0, 1, 1),
])
def test_pass_matches_oracle(amh, oracle_mod, w, h, n, t, colour, refine, own):
    say("case half-pass", w, h, n, t, colour, refine, own)
    _pass_parity(amh, oracle_mod, scene(w, h, n), t, colour, seed=4, refine=refine, include_self=own)


@pytest.mark.parametrize("w,h,n", [(131, 77, 4), (203, 165, 6)])
@pytest.mark.parametrize("own", [0, 1])
def test_one_plane_everywhere(amh, oracle_mod, w, h, n, own):
    """Every row of every pixel, and its own, holds the same plane: costs, selection and counters as the oracle's."""
    say("case one plane", w, h, n, own)
    O, sc = oracle_mod, scene(w, h, n)
    pl = np.tile(np.array([0.05, -0.1, -0.99, 4.1], np.float32), (h, w, 1))
    cost = np.full((h, w), 0.5, np.float32)
    S, v = np.full((h, w), 1, np.uint32), np.zeros((h, w), np.int32)
    with make_ctx(amh, sc, refine=0, seed=4, include_self=own) as ctx:
        ctx.begin(0, list(range(1, n + 1)))
        ctx.set_state(pl, cost, S, v)
        ctx.pass_(1, 0)
        gpl, gc, gS, gv = ctx.get_state()
        st = ctx.get_stats()
    ost = O.State.from_arrays(pl, cost, S, v)
    order = np.array([i for i in range(w * h) if (i % w + i // w) % 2 == 0], np.int32)
    dg = O.run_pass(O.Views(sc.images, sc.cams), O.Params(refine=0, seed=4, include_self=own), ost, 1, 0, order=order,
                    diag=True)
    robust = np.array([(d.robust & 5) == 5 for d in dg])  # the views' tests and the top-k cut clear their margins
    flat = lambda a: np.asarray(a).reshape(w * h, -1)[order]
    assert np.array_equal(flat(gpl), flat(pl))
    assert robust.mean() > 0.9
    assert np.abs(flat(gc) - flat(ost.cost))[robust].max() <= 1e-4
    rows = int(sum(sum(d.row_valid[r] for r in range(9)) for d in dg))
    assert st["evals_propagation"] == rows * n
    per = np.array([sum(d.row_valid[r] for r in range(9)) for d in dg])
    xy = np.c_[order % w, order // w]
    short = short_mask(sc, xy, flat(pl), 2.0, 6.0).reshape(len(order), -1).sum(1)
    want = int((per * short).sum())
    assert abs(st["evals_short"] - want) <= 2 + 0.002 * want


def test_short_counter_with_the_own_planes_scored_last(amh, oracle_mod):
    """evals_short counts the own planes' evaluations on views without weight too (more views than kOwnFirst)."""
    w, h, n = 203, 165, 7
    say("case short counter", w, h, n)
    O, sc = oracle_mod, scene(w, h, n)
    with make_ctx(amh, sc, refine=0, seed=5) as ctx:
        ctx.begin(0, list(range(1, n + 1)))
        ctx.init_hypotheses()
        ctx.pass_(0, 0)
        ctx.pass_(0, 1)
        s0 = ctx.get_stats()
        pl, c, S, v = ctx.get_state()
        ctx.pass_(1, 0)
        s1 = ctx.get_stats()
    order = np.array([i for i in range(w * h) if (i % w + i // w) % 2 == 0], np.int32)
    dg = O.run_pass(O.Views(sc.images, sc.cams), O.Params(refine=0, seed=5), O.State.from_arrays(pl, c, S, v), 1, 0,
                    order=order, diag=True)
    dx, dy, _ = O.acp_offsets()
    fl, xy, rows = pl.reshape(-1, 4), [], []
    for q, d in zip(order, dg):
        for r in range(9):
            if d.row_valid[r]:
                ci = d.cand_index[r] if r < 8 else None
                xy.append((q % w, q // w))
                rows.append(fl[q if r == 8 else (q // w + dy[ci]) * w + q % w + dx[ci]])
    want = int(short_mask(sc, np.array(xy), np.array(rows), 2.0, 6.0).sum())
    assert s1["evals_propagation"] - s0["evals_propagation"] == len(rows) * n
    assert abs(s1["evals_short"] - s0["evals_short"] - want) <= 2 + 0.002 * want


@pytest.mark.parametrize("w,h,n,iters,own,dtype", [(17, 9, 1, 2, 1, "f32"), (48, 37, 3, 4, 0, "f32"),
                                                   (131, 77, 4, 4, 1, "f32"), (131, 77, 5, 4, 1, "f16"),
                                                   (131, 77, 12, 2, 1, "f32"), (131, 77, 13, 4, 1, "f32"),
                                                   (131, 77, 21, 2, 1, "f16")])
def test_tile_shapes_agree_bit_for_bit(amh, w, h, n, iters, own, dtype):
    """One-row tiles (a small single image) against the batch's 4-row (3-row from 13 views) and 2-row tiles."""
    say("case tile shapes", w, h, n, iters, own, dtype)
    sc = scene(w, h, n, dtype)
    srcs = list(range(1, n + 1))
    with make_ctx(amh, sc, refine=1, seed=9, include_self=own) as ctx:
        ctx.run_checkerboard(0, srcs, iters)
        want, ws = ctx.get_depth_normal_cost(), ctx.get_stats()
        for cfg in (0, 4):
            ctx.set_launch_config(cfg)
            ctx.run_batch([dict(ref=0, srcs=srcs, iters=iters)])
            got, gs = ctx.get_job_result(0), ctx.get_stats()
            for a, b in zip(want, got):
                assert np.array_equal(a, b), f"configuration {cfg}"
            for k in ("evals_propagation", "evals_refine", "evals_short"):
                assert ws[k] == gs[k], k
