"""Performance cases of the library: the calls its users make, over the range of sizes, source counts, storage types
and options the configurations, tests and benchmark of this repository use.

`listed()` names the standing cases, `draw(rng)` gives further ones of the same ranges, `prepare` builds what a
program holds before the call, `run` is one pass through the public entry points, `work` the bytes and operations a
pass cannot do without and `exact` its result in 64 bits where there is one.
"""
from __future__ import annotations

import math
import os
from types import SimpleNamespace

import numpy as np
import torch

import paper_1805_07920_amd as amh

D_MIN, D_MAX = 2.0, 6.0
WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(amh.__file__)), "weights", "proposal.bin")
# (name, c_in, c_out, kernel side) of the proposal network's layers in parameter order
LAYERS = (("enc0a", 16, 16, 3), ("enc0b", 16, 16, 3), ("enc1a", 16, 32, 3), ("enc1b", 32, 32, 3),
          ("enc2a", 32, 48, 3), ("enc2b", 48, 48, 3), ("enc3a", 48, 64, 3), ("enc3b", 64, 64, 3),
          ("dec2", 112, 48, 3), ("dec1", 80, 32, 3), ("dec0", 48, 16, 3), ("head", 16, 5, 1))
LEVEL = {"enc0a": 0, "enc0b": 0, "enc1a": 1, "enc1b": 1, "enc2a": 2, "enc2b": 2, "enc3a": 3, "enc3b": 3,
         "dec2": 2, "dec1": 1, "dec0": 0, "head": 0}
# vector operations of one hypothesis x view evaluation: 36 warped, interpolated, weighted samples and the epilogue
OPS_PER_EVAL = 950
TOP_K = 4  # views that carry weight in a pixel's cost


# --------------------------------------------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------------------------------------------

def listed():
    return [
        # the tiny configuration: a thumbnail, where launches and the host path count
        dict(name="depth_128x96_n4", kind="depth", width=128, height=96, n_src=4, arc=15.0, iters=3, refine=0,
             f16=False, register=False),
        # the training recipe's size (labels of the proposal network are made with it); views already registered
        dict(name="depth_640x480_n8", kind="depth", width=640, height=480, n_src=8, arc=40.0, iters=3, refine=1,
             f16=False, register=False),
        # the benchmark's step: views registered from device images, depth map, outputs
        dict(name="depth_1920x1280_n10", kind="depth", width=1920, height=1280, n_src=10, arc=40.0, iters=3,
             refine=1, f16=False, register=True),
        # the high-resolution recipe: sources stored in float16, 20 of them, a third of the planes textureless
        dict(name="depth_3200x2130_n20_f16", kind="depth", width=3200, height=2130, n_src=20, arc=40.0, iters=4,
             refine=1, f16=True, register=False),
        # a depth map started from the learned proposal
        dict(name="proposal_1920x1280_n10", kind="proposal", width=1920, height=1280, n_src=10, arc=40.0, iters=1,
             refine=1, f16=False),
        # uneven reference images in one batched launch
        dict(name="batch_4jobs", kind="batch", jobs=4, width=1100, height=820, n_src=7, iters=3, refine=1, f16=False),
        # one more iteration from an earlier depth map (per-pixel hypotheses) at an odd size with few sources
        dict(name="resume_1001x667_n5", kind="resume", width=1001, height=667, n_src=5, arc=30.0, iters=1, refine=1,
             f16=False),
        # matching costs of a caller's own hypotheses (host arrays in and out)
        dict(name="score_20000_n10", kind="score", width=960, height=640, n_src=10, arc=40.0, queries=20000,
             f16=False),
        # the proposal network on a 1920x1280 reference's grid
        dict(name="net_forward_320x480", kind="net_forward", batch=1, h=320, w=480),
        # a training step of the proposal network at its recipe's batch: forward, loss and gradients, Adam
        dict(name="net_train_16x120x160", kind="net_train", batch=16, h=120, w=160),
        # the median filter of one depth map
        dict(name="median_1920x1280", kind="median", width=1920, height=1280),
        # the scene's depth maps fused into a point cloud
        dict(name="fuse_11x1920x1280", kind="fuse", width=1920, height=1280, n_src=10, arc=40.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["depth", "depth", "depth", "depth", "proposal", "batch", "resume", "score", "net_forward",
                       "net_train", "median", "fuse"])
    w = _log_int(rng, 96, 2400)  # odd and even
    h = max(64, int(w * rng.uniform(0.5, 0.85)))
    n = rng.randint(2, 16)
    arc = rng.choice([15.0, 30.0, 40.0])
    f16 = rng.random() < 0.3
    if kind == "depth":
        return dict(kind=kind, width=w, height=h, n_src=n, arc=arc, iters=rng.randint(1, 4),
                    refine=int(rng.random() < 0.85), f16=f16, register=rng.random() < 0.5)
    if kind == "proposal":
        return dict(kind=kind, width=w, height=h, n_src=n, arc=arc, iters=rng.randint(1, 2), refine=1, f16=f16)
    if kind == "batch":
        w = min(w, 1400)
        return dict(kind=kind, jobs=rng.randint(2, 6), width=w, height=max(64, int(0.7 * w)), n_src=min(n, 10),
                    iters=rng.randint(1, 3), refine=1, f16=f16)
    if kind == "resume":
        return dict(kind=kind, width=w, height=h, n_src=n, arc=arc, iters=rng.randint(1, 2), refine=1, f16=f16)
    if kind == "score":
        return dict(kind=kind, width=min(w, 1600), height=min(h, 1100), n_src=n, arc=arc,
                    queries=_log_int(rng, 100, 30000), f16=False)
    if kind == "net_forward":
        return dict(kind=kind, batch=rng.randint(1, 3), h=8 * _log_int(rng, 2, 60), w=8 * _log_int(rng, 2, 80))
    if kind == "net_train":
        return dict(kind=kind, batch=rng.randint(1, 16), h=8 * _log_int(rng, 3, 20), w=8 * _log_int(rng, 3, 25))
    if kind == "median":
        return dict(kind=kind, width=_log_int(rng, 96, 4000), height=_log_int(rng, 96, 3000))
    return dict(kind=kind, width=w, height=h, n_src=rng.randint(5, 12), arc=arc)


# --------------------------------------------------------------------------------------------------------------
# synthetic scenes: slanted textured rectangles before a textured background, rendered on the GPU
# --------------------------------------------------------------------------------------------------------------

def _cameras(width, height, n_src, arc):
    f = 100.0 * width / 128.0
    K = np.array([[f, 0.0, (width - 1) / 2.0], [0.0, f, (height - 1) / 2.0], [0.0, 0.0, 1.0]])
    # evenly spread over the arc, nearest to the reference first
    a = np.linspace(-arc / 2.0, arc / 2.0, n_src + 1)
    a = np.delete(a, int(np.argmin(np.abs(a))))
    a = np.deg2rad(a[np.argsort(np.abs(a), kind="stable")])
    cams = [SimpleNamespace(K=K, R=np.eye(3), t=np.zeros(3), width=width, height=height)]
    c = np.array([0.0, 0.0, 4.0])
    for th in a:
        pos = c + 4.0 * np.array([math.sin(th), 0.0, -math.cos(th)])
        z = (c - pos) / np.linalg.norm(c - pos)
        y = np.array([0.0, 1.0, 0.0])
        R = np.stack([np.cross(y, z), y, z])
        cams.append(SimpleNamespace(K=K, R=R, t=-R @ pos, width=width, height=height))
    return cams


def _scene(width, height, n_src, arc, seed, low_texture=False):
    """Cameras, images (float32 device tensors, [0, 255]), camera depths and normals per view; reference first."""
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    cams = _cameras(width, height, n_src, arc)
    Kinv = np.linalg.inv(cams[0].K)
    planes = []
    while len(planes) < 12:
        p0 = Kinv @ np.array([rng.uniform(0, width - 1), rng.uniform(0, height - 1), 1.0]) * rng.uniform(2.5, 5.5)
        tilt, az = math.radians(rng.uniform(0.0, 50.0)), rng.uniform(0.0, 2.0 * math.pi)
        nrm = np.array([math.sin(tilt) * math.cos(az), math.sin(tilt) * math.sin(az), -math.cos(tilt)])
        e1 = np.cross(nrm, np.array([0.0, 1.0, 0.0]) if abs(nrm[0]) > 0.5 else np.array([1.0, 0.0, 0.0]))
        e1 /= np.linalg.norm(e1)
        e2 = np.cross(nrm, e1)
        hu, hv = rng.uniform(0.5, 1.5, 2)
        zs = [(p0 + a * hu * e1 + b * hv * e2)[2] for a in (-1, 1) for b in (-1, 1)]
        if min(zs) < 2.2 or max(zs) > 5.8:
            continue
        planes.append((nrm, p0, e1, e2, hu, hv))
    planes.append((np.array([0.0, 0.0, -1.0]), np.array([0.0, 0.0, 5.9]), np.array([1.0, 0.0, 0.0]),
                   np.array([0.0, 1.0, 0.0]), 1e9, 1e9))
    table = torch.rand((1024, 1024), generator=gen, device="cuda") * 255.0
    shift = rng.integers(0, 1024, (len(planes), 2))
    const = [float(rng.uniform(50.0, 200.0)) if low_texture and k < 4 else -1.0 for k in range(len(planes))]
    spacing = 8.0 / cams[0].K[0, 0]  # two pixels at depth 4
    flat = table.reshape(-1)
    xs = torch.arange(width, device="cuda", dtype=torch.float32)[None, :]
    ys = torch.arange(height, device="cuda", dtype=torch.float32)[:, None]
    rx = (Kinv[0, 0] * xs + Kinv[0, 2]).expand(height, width)
    ry = (Kinv[1, 1] * ys + Kinv[1, 2]).expand(height, width)
    images, depths, normals = [], [], []
    for vi, cam in enumerate(cams):
        R, C = cam.R, -cam.R.T @ cam.t
        dw = [R[0, i] * rx + R[1, i] * ry + R[2, i] for i in range(3)]
        best = torch.full((height, width), float("inf"), device="cuda")
        img = torch.zeros((height, width), device="cuda")
        nrm = torch.zeros((height, width, 3), device="cuda")
        for k, (pn, p0, e1, e2, hu, hv) in enumerate(planes):
            s = float(pn @ (p0 - C)) / (pn[0] * dw[0] + pn[1] * dw[1] + pn[2] * dw[2])
            d = [float(C[i] - p0[i]) + s * dw[i] for i in range(3)]
            u = e1[0] * d[0] + e1[1] * d[1] + e1[2] * d[2]
            v = e2[0] * d[0] + e2[1] * d[1] + e2[2] * d[2]
            hit = (s > 1e-3) & (s < best) & (u.abs() <= hu) & (v.abs() <= hv)
            if const[k] >= 0.0:
                val = const[k] * (1.0 + 0.01 * (2.0 * torch.rand(s.shape, generator=gen, device="cuda") - 1.0))
            else:
                su, sv = (u / spacing).clamp(-1e6, 1e6), (v / spacing).clamp(-1e6, 1e6)
                iu, iv = torch.floor(su), torch.floor(sv)
                fu, fv = su - iu, sv - iv
                a = (iu.to(torch.int64) + int(shift[k, 0])) & 1023
                b = (iv.to(torch.int64) + int(shift[k, 1])) & 1023
                a1, b1 = (a + 1) & 1023, (b + 1) & 1023
                top = flat[b * 1024 + a] * (1 - fu) + flat[b * 1024 + a1] * fu
                bot = flat[b1 * 1024 + a] * (1 - fu) + flat[b1 * 1024 + a1] * fu
                val = top * (1 - fv) + bot * fv
            best = torch.where(hit, s, best)
            img = torch.where(hit, val, img)
            nc = R @ pn  # the planes face the reference: turn the normal towards this camera's ray
            away = (nc[0] * rx + nc[1] * ry + nc[2]) > 0
            for i in range(3):
                nrm[..., i] = torch.where(hit, torch.where(away, -float(nc[i]), float(nc[i])), nrm[..., i])
        gain = 1.0 if vi == 0 else float(rng.uniform(0.95, 1.05))
        images.append((img * gain).clamp(0.0, 255.0).contiguous())
        depths.append(best.contiguous())
        normals.append(nrm.contiguous())
    return cams, images, depths, normals


def _outputs(h, w):
    return (torch.empty((h, w), device="cuda"), torch.empty((h, w, 3), device="cuda"),
            torch.empty((h, w), device="cuda"))


def _features(case, seed):
    """Network inputs as the plane sweep writes them, and training targets."""
    n, h, w = case["batch"], case["h"], case["w"]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))

    def rnd(*s):
        return torch.rand(s, generator=gen, device="cuda")

    agg = rnd(n, h, w, 12)
    best, idx = agg.max(dim=3)
    pos = 2.0 * (idx.to(torch.float32) + rnd(n, h, w)) / 12.0 - 1.0
    feats = torch.cat([(rnd(n, h, w, 1) * 255.0 - 127.5) / 64.0, rnd(n, h, w, 1), pos[..., None], best[..., None],
                       agg], dim=3).to(torch.bfloat16).contiguous()
    q_far, q_near = 1.0 / D_MAX, 1.0 / D_MIN
    q_ref = (q_far + (pos + 1.0) / 2.0 * (q_near - q_far)).contiguous()
    nv = torch.randn((n, h, w, 3), generator=gen, device="cuda") * 0.3
    nv[..., 2] = -1.0
    conf = rnd(n, h, w, 1)
    depth = 1.0 / (q_ref + 0.01 * (rnd(n, h, w) - 0.5)).clamp(q_far, q_near)
    target = torch.cat([depth[..., None], nv / nv.norm(dim=3, keepdim=True), conf, conf], dim=3).contiguous()
    return feats, q_ref, target


def _queries(case, seed, depth, normal):
    """Hypotheses near the surface and away from it, at random pixels (host arrays, as the call takes them)."""
    q, w, h = case["queries"], case["width"], case["height"]
    rng = np.random.default_rng(seed + 17)
    pix = np.stack([rng.integers(0, w, q), rng.integers(0, h, q)], 1).astype(np.int32)
    d = depth.cpu().numpy()[pix[:, 1], pix[:, 0]].astype(np.float64)
    n = normal.cpu().numpy()[pix[:, 1], pix[:, 0]].astype(np.float64)
    n = n + 0.1 * rng.standard_normal((q, 3))
    n /= np.linalg.norm(n, axis=1, keepdims=True)
    d = np.where(rng.random(q) < 0.5, d * (1.0 + 0.01 * rng.standard_normal(q)), rng.uniform(D_MIN, D_MAX, q))
    K = _cameras(w, h, 1, case["arc"])[0].K
    ray = np.stack([(pix[:, 0] - K[0, 2]) / K[0, 0], (pix[:, 1] - K[1, 2]) / K[1, 1], np.ones(q)], 1)
    nr = (n * ray).sum(1)
    n = np.where((nr > 0)[:, None], -n, n)
    planes = np.concatenate([n, (d * np.abs(nr))[:, None]], 1).astype(np.float32)
    return planes, pix


def _store(case):
    return amh.AMH_F16 if case.get("f16") else amh.AMH_F32


def _stored(case, images):
    # float16 recipes hand the sources over in float16
    return [images[0]] + [im.to(torch.float16) for im in images[1:]] if case.get("f16") else images


# --------------------------------------------------------------------------------------------------------------
# what a program holds before the call
# --------------------------------------------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind, "case": case}
    if kind in ("net_forward", "net_train"):
        ctx = amh.Context(depth_min=D_MIN, depth_max=D_MAX)
        if kind == "net_forward":
            ctx.nn_load(WEIGHTS)
        else:
            ctx.nn_init(int(seed))
        feats, q_ref, target = _features(case, seed)
        out = torch.empty(q_ref.shape + (5,), device="cuda")
        return {**st, "ctx": ctx, "feats": feats, "q_ref": q_ref, "target": target, "out": out}
    if kind == "median":
        gen = torch.Generator(device="cuda").manual_seed(int(seed))
        h, w = case["height"], case["width"]
        y = torch.linspace(0, 9.0, h, device="cuda")[:, None]
        x = torch.linspace(0, 13.0, w, device="cuda")[None, :]
        src = 4.0 + torch.sin(x) * torch.cos(y) + 0.01 * torch.randn((h, w), generator=gen, device="cuda")
        spikes = torch.rand((h, w), generator=gen, device="cuda")
        src = torch.where(spikes < 0.05, 2.0 + 80.0 * spikes, src).contiguous()
        return {**st, "ctx": amh.Context(), "src": src, "dst": torch.empty_like(src)}
    if kind == "batch":
        rng = np.random.default_rng(case["jobs"])  # the uneven sizes belong to the case, the images to the seed
        images, cams, jobs, outs = [], [], [], []
        for j in range(case["jobs"]):
            s = 0.45 + 0.55 * (j + 1) / case["jobs"]
            w, h = 2 * int(case["width"] * s / 2), 2 * int(case["height"] * s / 2)
            n = max(2, case["n_src"] - 3 + int(rng.integers(0, 7)))
            cm, im, _, _ = _scene(w, h, n, 40.0, seed * 64 + j)
            jobs.append(dict(ref=len(images), srcs=list(range(len(images) + 1, len(images) + n + 1)),
                             iters=case["iters"]))
            images += _stored(case, im)
            cams += cm
            outs.append(_outputs(h, w))
        ctx = amh.Context(depth_min=D_MIN, depth_max=D_MAX, refine=case["refine"], seed=7)
        ctx.init_views(images, cams, _store(case))
        return {**st, "ctx": ctx, "jobs": jobs, "outs": outs}
    low = case["kind"] == "depth" and bool(case.get("f16"))
    cams, images, depths, normals = _scene(case["width"], case["height"], case["n_src"], case["arc"], seed, low)
    srcs = list(range(1, case["n_src"] + 1))
    if kind == "fuse":
        gen = torch.Generator(device="cuda").manual_seed(int(seed) + 5)
        maps = []
        for d in depths:
            bad = torch.rand(d.shape, generator=gen, device="cuda")
            d = d * (1.0 + 2e-4 * torch.randn(d.shape, generator=gen, device="cuda"))
            maps.append(torch.where(bad < 0.03, 2.0 + 130.0 * bad, d).contiguous())
        ctx = amh.Context()
        ctx.init_views(images, cams)
        return {**st, "ctx": ctx, "views": list(range(len(cams))), "depths": maps, "normals": normals}
    ctx = amh.Context(depth_min=D_MIN, depth_max=D_MAX, refine=case.get("refine", 1), seed=7)
    images = _stored(case, images)
    st.update(ctx=ctx, images=images, cams=cams, srcs=srcs, outs=_outputs(case["height"], case["width"]))
    ctx.init_views(images, cams, _store(case))
    if kind == "proposal":
        ctx.nn_load(WEIGHTS)
    elif kind == "resume":
        gen = torch.Generator(device="cuda").manual_seed(int(seed) + 5)
        noise = torch.randn(depths[0].shape, generator=gen, device="cuda")
        st["depth0"] = (depths[0] * (1.0 + 0.01 * noise)).contiguous()
        st["normal0"] = normals[0]
        st["conf0"] = torch.rand(depths[0].shape, generator=gen, device="cuda")
    elif kind == "score":
        ctx.begin(0, srcs)
        st["planes"], st["pix"] = _queries(case, seed, depths[0], normals[0])
    return st


# --------------------------------------------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------------------------------------------

def run(st):
    kind, case, ctx = st["kind"], st["case"], st["ctx"]
    if kind == "depth":
        if case["register"]:
            ctx.init_views(st["images"], st["cams"], _store(case))
        ctx.run_checkerboard(0, st["srcs"], case["iters"])
        return ctx.get_depth_normal_cost(*st["outs"])
    if kind == "proposal":
        ctx.run_proposal(0, st["srcs"], case["iters"])
        return ctx.get_depth_normal_cost(*st["outs"])
    if kind == "batch":
        ctx.run_batch(st["jobs"])
        return [ctx.get_job_result(j, *o) for j, o in enumerate(st["outs"])]
    if kind == "resume":
        ctx.begin(0, st["srcs"])
        ctx.set_initial_hypotheses(st["depth0"], st["normal0"], st["conf0"])
        for t in range(case["iters"]):
            ctx.pass_(t, 0)
            ctx.pass_(t, 1)
        return ctx.get_depth_normal_cost(*st["outs"])
    if kind == "score":
        return ctx.score_fixed(st["planes"], st["pix"])
    if kind == "net_forward":
        return ctx.nn_forward(st["feats"], st["q_ref"], st["out"])
    if kind == "net_train":
        # a step with its gradient read back, as a program that logs or clips it does
        out = ctx.nn_forward(st["feats"], st["q_ref"], st["out"])
        loss = ctx.nn_backward(st["target"])
        grads = ctx.nn_get_grads()
        ctx.nn_adam_step(1e-3)
        return {"out": out, "loss": loss, "grads": grads}
    if kind == "median":
        return ctx.median_filter4(st["src"], st["dst"])
    # into buffers for as many points as one view has pixels (a cloud of this many views holds more)
    cap = case["width"] * case["height"]
    pts, nrm, org, total = ctx.fuse(st["views"], st["depths"], st["normals"], capacity=cap)
    return {"points": pts, "normals": nrm, "origin": org, "total": total}


# --------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------------------------------------------

def _depth_work(w, h, n, iters, refine, f16, init=1.0):
    """Initial cost on every view; per pixel and iteration the 8 propagated planes on every view, the pixel's own on
    the views that carry weight, and refinement candidates on at least one view each."""
    p = float(w) * h
    k = min(TOP_K, n)
    evals = init * p * n + sum(p * (8 * n + k + (refine * (3 if t < 3 else 6))) for t in range(iters))
    return {"bytes": p * (4 + n * (2 if f16 else 4)) + 20.0 * p, "flops": OPS_PER_EVAL * evals}


def work(case):
    kind = case["kind"]
    if kind in ("net_forward", "net_train"):
        px = float(case["batch"]) * case["h"] * case["w"]
        flops = sum(2.0 * px / 4 ** LEVEL[n] * ci * co * k * k for n, ci, co, k in LAYERS)
        params = sum(ci * co * k * k + co for _, ci, co, k in LAYERS)
        if kind == "net_forward":
            return {"bytes": px * (32 + 4 + 20) + 2.0 * params, "flops": flops}
        # the gradients of the inputs and of the weights, each as much as the forward; Adam's state
        return {"bytes": px * (32 + 4 + 20 + 24) + 32.0 * params, "flops": 3.0 * flops}
    p = float(case["width"]) * case["height"]
    if kind == "median":
        return {"bytes": 8.0 * p, "flops": 63.0 * p}  # a sorting network of 16 takes 60 exchanges and more
    if kind == "fuse":
        n = case["n_src"] + 1
        # every view's depth and normals once, its mark, and the points (at most one per pixel of the reference)
        return {"bytes": n * p * 17 + 36.0 * p, "flops": 40.0 * p * n * (n - 1)}
    if kind == "score":
        q, n = float(case["queries"]), case["n_src"]
        return {"bytes": q * (24 + 4 * n) + min(p, 36 * q) * 4 * (n + 1), "flops": OPS_PER_EVAL * q * n}
    if kind == "batch":
        tot = {"bytes": 0.0, "flops": 0.0}
        rng = np.random.default_rng(case["jobs"])
        for j in range(case["jobs"]):
            s = 0.45 + 0.55 * (j + 1) / case["jobs"]
            n = max(2, case["n_src"] - 3 + int(rng.integers(0, 7)))
            one = _depth_work(2 * int(case["width"] * s / 2), 2 * int(case["height"] * s / 2), n, case["iters"],
                              case["refine"], case["f16"])
            tot = {k: tot[k] + one[k] for k in tot}
        return tot
    one = _depth_work(case["width"], case["height"], case["n_src"], case["iters"], case["refine"], case["f16"])
    if kind == "proposal":
        # the sweep: 12 m planes on the nearest sources at one pixel of each 4 x 4 cell
        m = max(1, (case["width"] + 80) // 160)
        one["flops"] += OPS_PER_EVAL * (p / 16.0) * 12 * m * min(4, case["n_src"])
        one["flops"] += sum(2.0 * p / 16.0 / 4 ** LEVEL[n] * ci * co * k * k for n, ci, co, k in LAYERS)
    return one


# --------------------------------------------------------------------------------------------------------------
# results in 64 bits
# --------------------------------------------------------------------------------------------------------------

def exact(case, seed):
    """Depth maps and point clouds follow thousands of discrete decisions per pixel and have no such value; the
    costs of given hypotheses, the network and the median do."""
    kind = case["kind"]
    if kind == "median":
        return _median64(prepare(case, seed)["src"])
    if kind == "score":
        return _score64(prepare(case, seed))
    if kind in ("net_forward", "net_train"):
        return _net64(case, seed)
    return None


def _median64(src):
    h, w = src.shape
    pad = torch.full((h + 3, w + 3), float("nan"), dtype=torch.float64, device=src.device)
    pad[1:h + 1, 1:w + 1] = src.double()
    win = torch.stack([pad[dy:dy + h, dx:dx + w] for dy in range(4) for dx in range(4)])
    win = torch.where(torch.isnan(win), torch.full_like(win, float("inf")), win).sort(dim=0).values
    n = torch.isfinite(win).sum(0)
    hi = win.gather(0, (n // 2)[None].clamp(max=15))[0]
    lo = win.gather(0, (n // 2 - 1)[None].clamp(min=0))[0]
    return torch.where(n % 2 == 1, hi, 0.5 * (lo + hi))


def _score64(st):
    """Bilaterally weighted NCC costs (36 samples over 11 x 11) of the hypotheses on every source."""
    cams, case = st["cams"], st["case"]
    w, h = case["width"], case["height"]
    planes = torch.tensor(st["planes"], dtype=torch.float64, device="cuda")
    px = torch.tensor(st["pix"], dtype=torch.int64, device="cuda")
    off = torch.tensor([(u, v) for v in range(-5, 6, 2) for u in range(-5, 6, 2)], device="cuda")
    K = torch.tensor(cams[0].K, dtype=torch.float64, device="cuda")
    Ki = torch.linalg.inv(K.cpu()).cuda()
    ref = st["images"][0].double()
    wx, wy = px[:, 0:1] + off[None, :, 0], px[:, 1:2] + off[None, :, 1]
    a = ref[wy.clamp(0, h - 1), wx.clamp(0, w - 1)]
    ac = ref[px[:, 1], px[:, 0]][:, None]
    wt = torch.exp(-(a - ac).abs() / 18.0 - off.double().norm(dim=1)[None] / 1800.0)
    wt = wt / wt.sum(1, keepdim=True)

    def inv_depth(x, y):  # of the plane along the ray of (x, y)
        rx, ry = Ki[0, 0] * x + Ki[0, 1] * y + Ki[0, 2], Ki[1, 1] * y + Ki[1, 2]
        return -(planes[:, 0:1] * rx + planes[:, 1:2] * ry + planes[:, 2:3]) / planes[:, 3:4]

    q0, qs = inv_depth(px[:, 0:1].double(), px[:, 1:2].double()), inv_depth(wx.double(), wy.double())
    base = (q0[:, 0] >= 1.0 / (D_MAX * (1 + 1e-5))) & (q0[:, 0] <= 1.0 / (D_MIN * (1 - 1e-5))) & (qs.min(1).values > 0)
    am = (wt * a).sum(1, keepdim=True)
    va = (wt * (a - am) ** 2).sum(1)
    out = []
    for cam, im in zip(cams[1:], st["images"][1:]):
        A = torch.tensor(cam.K @ cam.R @ np.linalg.inv(cams[0].K), dtype=torch.float64, device="cuda")
        b = torch.tensor(cam.K @ cam.t, dtype=torch.float64, device="cuda")

        def warp(x, y, q):
            return [A[i, 0] * x + A[i, 1] * y + A[i, 2] + b[i] * q for i in range(3)]

        X, Y, Z = warp(wx.double(), wy.double(), qs)
        cx, cy, cz = warp(px[:, 0:1].double(), px[:, 1:2].double(), q0)
        ok = base & (cz[:, 0] > 0) & (cx[:, 0] >= 0) & (cx[:, 0] <= (w - 1) * cz[:, 0]) & (cy[:, 0] >= 0)
        ok = ok & (cy[:, 0] <= (h - 1) * cz[:, 0]) & (Z.min(1).values > 1e-20)
        Zs = torch.where(ok[:, None], Z, torch.ones_like(Z))
        X, Y = X / Zs, Y / Zs
        x0, y0 = torch.floor(X).clamp(-1e6, 1e6), torch.floor(Y).clamp(-1e6, 1e6)
        fx, fy = X - x0, Y - y0
        x0, y0 = x0.to(torch.int64), y0.to(torch.int64)
        s = im.double()

        def at(xx, yy):
            return s[yy.clamp(0, h - 1), xx.clamp(0, w - 1)]

        v = ((at(x0, y0) * (1 - fx) + at(x0 + 1, y0) * fx) * (1 - fy)
             + (at(x0, y0 + 1) * (1 - fx) + at(x0 + 1, y0 + 1) * fx) * fy)
        vm = (wt * v).sum(1, keepdim=True)
        vb = (wt * (v - vm) ** 2).sum(1)
        cov = (wt * (a - am) * (v - vm)).sum(1)
        m = (1.0 - cov / torch.sqrt((va * vb).clamp(min=1e-300))).clamp(0.0, 2.0)
        out.append(torch.where(ok & (va >= 1e-5) & (vb >= 1e-5), m, torch.full_like(m, 2.0)))
    return torch.stack(out, 1).cpu().numpy()


def _conv64(x, wgt, bias):
    """x (n, h, w, c), wgt (co, k, k, ci): same-size convolution as one product over the taps."""
    n, h, w, _ = x.shape
    k = wgt.shape[1]
    r = k // 2
    xp = torch.nn.functional.pad(x, (0, 0, r, r, r, r))
    y = bias
    for ky in range(k):
        for kx in range(k):
            y = y + xp[:, ky:ky + h, kx:kx + w, :] @ wgt[:, ky, kx, :].T
    return y


def _net64(case, seed):
    st = prepare(case, seed)
    flat = torch.tensor(st["ctx"].nn_get_params().astype(np.float64), device="cuda")
    train = case["kind"] == "net_train"
    flat.requires_grad_(train)
    P, o = {}, 0
    for name, ci, co, k in LAYERS:
        wgt = flat[o:o + co * k * k * ci].reshape(co, k, k, ci)
        o += co * k * k * ci
        P[name] = (wgt, flat[o:o + co])
        o += co

    def c(name, x):
        return torch.relu(_conv64(x, *P[name]))

    def pool(x):
        return 0.25 * (x[:, ::2, ::2] + x[:, 1::2, ::2] + x[:, ::2, 1::2] + x[:, 1::2, 1::2])

    def up(x):
        return x.repeat_interleave(2, 1).repeat_interleave(2, 2)

    with torch.set_grad_enabled(train):
        e0 = c("enc0b", c("enc0a", st["feats"].double()))
        e1 = c("enc1b", c("enc1a", pool(e0)))
        e2 = c("enc2b", c("enc2a", pool(e1)))
        e3 = c("enc3b", c("enc3a", pool(e2)))
        d2 = c("dec2", torch.cat([up(e3), e2], 3))
        d1 = c("dec1", torch.cat([up(d2), e1], 3))
        d0 = c("dec0", torch.cat([up(d1), e0], 3))
        z = _conv64(d0, *P["head"])
        q_far, q_near = 1.0 / D_MAX, 1.0 / D_MIN
        q = (st["q_ref"].double() + (q_near - q_far) / 12.0 * torch.tanh(z[..., 0])).clamp(q_far, q_near)
        nh = z[..., 1:4] / z[..., 1:4].norm(dim=3, keepdim=True)
        out = torch.cat([(1.0 / q)[..., None], nh, torch.sigmoid(z[..., 4:5])], 3)
        if not train:
            return out
        t = st["target"].double()
        diff = (1.0 / q - t[..., 0]).abs() / (D_MAX - D_MIN)
        cosang = (nh * t[..., 1:4]).sum(3)
        loss = (t[..., 5] * (diff + 1.0 - cosang) + torch.nn.functional.softplus(z[..., 4]) - t[..., 4] * z[..., 4])
        loss = loss.mean()
        loss.backward()
    return {"out": out.detach(), "loss": float(loss), "grads": flat.grad.cpu().numpy()}
