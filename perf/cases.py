"""The work that programs built on this library have it do, as cases that can be timed and compared.

A pass starts where a training or inference step starts: raw voxel coordinates of a new batch are in device memory,
features and weights too.  Every batch holds new clouds, so hashing the coordinates and building the kernel maps are
part of every pass, as they are of every step in use.

Kinds of pass
  layer   coordinates + kernel map + one sparse convolution: forward, data gradient, weight gradient
  updown  coordinates + k2s2 map + downsampling convolution and its transposed counterpart; training or inference
  stack   one training step of the 8-convolution classifier (5 maps, BN+ReLU, pooling, linear, loss, all gradients)
  pool    coordinates + map + max pooling, forward and backward

Clouds are drawn on the GPU: points on surfaces in sampling order, quantised to voxels, duplicates left in.
  sphere  points uniform on a sphere of radius 0.9 in [-1, 1]^3
  shapes  points on 1-4 boxes, spheres and cylinders in the unit cube (scale `lo`..`hi`); a fraction U[0, 1-keep] dropped
  room    a 10 x 10 x 3 m room with 30 boxes of furniture, five points per voxel face, 1 cm of jitter
"""
from __future__ import annotations

import math
import zlib

import numpy as np
import torch

from paper_2012_13846_amd import binding as sp

STACK_CHANNELS = [32, 32, 64, 64, 128, 128, 256, 256, 256]
STACK_STRIDES = [1, 1, 1, 2, 1, 2, 1, 1]
STACK_CLASSES = 40
_SOURCE_KEYS = ("source", "clouds", "points", "grid", "lo", "hi", "keep", "voxel")


# ---- clouds ----------------------------------------------------------------------------------------------------
def _quantize(p, origin, voxel, batch):
    v = torch.floor((p - origin) / voxel).to(torch.int32)
    return torch.cat([batch.to(torch.int32)[:, None], v], dim=1)


def _unit(n, g):
    v = torch.randn((n, 3), device="cuda", generator=g)
    return v / v.norm(dim=1, keepdim=True).clamp_min(1e-12)


def _sphere(case, g):
    n, grid = case["clouds"] * case["points"], case["grid"]
    batch = torch.arange(n, device="cuda") // case["points"]
    raw = _quantize(0.9 * _unit(n, g), -1.0, 2.0 / grid, batch)
    raw[:, 1:].clamp_(0, grid - 1)
    return raw


def _rotation(rng):
    w, x, y, z = (lambda q: q / np.linalg.norm(q))(rng.standard_normal(4))
    return np.array([[1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w)],
                     [2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w)],
                     [2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)]])


def _shapes(case, g, rng):
    clouds, points, grid = case["clouds"], case["points"], case["grid"]
    kind, par = np.zeros((clouds, 4), np.int64), np.zeros((clouds, 4, 3))
    rot, centre, area = np.zeros((clouds, 4, 3, 3)), np.zeros((clouds, 4, 3)), np.zeros((clouds, 4))
    for c in range(clouds):
        for j in range(int(rng.integers(1, 5))):
            kind[c, j], scale = rng.integers(0, 3), rng.uniform(case["lo"], case["hi"])
            if kind[c, j] == 0:                                             # box: half extents
                p = 0.5 * scale * rng.uniform(0.5, 1.0, 3)
                area[c, j], reach = 8 * (p[0] * p[1] + p[1] * p[2] + p[0] * p[2]), np.linalg.norm(p)
            elif kind[c, j] == 1:                                           # sphere: radius
                p = np.full(3, 0.5 * scale)
                area[c, j], reach = 4 * np.pi * p[0] ** 2, p[0]
            else:                                                           # cylinder: radius, half height
                p = 0.5 * scale * np.array([rng.uniform(0.3, 1.0), rng.uniform(0.5, 1.0), 0.0])
                area[c, j], reach = 4 * np.pi * p[0] * p[1] + 2 * np.pi * p[0] ** 2, np.hypot(p[0], p[1])
            m = min(reach * 0.8, 0.5)
            par[c, j], rot[c, j], centre[c, j] = p, _rotation(rng), rng.uniform(m, 1 - m, 3) if m < 0.5 else 0.5
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    n = clouds * points
    batch = torch.arange(n, device="cuda") // points
    u = torch.rand((n, 6), device="cuda", generator=g)
    cum = dev(np.cumsum(area, axis=1) / area.sum(axis=1, keepdims=True)).float()
    which = (u[:, :1] > cum[batch][:, :3]).sum(dim=1)
    at = batch * 4 + which
    pr, kd = dev(par).float().reshape(-1, 3)[at], dev(kind).reshape(-1)[at]
    # box: a face by area, a point on it
    ar = torch.stack([pr[:, 1] * pr[:, 2], pr[:, 0] * pr[:, 2], pr[:, 0] * pr[:, 1]], dim=1)
    axis = (u[:, 1:2] > (torch.cumsum(ar, 1) / ar.sum(1, keepdim=True).clamp_min(1e-20))[:, :2]).sum(dim=1)
    box = (2 * u[:, 2:5] - 1) * pr
    sign = torch.where(u[:, 5] < 0.5, -1.0, 1.0)
    box.scatter_(1, axis[:, None], (sign * pr.gather(1, axis[:, None])[:, 0])[:, None])
    ball = _unit(n, g) * pr[:, :1]
    side = 2 * pr[:, 1] / (2 * pr[:, 1] + pr[:, 0]).clamp_min(1e-20)         # share of the mantle
    phi, cap = 2 * math.pi * u[:, 2], u[:, 1] > side
    r = torch.where(cap, pr[:, 0] * u[:, 3].sqrt(), pr[:, 0])
    z = torch.where(cap, sign * pr[:, 1], (2 * u[:, 4] - 1) * pr[:, 1])
    cyl = torch.stack([r * phi.cos(), r * phi.sin(), z], dim=1)
    loc = torch.where((kd == 0)[:, None], box, torch.where((kd == 1)[:, None], ball, cyl))
    pts = (dev(rot).float().reshape(-1, 3, 3)[at] * loc[:, None, :]).sum(dim=2) + dev(centre).float().reshape(-1, 3)[at]
    inside = ((pts >= 0) & (pts < 1)).all(dim=1)
    kept = dev(np.ceil(points * (1 - rng.uniform(0, 1 - case["keep"], clouds)))) if case["keep"] < 1 else None
    if kept is not None:
        inside &= (torch.arange(n, device="cuda") % points) < kept[batch]
    raw = _quantize(pts, 0.0, 1.0 / grid, batch)[inside]
    raw[:, 1:].clamp_(0, grid - 1)
    return raw


def _room(case, g, rng):
    voxel, (X, Y, Z) = case["voxel"], (10.0, 10.0, 3.0)
    rects = [((0, 0, 0), (X, 0, 0), (0, Y, 0)), ((0, 0, Z), (X, 0, 0), (0, Y, 0)), ((0, 0, 0), (X, 0, 0), (0, 0, Z)),
             ((0, Y, 0), (X, 0, 0), (0, 0, Z)), ((0, 0, 0), (0, Y, 0), (0, 0, Z)), ((X, 0, 0), (0, Y, 0), (0, 0, Z))]
    for _ in range(30):
        e = rng.uniform(0.3, 2.0, 3)
        o = np.array([rng.uniform(0.05, X - e[0] - 0.05), rng.uniform(0.05, Y - e[1] - 0.05), 0.0])
        ex, ey, ez = np.diag(e)
        rects += [(o + ez, ex, ey), (o, ex, ez), (o + ey, ex, ez), (o, ey, ez), (o + ex, ey, ez)]
    O, U, V = (torch.tensor(np.array([r[i] for r in rects], np.float32), device="cuda") for i in range(3))
    area = torch.linalg.cross(U, V).norm(dim=1)
    n = int(5.0 * float(area.sum()) / voxel ** 2)
    u = torch.rand((n, 6), device="cuda", generator=g)
    which = torch.searchsorted(torch.cumsum(area, 0) / area.sum(), u[:, 0].contiguous()).clamp_max(len(rects) - 1)
    p = O[which] + u[:, 1:2] * U[which] + u[:, 2:3] * V[which] + 0.02 * u[:, 3:6] - 0.01
    p = torch.minimum(p.clamp_min(0), torch.tensor([X, Y, Z], device="cuda") - 1e-5)
    return _quantize(p, 0.0, voxel, torch.zeros(n, device="cuda"))


def _raw(case, seed):
    """The case's clouds, as batch number `seed` of an epoch that shows them again: clouds in another order, each turned
    and mirrored along the axes, its points in another order (the number of voxels stays the same)."""
    base = zlib.crc32(repr(sorted((k, v) for k, v in case.items() if k in _SOURCE_KEYS)).encode())
    g, rng = torch.Generator(device="cuda").manual_seed(base), np.random.default_rng(base)
    make = {"sphere": lambda: _sphere(case, g), "shapes": lambda: _shapes(case, g, rng), "room": lambda: _room(case, g, rng)}
    raw = make[case["source"]]()
    g, rng = torch.Generator(device="cuda").manual_seed(seed), np.random.default_rng(seed)
    clouds = case.get("clouds", 1)
    order = torch.from_numpy(rng.permutation(clouds)).cuda()
    turn = torch.from_numpy(np.array([rng.permutation(3) for _ in range(clouds)])).cuda()
    flip = torch.from_numpy(rng.integers(0, 2, (clouds, 3)).astype(np.int32)).cuda()
    b = raw[:, 0].long()
    xyz = raw[:, 1:].gather(1, turn[b])
    top = 8 * int(xyz.max() // 8) + 7              # mirrored cells of a coarser level are cells again
    xyz = torch.where(flip[b] == 1, top - xyz, xyz)
    raw = torch.cat([order[b].to(torch.int32)[:, None], xyz], dim=1)
    mixed = torch.randperm(len(raw), device="cuda", generator=g)
    at = mixed[torch.argsort(raw[mixed, 0], stable=True)]
    return raw[at].contiguous(), g


# ---- the cases -------------------------------------------------------------------------------------------------
def _shape_batch(clouds, points, grid, lo=0.2, hi=0.8, keep=1.0):
    return {"source": "shapes", "clouds": clouds, "points": points, "grid": grid, "lo": lo, "hi": hi, "keep": keep}


def _spheres(clouds, points, grid):
    return {"source": "sphere", "clouds": clouds, "points": points, "grid": grid}


def _layer(src, cin, cout, dtype, kernel=3, stride=1, dilation=1):
    return {"kind": "layer", **src, "kernel": kernel, "stride": stride, "dilation": dilation, "cin": cin, "cout": cout,
            "dtype": dtype}


def _updown(src, c, dtype, train):
    return {"kind": "updown", **src, "kernel": 2, "stride": 2, "dilation": 1, "cin": c, "cout": 2 * c, "dtype": dtype,
            "train": train}


def listed():
    sweep = dict(lo=0.6, hi=1.0)
    return [
        # a single object at the coarsest grid: the smallest step there is, all latency
        {"name": "one_shape_c16_f32", **_layer(_spheres(1, 2048, 32), 16, 16, "f32")},
        # first layer of a network on a batch of scans: three input channels (a colour or a normal per point)
        {"name": "input_c3x32_f32", **_layer(_shape_batch(8, 20000, 128), 3, 32, "f32")},
        # the benchmark's layer: a batch of 8 objects at a fine grid
        {"name": "batch8_c32x64_f32", **_layer(_shape_batch(8, 20000, 128), 32, 64, "f32")},
        # the published training batch: 256 objects of 4096 points at 32^3
        {"name": "sweep32_b256_c64_f32", **_layer(_shape_batch(256, 4096, 32, **sweep), 64, 64, "f32")},
        # a wide fp32 layer of the same classifier, half of the points dropped out, 50^3
        {"name": "sweep50_c128_f32", **_layer(_shape_batch(64, 4096, 50, keep=0.5, **sweep), 128, 128, "f32")},
        # a width that is no power of two
        {"name": "batch8_c48_f32", **_layer(_shape_batch(8, 20000, 128), 48, 48, "f32")},
        # encoder/decoder pair, inference on small sparse clouds: latency
        {"name": "updown_small_infer_bf16", **_updown(_spheres(8, 2048, 256), 64, "bf16", False)},
        # the same pair in training on full clouds
        {"name": "updown_c64x128_bf16", **_updown(_spheres(8, 131072, 256), 64, "bf16", True)},
        # a bf16 layer on a micro-batch of four fine clouds
        {"name": "batch4_c64_bf16", **_layer(_spheres(4, 131072, 256), 64, 64, "bf16")},
        # one indoor scene of about a million voxels
        {"name": "room_c64_bf16", **_layer({"source": "room", "voxel": 0.025}, 64, 64, "bf16")},
        # a whole training step of the classifier: wide layers, strided maps, all the layers between
        {"name": "stack_b4_bf16", "kind": "stack", **_spheres(4, 131072, 256), "dtype": "bf16"},
        # pooling between two blocks
        {"name": "pool_c64_bf16", "kind": "pool", **_spheres(4, 131072, 256), "kernel": 2, "stride": 2, "channels": 64,
         "dtype": "bf16"},
    ]


def draw(rng):
    def span(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def source(most):
        """A batch of at most `most` points."""
        pick = rng.choice(["sphere", "shapes", "shapes", "room"])
        if pick == "room":  # about 2900 points at a voxel of 1 m; grows with 1 / voxel^2
            lo = max(0.025, math.sqrt(3000.0 / most))
            return {"source": "room", "voxel": round(math.exp(rng.uniform(math.log(lo), math.log(max(0.1, lo * 2)))), 4)}
        n = span(2000, min(most, 1_000_000))
        if pick == "sphere":
            clouds = rng.randint(1, 8)
            return _spheres(clouds, max(500, n // clouds), rng.choice([32, 64, 100, 128, 256]))
        clouds = min(span(1, 256), max(1, n // 1000))
        return _shape_batch(clouds, max(500, n // clouds), rng.choice([32, 50, 64, 128]), *rng.choice([(0.2, 0.8), (0.6, 1.0)]),
                            keep=rng.choice([1.0, 0.5, 0.25]))

    kind = rng.choice(["layer"] * 5 + ["updown", "stack", "pool"])
    if kind == "layer":
        dtype = rng.choice(["f32", "bf16"])
        group = rng.choice(["input", "even", "even", "even", "odd"])
        if group == "input":
            cin, cout, most = rng.randint(3, 6), rng.choice([16, 32, 64]), 160_000
        elif group == "even":
            cin, cout = rng.choice([(16, 16), (32, 32), (32, 64), (64, 64), (64, 128), (128, 128)])
            most = 4_000_000 if (dtype == "bf16" and cin == 64) else 1_000_000 * 4096 // max(4096, cin * cout)
        else:
            cin, cout, most = rng.choice([20, 24, 48, 80]), rng.choice([24, 40, 48]), 100_000
        kernel, stride, dilation = rng.choice([(3, 1, 1), (3, 1, 1), (3, 1, 1), (3, 1, 2), (3, 2, 1)])
        return _layer(source(most), cin, cout, dtype, kernel, stride, dilation)
    if kind == "updown":
        return _updown(source(1_000_000), rng.choice([32, 64]), rng.choice(["f32", "bf16", "bf16"]), rng.choice([True, False]))
    if kind == "stack":
        clouds = rng.randint(1, 8)
        return {"kind": "stack", **_spheres(clouds, span(2000, 500_000 // clouds), rng.choice([64, 128, 256])), "dtype": "bf16"}
    kernel = rng.choice([2, 3])
    return {"kind": "pool", **source(1_000_000), "kernel": kernel, "stride": 2, "channels": rng.choice([5, 32, 64, 128]),
            "dtype": rng.choice(["f32", "bf16"])}


# ---- a pass ----------------------------------------------------------------------------------------------------
def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def prepare(case, seed):
    """What a program holds when a step begins: the batch's raw coordinates, the rows' features and the gradients that
    arrive from the layers behind (both in the row order that the library numbers the voxels in), weights."""
    raw, g = _raw(case, seed)
    dt = _dtype(case)

    def rows(n, c):
        return torch.randn((n, c), device="cuda", generator=g).to(dt)

    def weights(kvol, co, ci):
        return (torch.randn((kvol, co, ci), device="cuda", generator=g) / math.sqrt(kvol * ci)).to(dt)

    s = {"case": case, "raw": raw}
    c = sp.sp_coords_build(raw, 1)
    if case["kind"] == "stack":
        ch = STACK_CHANNELS
        s["clouds"] = case["clouds"]
        s["x"] = rows(c.n, ch[0])
        s["w"] = [weights(27, ch[i + 1], ch[i]) for i in range(8)]
        s["gamma"] = [1 + 0.1 * torch.randn(n, device="cuda", generator=g) for n in ch[1:]]
        s["beta"] = [0.1 * torch.randn(n, device="cuda", generator=g) for n in ch[1:]]
        s["w_fc"] = torch.randn((STACK_CLASSES, ch[8]), device="cuda", generator=g) / 16
        s["b_fc"] = torch.zeros(STACK_CLASSES, device="cuda")
        s["labels"] = torch.randint(0, STACK_CLASSES, (case["clouds"],), device="cuda", generator=g).to(torch.int32)
        c.close()
        return s
    km, co = sp.sp_kmap_build(c, case["kernel"], case["stride"], case.get("dilation", 1))
    n_in, n_out = km.n_in, km.n_out
    for h in (km, co, c):
        h.close()
    if case["kind"] == "pool":
        s["x"], s["dy"] = rows(n_in, case["channels"]), rows(n_out, case["channels"])
        return s
    kvol, cin, cout = case["kernel"] ** 3, case["cin"], case["cout"]
    s["x"], s["w"], s["dy"] = rows(n_in, cin), weights(kvol, cout, cin), rows(n_out, cout)
    if case["kind"] == "updown":
        s["w_up"], s["dz"] = weights(kvol, cin, cout), rows(n_in, cin)
    return s


def _run_stack(s):
    c0 = sp.sp_coords_build(s["raw"], 1)
    maps, by_key, cur, level, handles = [], {}, c0, 0, [c0]
    for st in STACK_STRIDES:                       # layers of one level with one stride share their map
        if (level, st) not in by_key:
            by_key[(level, st)] = sp.sp_kmap_build(cur, 3, st, 1)
            handles += by_key[(level, st)]
        km, co = by_key[(level, st)]
        maps.append(km)
        if st > 1:
            cur, level = co, level + 1
    x, saved, out = s["x"], [], {}
    for i in range(8):
        z = sp.sp_conv_fwd(maps[i], x, s["w"][i])
        y, mean, rstd = sp.sp_bn_relu_fwd(z, s["gamma"][i], s["beta"][i])
        saved.append((x, z, y, mean, rstd))
        x = y
    last = cur.coords()
    pooled, counts = sp.sp_pool_avg_fwd(last, x, s["clouds"])
    out["logits"] = sp.sp_linear_fwd(pooled, s["w_fc"], s["b_fc"])
    out["loss"], dlogits = sp.sp_softmax_ce(out["logits"], s["labels"])
    dpooled, out["dw_fc"], out["db_fc"] = sp.sp_linear_bwd(pooled, s["w_fc"], dlogits)
    g = sp.sp_pool_avg_bwd(last, dpooled, counts, x.shape[0], torch.bfloat16)
    for i in reversed(range(8)):
        xin, z, y, mean, rstd = saved[i]
        dz, out["dgamma%d" % i], out["dbeta%d" % i] = sp.sp_bn_relu_bwd(z, y, g, s["gamma"][i], mean, rstd)
        out["dw%d" % i] = sp.sp_conv_bwd_weight(maps[i], xin, dz)
        g = sp.sp_conv_bwd_data(maps[i], dz, s["w"][i])
    out["dx"] = g
    for h in handles:
        h.close()
    return out


def run(s):
    case = s["case"]
    if case["kind"] == "stack":
        return _run_stack(s)
    c = sp.sp_coords_build(s["raw"], 1)
    km, co = sp.sp_kmap_build(c, case["kernel"], case["stride"], case.get("dilation", 1))
    out = {}
    if case["kind"] == "pool":
        out["y"], arg = sp.sp_pool_fwd(km, s["x"], "max")
        out["arg"] = arg
        out["dx"] = sp.sp_pool_bwd(km, s["dy"], arg, "max")
    else:
        out["y"] = sp.sp_conv_fwd(km, s["x"], s["w"])
        train = case["kind"] == "layer" or case["train"]
        if case["kind"] == "updown":
            kt = sp.sp_kmap_transpose(km)
            out["z"] = sp.sp_conv_fwd(kt, out["y"], s["w_up"])
            dy = s["dy"]
            if train:
                out["dw_up"] = sp.sp_conv_bwd_weight(kt, out["y"], s["dz"])
                dy = out["dy"] = sp.sp_conv_bwd_data(kt, s["dz"], s["w_up"])
            kt.close()
        else:
            dy = s["dy"]
        if train:
            out["dw"] = sp.sp_conv_bwd_weight(km, s["x"], dy)
            out["dx"] = sp.sp_conv_bwd_data(km, dy, s["w"])
    out["pairs"] = km.total
    for h in (km, co, c):
        h.close()
    return out


# ---- what a pass cannot do without -----------------------------------------------------------------------------
def work(case):
    """Coordinates, features, weights and gradients once each; two operations per link, channel pair and direction."""
    raw, _ = _raw(case, 1)
    c = sp.sp_coords_build(raw, 1)
    elt = 2 if case["dtype"] == "bf16" else 4
    byts = 16.0 * raw.shape[0]
    if case["kind"] == "stack":
        flops, cur, handles = 0.0, c, [c]
        byts += 2.0 * c.n * STACK_CHANNELS[0] * elt
        for i, st in enumerate(STACK_STRIDES):
            km, co = sp.sp_kmap_build(cur, 3, st, 1)
            ci, cn = STACK_CHANNELS[i], STACK_CHANNELS[i + 1]
            # forward keeps z and y of every layer for the backward pass
            byts += 27.0 * ci * cn * (2 * elt + 4) + 4.0 * km.n_out * cn * elt
            flops += 6.0 * km.total * ci * cn
            handles += [km, co]
            cur = co
        for h in handles:
            h.close()
        return {"bytes": byts, "flops": flops}
    km, co = sp.sp_kmap_build(c, case["kernel"], case["stride"], case.get("dilation", 1))
    n_in, n_out, pairs = float(km.n_in), float(km.n_out), float(km.total)
    for h in (km, co, c):
        h.close()
    if case["kind"] == "pool":
        ch = case["channels"]
        return {"bytes": byts + 2 * (n_in + n_out) * ch * elt + n_out * ch, "flops": 2 * pairs * ch}
    cin, cout, kvol = case["cin"], case["cout"], case["kernel"] ** 3
    one = n_in * cin + n_out * cout                        # both sides' rows
    w = kvol * cin * cout
    if case["kind"] == "layer":
        return {"bytes": byts + 2 * one * elt + w * (elt + 4), "flops": 6 * pairs * cin * cout}
    if not case["train"]:
        return {"bytes": byts + (one + n_in * cin) * elt + 2 * w * elt, "flops": 4 * pairs * cin * cout}
    return {"bytes": byts + (2 * one + 2 * n_in * cin) * elt + 2 * w * (elt + 4), "flops": 12 * pairs * cin * cout}


def tolerance(case):
    """fp32: sums of 32-bit products in another order.  bf16: results rounded once to 8 bits of significand; over a
    whole training step such roundings pass through eight layers and back."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 4e-4}
    return {"rel": 1e-2 if case["kind"] == "stack" else 5e-3, "max": 0.2 if case["kind"] == "stack" else 0.05}
