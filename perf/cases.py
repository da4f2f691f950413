"""The calls that a user of this library makes, as cases that can be timed and compared.

kind       what it stands for
frame      the probe update of a scene traced in its baked grids, then the maps read back
analytic   the same on the scene's primitives instead of grids
learned    the learned form: few rays, the network, the plain update as fallback
batch      many scenes of uneven size updated together
sample     irradiance at the shading points of an image
blend      Eq. 3 on the payload of a caller's own tracer
bake       one grid level of a scene baked from its primitives
train      optimiser steps of the learned form's network
infer      that network on a feature array

Scenes are of the three families the tests and the benchmark use: the box room, the
open field of spheres and boxes with a cascade of grids, and the uneven scenes of the
batched form. ``exact`` is the method's definition in binary64 torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2007_14394_amd import denoiser_weights
from paper_2007_14394_amd import sdfddgi as S

DEV = "cuda:0"
RAY_SIZES = (16, 32, 48, 64, 80, 96, 112, 144, 160, 208, 256, 272, 384, 512)


def listed():
    return [
        # the smallest scene: one frame and its maps, latency and launches
        dict(name="frame_room", kind="frame", scene="room", nx=8, ny=8, nz=8, grid=64, levels=1,
             rays=144, irr=8, depth=16, fp16=False, frames=1),
        # the open field at the benchmark's size, frames back to back
        dict(name="frame_open", kind="frame", scene="open", nx=32, ny=16, nz=32, grid=128,
             levels=4, rays=256, irr=8, depth=16, fp16=False, frames=4),
        dict(name="frame_open_fp16", kind="frame", scene="open", nx=32, ny=16, nz=32, grid=128,
             levels=4, rays=256, irr=8, depth=16, fp16=True, frames=4),
        # the analytic backend at the ray count of the standalone query's benchmark
        dict(name="analytic_open", kind="analytic", nx=32, ny=16, nz=32, prims=400, cluster=8,
             rays=64, frames=1),
        # the learned form in its steady state
        dict(name="learned_open", kind="learned", nx=32, ny=16, nz=32, grid=128, rays=256,
             fp16=True, frames=4),
        # a third of the benchmark's batch
        dict(name="batch_24", kind="batch", scenes=24, frames=4),
        # a 1920 x 1080 image shaded from the open field's probes
        dict(name="sample_image", kind="sample", nx=32, ny=16, nz=32, irr=8, n=1920 * 1080),
        dict(name="blend_open", kind="blend", nx=32, ny=16, nz=32, rays=256, irr=8, depth=16,
             fp16=False),
        # odd probe count, few rays, maps of another size
        dict(name="blend_ragged", kind="blend", nx=13, ny=7, nz=11, rays=80, irr=6, depth=12,
             fp16=False),
        # one level of the open field's cascade
        dict(name="bake_128", kind="bake", n0=128, n1=128, n2=128, prims=400, albedo=True),
        # the training script's batch size
        dict(name="train_16384", kind="train", batch=16384, count=262144, steps=8),
        dict(name="infer_1m", kind="infer", n=1 << 20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "analytic", "learned", "batch", "sample",
                       "blend", "blend", "bake", "train", "infer"])
    n = dict(nx=_log_int(rng, 4, 32), ny=_log_int(rng, 3, 16), nz=_log_int(rng, 4, 32))
    maps = rng.choice([(8, 16), (8, 16), (8, 16), (6, 12), (5, 9), (10, 16)])
    maps = dict(irr=maps[0], depth=maps[1])
    if kind == "frame":
        scene = rng.choice(["room", "open"])
        return dict(kind=kind, scene=scene, grid=_log_int(rng, 24, 128),
                    levels=1 if scene == "room" else rng.randint(1, 4),
                    rays=rng.choice([r for r in RAY_SIZES if r <= 256]),
                    fp16=rng.random() < 0.4, frames=rng.randint(1, 4), **n, **maps)
    if kind == "analytic":
        return dict(kind=kind, prims=_log_int(rng, 24, 400), cluster=rng.choice([4, 8, 16]),
                    rays=rng.choice([16, 32, 48, 64]), frames=1, **n)
    if kind == "learned":
        return dict(kind=kind, grid=_log_int(rng, 40, 128), rays=rng.choice([64, 144, 256]),
                    fp16=rng.random() < 0.5, frames=rng.randint(1, 4), **n)
    if kind == "batch":
        return dict(kind=kind, scenes=rng.randint(2, 24), frames=rng.randint(1, 4))
    if kind == "sample":
        return dict(kind=kind, irr=maps["irr"], n=_log_int(rng, 500, 1920 * 1080), **n)
    if kind == "blend":
        return dict(kind=kind, rays=rng.choice([r for r in RAY_SIZES if r <= 256]),
                    fp16=rng.random() < 0.4, **n, **maps)
    if kind == "bake":
        return dict(kind=kind, n0=_log_int(rng, 24, 128), n1=_log_int(rng, 24, 128),
                    n2=_log_int(rng, 24, 128), prims=_log_int(rng, 8, 400),
                    albedo=rng.random() < 0.7)
    if kind == "train":
        batch = _log_int(rng, 500, 16384)
        return dict(kind=kind, batch=batch, count=batch * rng.randint(2, 16), steps=rng.randint(1, 8))
    return dict(kind="infer", n=_log_int(rng, 1000, 1 << 20))


# ------------------------------------------------------------------ scenes ---

def _field(rng, count, lo, hi, sizes):
    """Spheres and axis-aligned boxes, sizes log-uniform (sphere diameter, box edge)."""
    kind = (rng.random(count) < 0.5).astype(np.int32)          # 1: box
    center = rng.uniform(lo, hi, (count, 3))
    half = 0.5 * np.exp(rng.uniform(math.log(sizes[0]), math.log(sizes[1]), (count, 3)))
    half[kind == 0] = half[kind == 0][:, :1]
    return dict(kind=kind, center=center, half=half, albedo=rng.uniform(0.2, 0.8, (count, 3)))


def _open_field(rng, count):
    return _field(rng, count, (-32.0, 0.0, -32.0), (32.0, 16.0, 32.0), (0.05, 4.0))


def _room(rng):
    """Five slabs (no ceiling) with inner faces at +-0.9, two spheres."""
    kind, center, half = [], [], []
    for axis in range(3):
        for sign in (-1.0, 1.0):
            if axis == 1 and sign > 0:
                continue
            c, h = [0.0] * 3, [1.0] * 3
            c[axis], h[axis] = sign * 0.95, 0.05
            kind.append(1), center.append(c), half.append(h)
    for _ in range(2):
        r = rng.uniform(0.1, 0.3)
        kind.append(0), center.append(list(rng.uniform(-0.9 + r, 0.9 - r, 3))), half.append([r] * 3)
    return dict(kind=np.array(kind, np.int32), center=np.array(center), half=np.array(half),
                albedo=rng.uniform(0.2, 0.8, (len(kind), 3)))


def _light(elevation, azimuth):
    el, az = math.radians(elevation), math.radians(azimuth)
    return (math.cos(el) * math.cos(az), math.sin(el), math.cos(el) * math.sin(az))


def _scene(case, seed):
    """Primitives, grid levels (n, origin, spacing), probe grid and parameters."""
    rng = np.random.default_rng([11, seed])
    n = (case["nx"], case["ny"], case["nz"])
    if case.get("scene") == "room":
        prims, sides, centre = _room(rng), (2.0,), 0.0
        origin = tuple(-0.7875 for _ in n)
        spacing = tuple(1.575 / (k - 1) for k in n)
        t_max, sky = 2.0 * math.sqrt(3.0), 0.0
    else:
        prims = _open_field(rng, case.get("prims", 400))
        sides, centre = (8.0, 16.0, 32.0, 64.0)[4 - case.get("levels", 4):], 8.0
        origin = (-31.0, 0.5, -31.0)
        spacing = tuple(e / (k - 1) for e, k in zip((62.0, 15.0, 62.0), n))
        t_max, sky = 64.0 * math.sqrt(3.0), 0.5
    g = case.get("grid", 2)
    levels = [((g,) * 3, (-s / 2, centre - s / 2, -s / 2), s / (g - 1)) for s in sides]
    azimuth = float(rng.uniform(0.0, 360.0))
    seeds = [int(v) for v in rng.integers(0, 2 ** 63, 4096)]
    return dict(prims=prims, levels=levels, n=n, origin=origin, spacing=spacing, t_max=t_max,
                sky=sky, rays=case["rays"], irr=case.get("irr", 8), depth=case.get("depth", 16),
                azimuth=azimuth, elevation=45.0, seeds=seeds)


def _batch_scenes(case, seed):
    """Uneven sizes that the scene count fixes, contents of the seed."""
    size = np.random.default_rng([15, case["scenes"]])
    rng = np.random.default_rng([12, seed])
    seeds = [int(v) for v in rng.integers(0, 2 ** 63, 4096)]
    scenes = []
    for _ in range(case["scenes"]):
        nx, ny, nz, g = (int(round(math.exp(size.uniform(math.log(a), math.log(b)))))
                         for a, b in ((4, 24), (4, 12), (4, 24), (32, 192)))
        side = float(max(nx, ny, nz) + 1)
        count = min(150, 10 + (nx + 1) * (ny + 1) * (nz + 1) // 8)
        prims = _field(rng, count, (0.0,) * 3, (nx + 1.0, ny + 1.0, nz + 1.0), (0.2, 1.5))
        ground = dict(kind=[1], center=[[side / 2, -1.0, side / 2]], half=[[side, 1.0, side]],
                      albedo=rng.uniform(0.2, 0.8, (1, 3)))
        prims = {k: np.concatenate([np.asarray(ground[k], prims[k].dtype), prims[k]]) for k in prims}
        scenes.append(dict(prims=prims, levels=[((g,) * 3, (0.0,) * 3, side / (g - 1))],
                           n=(nx, ny, nz), origin=(1.0,) * 3, spacing=(1.0,) * 3,
                           t_max=side * math.sqrt(3.0), sky=0.5,
                           rays=int(size.choice((64, 128, 256, 512))), irr=8, depth=16,
                           elevation=float(rng.uniform(25.0, 65.0)),
                           azimuth=float(rng.uniform(0.0, 360.0)), seeds=seeds))
    return scenes


def _sun(sc, frame):
    return _light(sc["elevation"], sc["azimuth"] + frame), (3.0, 3.0, 3.0)


def _params(sc, **more):
    p = S.sdfddgi_default_params()
    p.rays_per_probe, p.irr_res, p.depth_res, p.t_max = sc["rays"], sc["irr"], sc["depth"], sc["t_max"]
    p.sky_rgb[:] = [sc["sky"]] * 3
    for k, v in more.items():
        setattr(p, k, v)
    return p


def _bake_levels(sc):
    pr = sc["prims"]
    out = []
    for n, origin, spacing in sc["levels"]:
        sdf, alb = S.sdfddgi_bake_sdf(pr["kind"], pr["center"], pr["half"], pr["albedo"], n, origin,
                                      spacing, device=DEV)
        out.append(dict(sdf=sdf, albedo=alb, origin=origin, spacing=spacing))
    return out


def _pad_index(n):
    """Flat interior texel behind each position of a padded octahedral tile (edges fold
    onto themselves mirrored, corners take the opposite one)."""
    src = np.empty((n + 2, n + 2), np.int64)
    for y in range(n + 2):
        for x in range(n + 2):
            i, j = x - 1, y - 1
            in_x, in_y = 0 <= i < n, 0 <= j < n
            if in_x and not in_y:
                i, j = n - x, 0 if y == 0 else n - 1
            elif in_y and not in_x:
                i, j = 0 if x == 0 else n - 1, n - y
            elif not in_x:
                i, j = n - 1 if x == 0 else 0, n - 1 if y == 0 else 0
            src[y, x] = j * n + i
    return torch.from_numpy(src.reshape(-1)).to(DEV)


def _pad(interior, n):
    """[P, n*n, c] -> padded tiles [P, n+2, n+2, c]."""
    return interior[:, _pad_index(n)].reshape(interior.shape[0], n + 2, n + 2, -1)


def _history(sc, seed):
    """Maps as an earlier frame may have left them."""
    g = torch.Generator(device=DEV).manual_seed(1000003 * 7 + seed)
    P = sc["n"][0] * sc["n"][1] * sc["n"][2]
    irr = 0.4 + 1.6 * torch.rand((P, sc["irr"] ** 2, 3), generator=g, device=DEV)
    mean = sc["t_max"] * (0.1 + 0.8 * torch.rand((P, sc["depth"] ** 2, 1), generator=g, device=DEV))
    var = mean * torch.rand(mean.shape, generator=g, device=DEV) * 0.25
    return (_pad(irr, sc["irr"]).contiguous(),
            _pad(torch.cat([mean, mean * mean + var], 2), sc["depth"]).contiguous())


# ---------------------------------------------------------------- the calls ---

def _make_context(case, sc, seed):
    flags = S.SDFDDGI_FLAG_FP16 if case.get("fp16") else 0
    if case["kind"] == "analytic":
        pr = sc["prims"]
        ctx = S.sdfddgi_create_analytic(pr["kind"], pr["center"], pr["half"], pr["albedo"], sc["n"],
                                        sc["origin"], sc["spacing"], _params(sc, flags=flags),
                                        case["cluster"], DEV)
    else:
        more = dict(flags=flags)
        if case["kind"] == "learned":
            w = denoiser_weights.load()
            more.update(learned_rays=w["learned_rays"], fallback_error=w["tau"])
        ctx = S.sdfddgi_create(_bake_levels(sc), sc["n"], sc["origin"], sc["spacing"],
                               _params(sc, **more))
    S.sdfddgi_set_maps(ctx, *_history(sc, seed))
    return ctx


def _features(case_seed, n):
    g = torch.Generator(device=DEV).manual_seed(1000003 * 5 + case_seed)
    f = torch.zeros((n, S.SDFDDGI_FEATURES), device=DEV)
    f[:, 3:6] = 0.2 + 0.8 * torch.rand((n, 3), generator=g, device=DEV)
    f[:, 0:3] = (f[:, 3:6] * (1 + 0.1 * torch.randn((n, 3), generator=g, device=DEV))).clamp_min(0)
    f[:, 6:7] = 0.3 + 5.0 * torch.rand((n, 1), generator=g, device=DEV)
    f[:, 7:8] = f[:, 6:7] * (1 + 0.1 * torch.rand((n, 1), generator=g, device=DEV))
    d = torch.randn((n, 3), generator=g, device=DEV)
    f[:, 8:11] = d / d.norm(dim=1, keepdim=True)
    f[:, 11] = 0.4 * torch.rand(n, generator=g, device=DEV)
    f[:, 12] = 1.0
    t = torch.empty((n, 4), device=DEV)
    t[:, :3] = 0.4 * (f[:, 0:3] - f[:, 3:6]) + 0.02 * torch.randn((n, 3), generator=g, device=DEV)
    t[:, 3] = (f[:, 3:6].sum(1) + 0.05)
    return f, t


def _image_points(case, sc, seed):
    """Shading points of an image of a rolling ground seen from above, row by row."""
    g = torch.Generator(device=DEV).manual_seed(1000003 * 3 + seed)
    n = case["n"]
    w = max(1, int(math.sqrt(n * 16 / 9)))
    i = torch.arange(n, device=DEV)
    u, v = (i % w).float() / w, (i // w).float() * w / n
    ph = torch.rand(6, generator=g, device=DEV) * 6.28
    x, z = -30.0 + 60.0 * u, -30.0 + 60.0 * v
    y = 6.0 + 3.0 * torch.sin(0.31 * x + ph[0]) + 2.0 * torch.sin(0.23 * z + ph[1])
    nx = -0.93 * torch.cos(0.31 * x + ph[0]) + 0.3 * torch.sin(9.0 * x + ph[2])
    nz = -0.46 * torch.cos(0.23 * z + ph[1]) + 0.3 * torch.sin(7.0 * z + ph[3])
    nrm = torch.stack([nx, torch.ones_like(nx), nz], 1)
    return torch.stack([x, y, z], 1).contiguous(), nrm.contiguous()


def _payload(sc, seed):
    """What a tracer hands over: mostly sky at t_max, the rest lit surfaces."""
    g = torch.Generator(device=DEV).manual_seed(1000003 * 9 + seed)
    P = sc["n"][0] * sc["n"][1] * sc["n"][2]
    out = torch.empty((P, sc["rays"], 4), device=DEV)
    out[..., :3] = 0.5
    out[..., 3] = sc["t_max"]
    hit = torch.rand((P, sc["rays"]), generator=g, device=DEV) < 0.3
    val = torch.rand(out.shape, generator=g, device=DEV)
    val[..., 3] *= 0.5 * sc["t_max"]
    return torch.where(hit[..., None], val, out).contiguous()


def _he_init(seed):
    rng = np.random.default_rng([13, seed])
    parts = []
    for rows, cols, bias in ((64, 16, 0), (64, 64, 64), (64, 64, 64), (4, 64, 4)):
        parts += [rng.normal(0.0, math.sqrt(2.0 / cols), rows * cols), np.zeros(bias)]
    th = np.concatenate(parts)
    th[-1] = -3.0
    return th.astype(np.float32)


TRAIN_SEED, TRAIN_LR, HEAD_WEIGHT, MIN_ERROR = 12345, 2e-4, 0.1, 1e-4


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case, frame=0)
    if kind in ("frame", "analytic", "learned"):
        sc = st["sc"] = _scene(case, seed)
        st["ctx"] = ctx = _make_context(case, sc, seed)
        st["irr"] = torch.empty(ctx.irr_shape, device=DEV)
        st["dep"] = torch.empty(ctx.depth_shape, device=DEV)
        if kind == "learned":
            w = denoiser_weights.load()
            st["den"] = S.sdfddgi_denoiser_create(w["params"], w["irr_scale"], w["depth_scale"], DEV)
            for _ in range(4):      # past the first frames, which take the fallback everywhere
                _learned_frame(st)
    elif kind == "batch":
        scs = st["scs"] = _batch_scenes(case, seed)
        rows = [dict(_bake_levels(sc)[0], probe_n=sc["n"], probe_origin=sc["origin"],
                     probe_spacing=sc["spacing"], params=_params(sc)) for sc in scs]
        st["batch"] = S.sdfddgi_batch_create(rows)
    elif kind in ("sample", "blend"):
        sc = st["sc"] = _scene(dict(case, grid=16, levels=1, prims=8, rays=case.get("rays", 16)), seed)
        st["ctx"] = _make_context(case, sc, seed)
        if kind == "sample":
            st["points"], st["normals"] = _image_points(case, sc, seed)
            st["out"] = torch.empty_like(st["points"])
        else:
            st["payload"] = _payload(sc, seed)
            st["irr"] = torch.empty(st["ctx"].irr_shape, device=DEV)
            st["dep"] = torch.empty(st["ctx"].depth_shape, device=DEV)
    elif kind == "bake":
        st["prims"] = _open_field(np.random.default_rng([14, seed]), case["prims"])
    elif kind == "train":
        st["features"], st["targets"] = _features(seed, case["count"])
        st["trainer"] = S.sdfddgi_trainer_create(_he_init(seed), HEAD_WEIGHT, MIN_ERROR, device=DEV)
        st["step"] = 0
    else:
        w = denoiser_weights.load()
        st["den"] = S.sdfddgi_denoiser_create(w["params"], w["irr_scale"], w["depth_scale"], DEV)
        st["features"], _ = _features(seed, case["n"])
        st["out"] = torch.empty((case["n"], 4), device=DEV)
    return st


def _learned_frame(st):
    light, rad = _sun(st["sc"], st["frame"])
    S.sdfddgi_update_frame_learned(st["ctx"], st["den"], light, rad,
                                   st["sc"]["seeds"][st["frame"] % 4096])
    st["frame"] += 1


def _bake_grid(case):
    longest = max(case["n0"], case["n1"], case["n2"])
    return (case["n0"], case["n1"], case["n2"]), (-16.0, -8.0, -16.0), 32.0 / (longest - 1)


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind in ("frame", "analytic"):
        sc = st["sc"]
        for _ in range(case["frames"]):
            light, rad = _sun(sc, st["frame"])
            S.sdfddgi_update_frame(st["ctx"], light, rad, sc["seeds"][st["frame"] % 4096])
            st["frame"] += 1
        return S.sdfddgi_get_maps(st["ctx"], st["irr"], st["dep"])
    if kind == "learned":
        for _ in range(case["frames"]):
            _learned_frame(st)
        return S.sdfddgi_get_maps(st["ctx"], st["irr"], st["dep"])
    if kind == "batch":
        for _ in range(case["frames"]):
            S.sdfddgi_batch_update_frame(st["batch"], [_sun(sc, st["frame"]) for sc in st["scs"]],
                                         st["scs"][0]["seeds"][st["frame"] % 4096])
            st["frame"] += 1
        return [S.sdfddgi_batch_get_maps(st["batch"], k) for k in range(case["scenes"])]
    if kind == "sample":
        return S.sdfddgi_sample_irradiance(st["ctx"], st["points"], st["normals"], st["out"])
    if kind == "blend":
        S.sdfddgi_blend(st["ctx"], st["payload"], st["sc"]["seeds"][st["frame"] % 4096])
        st["frame"] += 1
        return S.sdfddgi_get_maps(st["ctx"], st["irr"], st["dep"])
    if kind == "bake":
        n, origin, spacing = _bake_grid(case)
        pr = st["prims"]
        return S.sdfddgi_bake_sdf(pr["kind"], pr["center"], pr["half"], pr["albedo"], n, origin,
                                  spacing, with_albedo=case["albedo"], device=DEV)
    if kind == "train":
        for _ in range(case["steps"]):
            S.sdfddgi_trainer_step(st["trainer"], st["features"], st["targets"], case["batch"],
                                   TRAIN_SEED + 100003 * st["step"], TRAIN_LR)
            st["step"] += 1
        return S.sdfddgi_trainer_get_params(st["trainer"])
    return S.sdfddgi_denoiser_infer(st["den"], st["features"], st["out"])


# --------------------------------------------------------------------- work ---

def work(case):
    """Inputs once, outputs once; for the traces 10 samples a ray, 25 operations each
    (position, level, cell, seven lerps, step), one hit ray in ten with a shadow ray."""
    kind = case["kind"]

    def update(P, R, irr, depth, grid_bytes):
        maps = P * ((irr + 2) ** 2 * 3 + (depth + 2) ** 2 * 2) * 4
        flops = P * R * (25 * 10 * 1.2 + 2 * (3 * irr * irr + 2 * depth * depth))
        return grid_bytes + 2 * maps, flops, maps

    if kind in ("frame", "analytic", "learned"):
        P = case["nx"] * case["ny"] * case["nz"]
        R = 32 if kind == "learned" else case["rays"]
        irr, depth = case.get("irr", 8), case.get("depth", 16)
        levels = 0 if kind == "analytic" else case.get("levels", 4)
        grids = levels * case.get("grid", 0) ** 3 * (2 if case.get("fp16") else 4)
        b, f, maps = update(P, R, irr, depth, grids)
        if kind == "learned":
            f += P * irr * irr * 2 * 9472
        return dict(bytes=case["frames"] * b + 2 * maps, flops=case["frames"] * f)
    if kind == "batch":
        scs = _batch_scenes(case, 0)
        total = dict(bytes=0.0, flops=0.0)
        for sc in scs:
            P = sc["n"][0] * sc["n"][1] * sc["n"][2]
            b, f, maps = update(P, sc["rays"], 8, 16, sc["levels"][0][0][0] ** 3 * 2)
            total["bytes"] += case["frames"] * b + 2 * maps
            total["flops"] += case["frames"] * f
        return total
    if kind == "sample":
        atlas = case["nx"] * case["ny"] * case["nz"] * (case["irr"] + 2) ** 2 * 12
        return dict(bytes=36 * case["n"] + atlas, flops=case["n"] * 8 * 30)
    if kind == "blend":
        P, R = case["nx"] * case["ny"] * case["nz"], case["rays"]
        maps = P * ((case["irr"] + 2) ** 2 * 3 + (case["depth"] + 2) ** 2 * 2) * 4
        return dict(bytes=16 * P * R + 4 * maps,
                    flops=2 * P * R * (3 * case["irr"] ** 2 + 2 * case["depth"] ** 2))
    if kind == "bake":
        nv = case["n0"] * case["n1"] * case["n2"]
        return dict(bytes=nv * (16 if case["albedo"] else 4), flops=20 * nv)
    if kind == "train":
        return dict(bytes=80 * case["batch"] * case["steps"],
                    flops=3 * 2 * 9472 * case["batch"] * case["steps"])
    return dict(bytes=80 * case["n"], flops=2 * 9472 * case["n"])


# -------------------------------------------------------------------- exact ---

def _splitmix(state):
    state = (state + 0x9E3779B97F4A7C15) & (2 ** 64 - 1)
    z = state
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & (2 ** 64 - 1)
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & (2 ** 64 - 1)
    return state, z ^ (z >> 31)


def _directions(seed, R):
    us, state = [], seed
    for _ in range(3):
        state, z = _splitmix(state)
        us.append((z >> 11) * 2.0 ** -53)
    u1, a1, a2 = us[0], 2 * math.pi * us[1], 2 * math.pi * us[2]
    x, y = math.sqrt(1 - u1) * math.sin(a1), math.sqrt(1 - u1) * math.cos(a1)
    z, w = math.sqrt(u1) * math.sin(a2), math.sqrt(u1) * math.cos(a2)
    q = np.array([[1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w)],
                  [2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w)],
                  [2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)]])
    i = np.arange(R)
    cz = 1 - (2 * i + 1) / R
    phi = 2 * np.pi * np.modf(i * ((math.sqrt(5) - 1) / 2))[0]
    r = np.sqrt(1 - cz * cz)
    return torch.from_numpy(np.stack([r * np.cos(phi), r * np.sin(phi), cz], 1) @ q.T).to(DEV)


def _texel_dirs(n):
    c = (np.arange(n) + 0.5) / n * 2 - 1
    u, v = np.meshgrid(c, c)
    z = 1 - np.abs(u) - np.abs(v)
    su, sv = np.where(u >= 0, 1.0, -1.0), np.where(v >= 0, 1.0, -1.0)
    fu, fv = np.where(z < 0, (1 - np.abs(v)) * su, u), np.where(z < 0, (1 - np.abs(u)) * sv, v)
    d = np.stack([fu, fv, z], -1).reshape(-1, 3)
    return torch.from_numpy(d / np.linalg.norm(d, axis=1, keepdims=True)).to(DEV)


def _cell(u, n):
    i = u.floor().clamp(0, n - 2)
    return i.long(), (u - i).clamp(0, 1)


def _trilinear(grid, x, origin, spacing):
    """Values [m] or [m, c] of a vertex grid [n2, n1, n0(, c)] at points x [m, 3]."""
    n2, n1, n0 = grid.shape[:3]
    (i, fx), (j, fy), (k, fz) = (_cell((x[:, a] - origin[a]) / spacing, n)
                                 for a, n in enumerate((n0, n1, n2)))
    if grid.dim() == 4:
        fx, fy, fz = fx[:, None], fy[:, None], fz[:, None]

    def at(dx, dy, dz):
        return grid[k + dz, j + dy, i + dx].double()

    def edge(dy, dz):
        return at(0, dy, dz) * (1 - fx) + at(1, dy, dz) * fx

    return ((edge(0, 0) * (1 - fy) + edge(1, 0) * fy) * (1 - fz) +
            (edge(0, 1) * (1 - fy) + edge(1, 1) * fy) * fz)


class _Grids:
    """The cascade as the update defines it: distances, levels, normals, albedo."""

    def __init__(self, levels):
        self.levels = levels
        self.boxes = []
        for a, lv in enumerate(levels):
            n = lv["sdf"].shape[::-1]
            m = 1 if a < len(levels) - 1 else 0
            o, s = lv["origin"], lv["spacing"]
            self.boxes.append(([o[c] + m * s for c in range(3)],
                               [o[c] + (n[c] - 1 - m) * s for c in range(3)]))

    def level(self, x):
        out = torch.full((x.shape[0],), -1, dtype=torch.long, device=x.device)
        for a in reversed(range(len(self.levels))):
            lo, hi = (torch.tensor(b, dtype=torch.float64, device=x.device) for b in self.boxes[a])
            out[((x >= lo) & (x <= hi)).all(1)] = a
        return out

    def each(self, lev, fn, like):
        for a, lv in enumerate(self.levels):
            at = (lev == a).nonzero()[:, 0]
            if at.numel():
                like[at] = fn(lv, at)
        return like

    def sample(self, x):
        lev = self.level(x)
        d = torch.zeros(x.shape[0], dtype=torch.float64, device=x.device)
        self.each(lev, lambda lv, at: _trilinear(lv["sdf"], x[at], lv["origin"], lv["spacing"]), d)
        return d, lev, lev < 0

    def surface(self, x, w, lev):
        def normal(lv, at):
            g = torch.empty((at.numel(), 3), dtype=torch.float64, device=x.device)
            for a in range(3):
                e = torch.zeros(3, dtype=torch.float64, device=x.device)
                e[a] = 0.5 * lv["spacing"]
                g[:, a] = (_trilinear(lv["sdf"], x[at] + e, lv["origin"], lv["spacing"]) -
                           _trilinear(lv["sdf"], x[at] - e, lv["origin"], lv["spacing"]))
            return g
        g = self.each(lev, normal, torch.zeros_like(x))
        alb = self.each(lev, lambda lv, at: _trilinear(lv["albedo"], x[at], lv["origin"],
                                                       lv["spacing"]), torch.zeros_like(x))
        return _unit_or(g, -w), alb


def _unit_or(g, other):
    l2 = (g * g).sum(1, keepdim=True)
    return torch.where(l2 >= 1e-24, g / l2.clamp_min(1e-30).sqrt(), other)


def _prim_distances(prims, x):
    """[m, prims] signed distances."""
    c, h = (torch.from_numpy(prims[k]).to(x) for k in ("center", "half"))
    ball = torch.from_numpy(prims["kind"]).to(x.device) == 0
    d = x[:, None] - c
    q = d.abs() - h
    box = q.clamp_min(0).square_().sum(2).sqrt_() + q.amax(2).clamp_max(0)
    return torch.where(ball, d.square().sum(2).sqrt_() - h[:, 0], box)


class _Prims:
    """The union of primitives itself: no box, the nearest primitive's normal and albedo."""

    def __init__(self, prims):
        self.prims = prims
        self.albedo = torch.from_numpy(prims["albedo"]).to(DEV)

    def sample(self, x):
        d = torch.empty(x.shape[0], dtype=torch.float64, device=x.device)
        slot = torch.empty(x.shape[0], dtype=torch.long, device=x.device)
        for a in range(0, x.shape[0], 1 << 17):
            d[a:a + (1 << 17)], slot[a:a + (1 << 17)] = _prim_distances(self.prims,
                                                                       x[a:a + (1 << 17)]).min(1)
        return d, slot, torch.zeros_like(slot, dtype=torch.bool)

    def surface(self, x, w, slot):
        c, h = (torch.from_numpy(self.prims[k]).to(x)[slot] for k in ("center", "half"))
        ball = (torch.from_numpy(self.prims["kind"]).to(x.device) == 0)[slot][:, None]
        d = x - c
        q = d.abs() - h
        sign = torch.where(d >= 0, 1.0, -1.0).double()
        face = torch.nn.functional.one_hot(q.argmax(1), 3).double()
        box = torch.where(q.amax(1, keepdim=True) > 0, q.clamp_min(0), face) * sign
        return _unit_or(torch.where(ball, d, box), -w), self.albedo[slot]


def _march(world, o, w, t_max, primary, eps=1e-3, steps=64):
    """(outcome 0 miss, 2 hit, 4 inside; t; what the last sample found) of rays."""
    m = o.shape[0]
    kind = torch.zeros(m, dtype=torch.long, device=o.device)
    where = torch.zeros(m, dtype=torch.long, device=o.device)
    t = torch.zeros(m, dtype=torch.float64, device=o.device)
    live = torch.arange(m, device=o.device)
    for k in range(steps):
        live = live[t[live] <= t_max]
        if not live.numel():
            break
        d, tag, gone = world.sample(o[live] + t[live, None] * w[live])
        inside = (d < 0) & ~gone if primary and k == 0 else torch.zeros_like(gone)
        last = ~gone & ~inside & ((d < eps) | (k == steps - 1))
        where[live] = tag
        kind[live[inside]] = 4
        kind[live[last]] = 2
        go = ~(gone | inside | last)
        t[live[go]] += d[go]
        live = live[go]
    return kind, t, where


def _lookup(atlas, sc, x, n):
    """Trilinear over the eight probes around x, bilinear in each one's padded tile."""
    res, (nx, ny, nz) = sc["irr"], sc["n"]
    cells = [_cell((x[:, a] - sc["origin"][a]) / sc["spacing"][a], sc["n"][a]) for a in range(3)]
    p = n / n.abs().sum(1, keepdim=True)
    u, v = p[:, 0], p[:, 1]
    su, sv = torch.where(u >= 0, 1.0, -1.0).double(), torch.where(v >= 0, 1.0, -1.0).double()
    low = n[:, 2] < 0
    u, v = torch.where(low, (1 - v.abs()) * su, u), torch.where(low, (1 - u.abs()) * sv, v)
    (au, fu), (av, fv) = (_cell((res * (s + 1) + 1) * 0.5, res + 2) for s in (u, v))
    out = torch.zeros_like(x)
    for c in range(8):
        q, wp = 0, 1.0
        for a, stride in enumerate((1, nx, nx * ny)):
            i, f = cells[a]
            up = (c >> a) & 1
            q = q + (i + up) * stride
            wp = wp * (f if up else 1 - f)
        for dv in (0, 1):
            for du in (0, 1):
                wt = (fu if du else 1 - fu) * (fv if dv else 1 - fv)
                out += (wp * wt)[:, None] * atlas[q, av + dv, au + du].double()
    return out


def _mix(payload, dirs, sc, irr, dep, h=0.97, sharp=50.0):
    """Eq. 3 on [P, R, 4], mixed with the padded maps irr and dep, padded."""
    out = []
    for n, prev, s, vals, scale in ((sc["irr"], irr, 1.0, payload[..., :3], math.pi),
                                    (sc["depth"], dep, sharp,
                                     torch.stack([payload[..., 3], payload[..., 3] ** 2], -1), 1.0)):
        wt = (_texel_dirs(n) @ dirs.T).clamp_min(0) ** s
        e = scale * torch.matmul(wt / wt.sum(1, keepdim=True), vals.contiguous())
        old = prev[:, 1:-1, 1:-1].reshape(prev.shape[0], n * n, -1).double()
        out.append(_pad(h * old + (1 - h) * e, n))
    return out


def _frames(sc, world, irr, dep, frames, fresh=False):
    """The update's frames 0 .. frames-1 from the maps irr, dep."""
    n = sc["n"]
    idx = torch.arange(n[0] * n[1] * n[2], device=DEV)
    idx = torch.stack([idx % n[0], idx // n[0] % n[1], idx // (n[0] * n[1])], 1).double()
    pos = (torch.tensor(sc["origin"], device=DEV, dtype=torch.float64) +
           idx * torch.tensor(sc["spacing"], device=DEV, dtype=torch.float64))
    R = sc["rays"]
    for f in range(frames):
        light, rad = _sun(sc, f)
        to_sun = torch.tensor(light, device=DEV, dtype=torch.float64)
        dirs = _directions(sc["seeds"][f], R)
        parts = []
        for a in range(0, pos.shape[0], 4096):
            o = pos[a:a + 4096].repeat_interleave(R, 0)
            w = dirs.repeat(o.shape[0] // R, 1)
            kind, t, tag = _march(world, o, w, sc["t_max"], True)
            pay = torch.full((o.shape[0], 4), float(sc["sky"]), device=DEV, dtype=torch.float64)
            pay[:, 3] = sc["t_max"]
            pay[kind == 4] = 0.0
            at = (kind == 2).nonzero()[:, 0]
            if at.numel():
                x = o[at] + t[at, None] * w[at]
                nrm, alb = world.surface(x, w[at], tag[at])
                ndl = nrm @ to_sun
                up = (ndl > 0).nonzero()[:, 0]
                lit = torch.zeros_like(ndl)
                if up.numel():
                    blocked = _march(world, x[up] + 4e-3 * nrm[up], to_sun.expand(up.numel(), 3),
                                     sc["t_max"], False)[0]
                    lit[up] = torch.where(blocked == 0, ndl[up], 0.0)
                e = lit[:, None] * torch.tensor(rad, device=DEV, dtype=torch.float64)
                pay[at, :3] = alb / math.pi * (e + _lookup(irr, sc, x, nrm))
                pay[at, 3] = t[at]
            parts.append(pay.reshape(-1, R, 4))
        irr, dep = _mix(torch.cat(parts), dirs, sc, irr, dep, 0.0 if fresh and f == 0 else 0.97)
    return irr, dep


def _network(theta, x):
    off, mats = 0, []
    for rows, cols, bias in ((64, 16, 0), (64, 64, 64), (64, 64, 64), (4, 64, 4)):
        w = theta[off:off + rows * cols].reshape(rows, cols)
        off += rows * cols
        mats.append((w, theta[off:off + bias] if bias else None))
        off += bias
    for k, (w, b) in enumerate(mats):
        x = x @ w.T if b is None else x @ w.T + b
        x = x.relu() if k < 3 else x
    return x


def _trained(case, seed):
    x, t = (v.double() for v in _features(seed, case["count"]))
    theta = torch.from_numpy(_he_init(seed)).to(DEV).double().requires_grad_(True)
    m, v = torch.zeros_like(theta), torch.zeros_like(theta)
    for k in range(case["steps"]):
        pick = np.array([_splitmix(TRAIN_SEED + 100003 * k + i)[1] % case["count"]
                         for i in range(case["batch"])])
        pick = torch.from_numpy(pick.astype(np.int64)).to(DEV)
        o, z = _network(theta, x[pick]), t[pick]
        d = o[:, :3] - z[:, :3]
        r = (d.abs().sum(1) / z[:, 3]).detach().clamp_min(MIN_ERROR)
        loss = (d.square().sum(1) + HEAD_WEIGHT * (o[:, 3] - r.log()).square()).mean()
        g, = torch.autograd.grad(loss, theta)
        with torch.no_grad():
            m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
            theta -= TRAIN_LR * (m / (1 - 0.9 ** (k + 1))) / (
                (v / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
    return theta.detach().cpu()


def exact(case, seed):
    kind = case["kind"]
    if kind == "learned":       # the fallback's choice of probes hangs on 16-bit roundings
        return None
    if kind in ("frame", "analytic"):
        sc = _scene(case, seed)
        world = _Prims(sc["prims"]) if kind == "analytic" else _Grids(_exact_levels(sc))
        return _frames(sc, world, *_history(sc, seed), case["frames"])
    if kind == "batch":
        out = []
        for sc in _batch_scenes(case, seed):
            zero = [torch.zeros_like(m) for m in _history(sc, 0)]
            out.append(_frames(sc, _Grids(_exact_levels(sc)), *zero, case["frames"], fresh=True))
        return out
    if kind in ("sample", "blend"):
        sc = _scene(dict(case, grid=16, levels=1, prims=8, rays=case.get("rays", 16)), seed)
        irr, dep = _history(sc, seed)
        if kind == "sample":
            x, n = _image_points(case, sc, seed)
            return _lookup(irr, sc, x.double(), n.double())
        return _mix(_payload(sc, seed).double(), _directions(sc["seeds"][0], sc["rays"]), sc, irr, dep)
    if kind == "bake":
        n, origin, spacing = _bake_grid(case)
        prims = _open_field(np.random.default_rng([14, seed]), case["prims"])
        lv = _exact_level(prims, n, origin, spacing)
        return lv["sdf"], lv["albedo"] if case["albedo"] else None
    if kind == "train":
        return _trained(case, seed)
    theta = torch.from_numpy(denoiser_weights.load()["params"]).to(DEV)
    x, _ = _features(seed, case["n"])
    return _network(theta.bfloat16().double(), x.bfloat16().double())


def _exact_level(prims, n, origin, spacing):
    axes = [o + spacing * torch.arange(k, device=DEV, dtype=torch.float64) for o, k in zip(origin, n)]
    z, y, x = torch.meshgrid(axes[2], axes[1], axes[0], indexing="ij")
    pts = torch.stack([x, y, z], -1).reshape(-1, 3)
    sdf, slot, _ = _Prims(prims).sample(pts)
    alb = torch.from_numpy(prims["albedo"]).to(DEV)[slot]
    return dict(sdf=sdf.reshape(n[2], n[1], n[0]), albedo=alb.reshape(n[2], n[1], n[0], 3),
                origin=origin, spacing=spacing)


def _exact_levels(sc):
    """The levels a context is given: distances and albedo rounded to binary32."""
    out = []
    for n, origin, spacing in sc["levels"]:
        lv = _exact_level(sc["prims"], n, origin, spacing)
        out.append(dict(lv, sdf=lv["sdf"].float(), albedo=lv["albedo"].float()))
    return out
