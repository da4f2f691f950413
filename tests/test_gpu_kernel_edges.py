"""The device baker, the map read-back and the trace at the sizes where their tilings
can go wrong: grids thinner and longer than a brick, ragged bricks, primitive counts
around the staging chunk, equal and non-finite primitives; maps whose float counts are
not multiples of four; grids at the edges of the trace's cell bricks, too long for its
24-bit products, and levels that are not nested; analytic scenes whose candidate cells
hold one to too many primitives, and rays beyond them; the blend's groups and tiles; training
steps and inference around their workgroups' sizes."""
import sys

import numpy as np
import pytest

import oracle
import scenegen
from scenegen import Params, Primitives, ProbeGrid, SDFLevel, Workload
from tests.helpers import fp16_grid, frame

pytestmark = pytest.mark.gpu


def announce(msg):
    print(f"[gpu] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def S():
    import torch
    from paper_2007_14394_amd import sdfddgi
    assert torch.cuda.is_available(), "GPU tests need a visible gfx950 device"
    sdfddgi.load_library()
    return sdfddgi


def bake_prims(count, special):
    rng = np.random.default_rng(count)
    p = scenegen.open_scene_primitives(rng, count, (-8.0, 0.0, -8.0), (8.0, 4.0, 8.0),
                                       size_range=(0.05, 6.0))
    if special == "ties":       # every primitive twice: the lower index keeps the albedo
        for f in (p.kind, p.center, p.half):
            f[count // 2:count // 2 * 2] = f[:count // 2]
    elif special == "far":      # huge, infinite and undefined centres never win by accident
        p.center[0] = 1e200
        p.center[1] = np.inf
        p.center[2] = np.nan
        p.half[3] = np.inf
    return p


@pytest.mark.parametrize("n,count,special", [
    ((2, 2, 2), 1, None), ((16, 4, 4), 255, None), ((17, 5, 3), 256, "ties"),
    ((2, 3, 301), 257, "ties"), ((300, 2, 2), 64, "far"), ((3, 90, 5), 513, "far"),
    ((33, 31, 29), 600, "ties")])
@pytest.mark.parametrize("spacing", [0.004, 0.7])
def test_bake_equals_the_host_baker(S, n, count, special, spacing):
    announce(f"bake {n} x {count} primitives {special} spacing {spacing}")
    p = bake_prims(count, special)
    origin = (-3.0, 0.4, -2.0)
    host = scenegen.bake(p, n, origin, spacing)
    sdf, alb = S.sdfddgi_bake_sdf(p.kind, p.center, p.half, p.albedo, n, origin, spacing)
    assert np.array_equal(sdf.cpu().numpy().view(np.int32), host.sdf.view(np.int32))
    assert np.array_equal(alb.cpu().numpy().view(np.int32), host.albedo.view(np.int32))


@pytest.mark.parametrize("res", [(2, 3), (5, 9), (8, 16)])
@pytest.mark.parametrize("offset", [0, 1])
def test_maps_read_back_as_installed(S, res, offset):
    import torch
    announce(f"get_maps {res} offset {offset}")
    w = scenegen.small_cascade(2, probes=(3, 3, 3), rays=16)
    ctx = S.context_from_workload(w, irr_res=res[0], depth_res=res[1])
    irr = torch.rand(ctx.irr_shape, device="cuda:0")
    dep = torch.rand(ctx.depth_shape, device="cuda:0")
    S.sdfddgi_set_maps(ctx, irr, dep)
    outs = []
    for t in (irr, dep):    # also at an address that is not a multiple of 16 bytes
        room = torch.full((t.numel() + 8,), -1.0, device="cuda:0")
        outs.append((room, room[offset:offset + t.numel()].reshape(t.shape)))
    S.sdfddgi_get_maps(ctx, outs[0][1], outs[1][1])
    for t, (room, view) in zip((irr, dep), outs):
        assert torch.equal(view, t)
        assert int((room == -1.0).sum()) == 8
    S.sdfddgi_destroy(ctx)


def random_level(n, origin, spacing, seed):
    """Distances of no scene: any value a sample may meet, few of them hits."""
    rng = np.random.default_rng(seed)
    sdf = (rng.uniform(0.02, 0.3, n[::-1]) * np.exp(rng.normal(size=n[::-1]))).astype(np.float32)
    sdf[rng.random(sdf.shape) < 0.03] = -0.2
    return SDFLevel(n=n, origin=origin, spacing=spacing, sdf=sdf, albedo=None)


def trace_workload(levels, probes, rays, t_max=30.0):
    none = Primitives(np.zeros(0, np.int32), np.zeros((0, 3)), np.zeros((0, 3)), np.zeros((0, 3)))
    return Workload("edges", none, levels, probes,
                    Params(rays_per_probe=rays, t_max=t_max, max_steps=24, hit_eps=5e-3), [])


def check_trace(S, w, half):
    import torch
    ref = fp16_grid(w) if half else w
    fr = frame((0.3, 1.0, 0.2), seed=77)
    ctx = S.context_from_workload(w, flags=S.SDFDDGI_FLAG_RECORD_RAYS |
                                  (S.SDFDDGI_FLAG_FP16 if half else 0))
    S.sdfddgi_update_frame(ctx, fr.dir_to_light, fr.radiance_rgb, fr.rotation_seed)
    rec = S.sdfddgi_get_ray_records(ctx).cpu().numpy()
    torch.cuda.synchronize()
    S.sdfddgi_destroy(ctx)
    chk = oracle.Checker(ref)
    irr0, dep0 = (np.zeros(s, np.float32) for s in scenegen.atlas_shapes(w.num_probes, w.params))
    _, _, _, ref_rec = chk.update_probes(fr, True, irr0, dep0, want_records=True)
    assert np.array_equal(rec, ref_rec)
    return ref_rec


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("n", [(2, 2, 2), (4, 4, 4), (5, 4, 3), (3, 8, 5), (13, 6, 10),
                               (66001, 3, 2), (2, 66001, 3), (3, 2, 66001)])
def test_trace_at_brick_edges(S, n, half):
    announce(f"trace on a {n} grid, half={half}")
    spacing = 0.25
    origin = (-1.0, 0.5, -2.0)
    ext = [spacing * (k - 1) for k in n]
    probes = ProbeGrid((3, 2, 3), tuple(o + 0.05 * min(e, 40.0) for o, e in zip(origin, ext)),
                       tuple(0.4 * min(e, 40.0) for e in ext))
    for rays in (16, 48):
        check_trace(S, trace_workload([random_level(n, origin, spacing, sum(n))], probes, rays),
                    half)


@pytest.mark.parametrize("half", [False, True])
def test_trace_through_levels_that_are_not_nested(S, half):
    announce(f"levels sticking out of the next coarser one, half={half}")
    levels = [random_level((9, 9, 9), (-1.0, -1.0, -1.0), 0.25, 5),
              random_level((10, 6, 10), (-0.5, -1.5, -1.5), 0.4, 6),     # cuts level 0's corner
              random_level((11, 12, 9), (-3.0, -3.0, -3.0), 0.55, 7)]
    probes = ProbeGrid((4, 3, 4), (-2.0, -2.0, -2.0), (0.9, 1.1, 0.9))
    rec = check_trace(S, trace_workload(levels, probes, 64), half)
    assert set(np.unique(rec[..., 0] >> 8)) >= {0, 1, 2}


@pytest.mark.parametrize("probes,rays", [((2, 2, 2), 16), ((5, 3, 7), 1008), ((17, 9, 11), 176)])
def test_trace_covers_every_ray(S, probes, rays):
    # the ray queue's claims: fewer rays than a wave, runs across probes, whole probes
    announce(f"{probes} probes x {rays} rays")
    w = scenegen.small_cascade(3, probes=probes, rays=rays)
    check_trace(S, w, False)

# Candidate cells of an analytic scene: lists of one, of up to 8 and up to 16 primitives,
# cells of more (equal primitives; many at one centre), which walk the clusters, rays that
# start and end beyond the outermost level, a plane of centres and one lone primitive.
@pytest.mark.parametrize("count,kind", [(1, "lone"), (60, "open"), (24, "equal"), (40, "shells"),
                                        (200, "flat"), (1024, "open")])
@pytest.mark.parametrize("t_max,spread", [(9.0, 1.0), (4000.0, 90.0)])
def test_analytic_candidate_cells(S, count, kind, t_max, spread):
    announce(f"candidates {count} {kind} t_max {t_max} spread {spread}")
    p = scenegen.open_scene_primitives(np.random.default_rng(count), count, (-4.0, 0.0, -4.0),
                                       (4.0, 2.0, 4.0), size_range=(0.1, 0.5))
    if kind == "equal":          # ties of every primitive: the lowest index is the nearest
        for f in (p.kind, p.center, p.half):
            f[:] = f[0]
    elif kind == "shells":       # 40 spheres about one centre, and as far from a far point
        p.kind[:] = 0
        p.center[:] = (0.5, 1.0, -0.25)
        p.half[:] = np.linspace(0.05, 0.6, count)[:, None]
    elif kind == "flat":
        p.center[:, 1] = 0.0
    params = Params(rays_per_probe=48, t_max=t_max, sky_rgb=(0.3, 0.2, 0.1))
    probes = ProbeGrid((4, 3, 4), (-1.7 * spread, 0.4, -1.6 * spread),
                       (1.1 * spread, 0.7 * spread, 1.05 * spread))
    w = Workload("candidates", p, [], probes, params, [])
    rec = []
    f = frame((0.3, 1.0, 0.2), seed=78)
    for cluster in (8, 5):
        ctx = S.context_from_workload(w, flags=S.SDFDDGI_FLAG_RECORD_RAYS, analytic=True,
                                      cluster_size=cluster)
        S.sdfddgi_update_frame(ctx, f.dir_to_light, f.radiance_rgb, f.rotation_seed)
        rec.append(S.sdfddgi_get_ray_records(ctx).cpu().numpy())
        S.sdfddgi_destroy(ctx)
    irr0, dep0 = (np.zeros(s, np.float32) for s in scenegen.atlas_shapes(w.num_probes, params))
    _, _, _, ref = oracle.Checker(w, analytic=True).update_probes(f, True, irr0, dep0,
                                                                  want_records=True)
    assert np.array_equal(rec[0], ref)
    assert np.array_equal(rec[1], ref)


# The blend's tilings: a few probes, ragged groups of 4 and 8 at either side of where the group
# changes, an odd number of 16-ray steps, rays that end within a chunk of 64, maps of one
# texel tile up to the largest of one pass and beyond it in either map.
@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("probes,rays,irr,depth", [
    ((2, 2, 2), 16, 8, 16), ((3, 3, 3), 48, 2, 3), ((2, 3, 341), 64, 8, 16), ((2, 3, 341), 80, 5, 9),
    ((32, 8, 8), 144, 8, 16), ((2, 5, 205), 272, 8, 16), ((2, 5, 205), 80, 11, 16),
    ((5, 3, 3), 96, 12, 16), ((3, 5, 3), 112, 8, 17), ((13, 3, 2), 208, 3, 24), ((2, 2, 3), 64, 32, 32)])
def test_blend_tilings(S, probes, rays, irr, depth, half):
    import torch
    announce(f"blend {probes} x {rays}, maps {irr} and {depth}, half={half}")
    params = Params(rays_per_probe=rays, irr_res=irr, depth_res=depth)
    none = Primitives(np.zeros(0, np.int32), np.zeros((0, 3)), np.zeros((0, 3)), np.zeros((0, 3)))
    w = Workload("blend", none, [random_level((4, 4, 4), (0.0,) * 3, 1.0, 1)],
                 ProbeGrid(probes, (0.5, 0.5, 0.5), (0.001, 0.01, 0.01)), params, [])
    irr0, dep0 = scenegen.random_atlas(w.num_probes, params, seed=15)
    pl = scenegen.random_payload(w.num_probes, rays, seed=16, t_max=params.t_max)
    ctx = S.context_from_workload(w, flags=S.SDFDDGI_FLAG_FP16 if half else 0)
    chk = oracle.Checker(w)
    cuda = [torch.from_numpy(x).to("cuda:0") for x in (irr0, dep0, pl)]
    check = np.unique(np.r_[0, w.num_probes - 1, np.random.default_rng(17).integers(
        0, w.num_probes, 24)])
    # binary32: sums of at most 272 products of one sign, (272 + 8) 2^-24 of the result;
    # precision form: a payload and two weight roundings of 2^-11 / 2^-9 of the largest value
    big = [np.pi * pl[..., :3].max(), np.array([pl[..., 3].max(), pl[..., 3].max() ** 2])]
    for reset in (True, False):
        S.sdfddgi_set_maps(ctx, cuda[0], cuda[1])
        if reset:
            S.sdfddgi_reset_history(ctx)
        S.sdfddgi_blend(ctx, cuda[2], 99 + reset)
        got = [m.cpu().numpy() for m in S.sdfddgi_get_maps(ctx)]
        for p in check:
            ref = chk.blend_probe(99 + reset, reset, pl[p], irr0[p], dep0[p])
            for g, r, top, ulp in zip(got, ref, big, (2.0 ** -11, 2.0 ** -9)):
                bound = 3 * ulp * top if half else 280 * 2.0 ** -24 * np.abs(r) + 1e-7 * np.mean(
                    np.abs(r))
                assert np.all(np.abs(g[p] - r) <= bound), (p, np.max(np.abs(g[p] - r) / bound))
    S.sdfddgi_destroy(ctx)


# A training step's samples over the workgroups (64 each, up to 256 of them, then strided),
# its sums, and the weights that Adam's step leaves in the packs.
@pytest.mark.parametrize("n", [1, 64, 65, 4000, 16385, 20000])
def test_training_parts(S, n):
    import torch
    announce(f"training on {n} samples")
    rng = np.random.default_rng(n)
    th = rng.normal(0, 0.1, oracle.MLP_PARAMS).astype(np.float32)
    x = rng.normal(0, 0.5, (n, 16)).astype(np.float32)
    tg = np.column_stack([rng.normal(0, 0.3, (n, 3)), rng.uniform(0.3, 2.0, n)]).astype(np.float32)
    xd, td = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(tg).to("cuda:0")
    make = lambda p: S.sdfddgi_trainer_create(p, head_weight=0.3, min_error=1e-4)
    tr = make(th)
    loss, g = S.sdfddgi_trainer_gradient(tr, xd, td)
    # the mean over parts is the mean of the parts' means, up to the sums' binary32 rounding:
    # 14 roundings deep, of partial sums no larger than the sum of the samples' magnitudes
    cut = [0, n // 3, n] if n > 2 else [0, n]
    parts = [(b - a, S.sdfddgi_trainer_gradient(tr, xd[a:b].contiguous(), td[a:b].contiguous()))
             for a, b in zip(cut, cut[1:])]
    ref = sum(k * p[1].astype(np.float64) for k, p in parts) / n
    # (each part's bfloat16 gradients are those of 1/n scaled: one more rounding of 2^-8)
    assert np.linalg.norm(g - ref) <= 2.0 ** -7 * np.linalg.norm(ref)
    assert abs(loss - sum(k * p[0] for k, p in parts) / n) <= 2e-6 * abs(loss)
    for seed in (3, 4):
        S.sdfddgi_trainer_step(tr, xd, td, n, seed, 1e-3)
    th2 = S.sdfddgi_trainer_get_params(tr)
    assert np.isfinite(th2).all() and not np.array_equal(th2, th)
    loss_a, g_a = S.sdfddgi_trainer_gradient(tr, xd, td)
    loss_b, g_b = S.sdfddgi_trainer_gradient(make(th2), xd, td)
    assert loss_a == loss_b and np.array_equal(g_a, g_b)


# Rows of the network alone: part of a tile, of a wave's four tiles, more than the grid, and
# arrays aligned to four bytes only.
@pytest.mark.parametrize("n", [1, 15, 64, 65, 300000])
@pytest.mark.parametrize("offset", [0, 1])
def test_infer_rows(S, n, offset):
    import torch
    announce(f"inference on {n} rows, offset {offset}")
    rng = np.random.default_rng(n)
    th = rng.normal(0, 0.1, oracle.MLP_PARAMS).astype(np.float32)
    x = rng.normal(0, 0.5, (n, 16)).astype(np.float32)
    den = S.sdfddgi_denoiser_create(th, 1.0, 1.0)
    flat = torch.zeros(16 * n + offset, device="cuda:0")
    xd = flat[offset:].view(n, 16)
    xd.copy_(torch.from_numpy(x))
    out = S.sdfddgi_denoiser_infer(den, xd).cpu().numpy()
    pick = np.unique(np.r_[0, n - 1, rng.integers(0, n, 40)])
    ref = oracle.mlp_forward(th.astype(np.float64), x[pick].astype(np.float64))
    # the same bfloat16 operands (an activation may round the other way): 2^-8 of the scale
    assert np.max(np.abs(out[pick] - ref)) <= 2.0 ** -8 * max(1.0, np.abs(ref).max())


# Frames with nothing but reads of the maps in between overlap as back-to-back ones do; what
# is read, and the next frames, must be those of a context that never overlaps (it keeps
# records). Plain, analytic and learned frames, and switches between them.
@pytest.mark.parametrize("form", ["plain", "fp16", "analytic", "learned"])
def test_map_reads_between_overlapping_frames(S, form):
    import torch
    from paper_2007_14394_amd import denoiser_weights
    announce(f"map reads between frames, {form}")
    w = scenegen.config2(2, probes=8192, frames=8, rays=64, grid=64)
    more = dict(analytic=dict(analytic=True), learned=dict(learned_rays=16, fallback_error=0.05))
    fl = S.SDFDDGI_FLAG_FP16 if form == "fp16" else 0
    ctxs = [S.context_from_workload(w, flags=fl, **more.get(form, {})),
            S.context_from_workload(w, flags=fl | S.SDFDDGI_FLAG_RECORD_RAYS, **more.get(form, {}))]
    net = denoiser_weights.load()
    den = S.sdfddgi_denoiser_create(net["params"], net["irr_scale"], net["depth_scale"])
    rng = np.random.default_rng(4)
    pts = torch.from_numpy(rng.uniform(-20, 20, (5000, 3)).astype(np.float32)).to("cuda:0")
    nrm = torch.from_numpy(rng.normal(size=(5000, 3)).astype(np.float32)).to("cuda:0")
    got = []
    for ctx in ctxs:
        reads = []
        for k, fr in enumerate(w.frames):
            args = (fr.dir_to_light, fr.radiance_rgb, fr.rotation_seed)
            if form == "learned" and k != 5:   # and one plain frame among the learned ones
                S.sdfddgi_update_frame_learned(ctx, den, *args)
            else:
                S.sdfddgi_update_frame(ctx, *args)
            if k != 3:
                reads += [m.clone() for m in S.sdfddgi_get_maps(ctx)]
            if k in (2, 3, 6):
                reads.append(S.sdfddgi_sample_irradiance(ctx, pts, nrm).clone())
            if k == 4:
                S.sdfddgi_reset_history(ctx)
                reads += [m.clone() for m in S.sdfddgi_get_maps(ctx)]
        got.append(reads)
        S.sdfddgi_destroy(ctx)
    assert len(got[0]) == len(got[1])
    for a, b in zip(*got):
        assert torch.equal(a, b)
