"""Grids that the trace's 24-bit products and 32-bit offsets do not cover: far along an axis
of more than 65536 vertices, and past 4 GiB of bricks. The single-scene trace and relocation
against the oracle, the batched form against single-scene contexts."""
import sys

import numpy as np
import pytest

import oracle
from scenegen import Params, ProbeGrid
from tests.helpers import fp16_grid, frame
from tests.test_gpu_kernel_edges import check_trace, random_level, trace_workload

pytestmark = pytest.mark.gpu

SPACING, ORIGIN = 0.25, (-1.0, 0.5, -2.0)


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


def spread_probes(n, probes=(3, 2, 3)):
    """Probes from one end of a grid to the other."""
    ext = [SPACING * (k - 1) for k in n]
    return ProbeGrid(probes, tuple(o + 0.03 * e for o, e in zip(ORIGIN, ext)),
                     tuple(0.94 * e / (p - 1) for e, p in zip(ext, probes)))


LONG = [(66001, 3, 2), (2, 66001, 3), (3, 2, 66001)]


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("n", LONG)
def test_trace_far_along_a_grid(S, n, half):
    announce(f"trace along {n}, half={half}")
    w = trace_workload([random_level(n, ORIGIN, SPACING, sum(n))], spread_probes(n), 48)
    rec = check_trace(S, w, half)
    assert len(np.unique(rec[..., 0] & 255)) > 1


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("n", LONG)
def test_relocation_far_along_a_grid(S, n, half):
    announce(f"relocation along {n}, half={half}")
    w = trace_workload([random_level(n, ORIGIN, SPACING, sum(n))], spread_probes(n, (8, 4, 8)), 16)
    ck = oracle.Checker(fp16_grid(w) if half else w)
    ctx = S.context_from_workload(w, flags=S.SDFDDGI_FLAG_FP16 if half else 0)
    S.sdfddgi_relocate_probes(ctx, 0.2, 0.02, 4, 0.01)
    got = S.sdfddgi_get_probe_positions(ctx).cpu().numpy()
    S.sdfddgi_destroy(ctx)
    pos, _ = ck.relocate_probes(ck.grid_positions(), 0.2, 0.02, 4, 0.01)
    assert np.array_equal(got.view(np.int32), pos.view(np.int32))
    assert np.any(got != ck.grid_positions())


# One scene that needs them moves all of a batch's scenes onto the kernels with general
# products and offsets (of the last: two scenes of 2.3 GiB of bricks, and one past both).
@pytest.mark.parametrize("n,copies", [(n, 1) for n in LONG] + [((800, 800, 800), 2)])
def test_batch_with_a_large_grid(S, n, copies):
    import torch
    announce(f"batch with a grid of {n}")
    params = S.params_from(Params(rays_per_probe=64, t_max=30.0, max_steps=24, hit_eps=5e-3))
    scenes = []
    for size, seed in ((n, 1), ((13, 6, 10), 2)):
        if np.prod(size, dtype=np.int64) < 1 << 24:
            sdf = torch.from_numpy(random_level(size, ORIGIN, SPACING, seed).sdf).to("cuda:0")
        else:
            sdf = torch.rand(size[::-1], device="cuda:0", generator=torch.Generator(
                "cuda:0").manual_seed(seed)).mul_(0.3).add_(0.02)
            sdf[::3, ::5, ::7] = -0.5
        pg = spread_probes(size)
        scenes += [dict(sdf=sdf, origin=ORIGIN, spacing=SPACING, probe_n=pg.n, params=params,
                        probe_origin=pg.origin, probe_spacing=pg.spacing)] * (copies if size == n
                                                                              else 1)
    frames = [frame((0.3, 1.0, 0.2), seed=5), frame((-0.2, 0.8, 0.4), seed=6)]
    b = S.sdfddgi_batch_create(scenes)
    for fr in frames:
        S.sdfddgi_batch_update_frame(b, [(fr.dir_to_light, fr.radiance_rgb)] * len(scenes),
                                     fr.rotation_seed)
    got = [[m.cpu().numpy() for m in S.sdfddgi_batch_get_maps(b, s)] for s in range(len(scenes))]
    S.sdfddgi_batch_destroy(b)
    for sc, maps in zip(scenes, got):
        single = S.params_from(Params(rays_per_probe=64, t_max=30.0, max_steps=24, hit_eps=5e-3),
                               S.SDFDDGI_FLAG_FP16)
        ctx = S.sdfddgi_create([sc], sc["probe_n"], sc["probe_origin"], sc["probe_spacing"], single)
        for fr in frames:
            S.sdfddgi_update_frame(ctx, fr.dir_to_light, fr.radiance_rgb, fr.rotation_seed)
        for got_map, ref in zip(maps, S.sdfddgi_get_maps(ctx)):
            ref = ref.cpu().numpy()
            assert ref.any() and np.array_equal(got_map.view(np.int32), ref.view(np.int32))
        S.sdfddgi_destroy(ctx)
