"""The device baker and the map read-back at the sizes where their tilings can go
wrong: grids thinner and longer than a brick, ragged bricks, primitive counts around
the staging chunk, equal and non-finite primitives; maps whose float counts are not
multiples of four."""
import sys

import numpy as np
import pytest

import scenegen

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
