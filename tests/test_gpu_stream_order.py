"""Order of a context's work on its streams: calls of every kind between frames that
would otherwise overlap, against a context that never overlaps them."""
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


@pytest.fixture(scope="module")
def scene():
    return scenegen.config2(2, probes=8192, frames=20, rays=64, grid=64)


def denoiser(S):
    from paper_2007_14394_amd import denoiser_weights
    net = denoiser_weights.load()
    return S.sdfddgi_denoiser_create(net["params"], net["irr_scale"], net["depth_scale"])


FORMS = {"plain": {}, "fp16": {}, "analytic": dict(analytic=True),
         "learned": dict(learned_rays=16, fallback_error=0.05)}


def context(S, w, form, **kw):
    flags = (S.SDFDDGI_FLAG_FP16 if form == "fp16" else 0) | kw.pop("flags", 0)
    return S.context_from_workload(w, flags=flags, **FORMS[form], **kw)


# f: a frame; m: the maps read; b: Eq. 3 on a payload; e: training examples; r: relocation;
# h: histories rejected. Two frames and more after each call, so that the frames take every
# ray set and every side stream; for learned frames the calls come at both parities.
SEQUENCES = {"plain": "ffbfmfmfbffmfrfmfmfhfmbfmffm", "fp16": "ffbfmfmfbffmfrfmfmfhfmbfmffm",
             "analytic": "ffbfmfmfbffmfmfhfmbfmffm", "learned": "ffefmfmfmefmffmferfmfmfefmffm"}


@pytest.mark.parametrize("form", SEQUENCES)
def test_calls_between_overlapping_frames(S, scene, form):
    import torch
    announce(f"{form}: {SEQUENCES[form]}")
    w, den, got = scene, denoiser(S), []
    payload = torch.from_numpy(scenegen.random_payload(
        w.num_probes, 64, seed=3, t_max=w.params.t_max)).to("cuda:0")
    # work that keeps the caller's stream busy while the host goes on to the next calls
    busy = torch.rand(6144, 6144, device="cuda:0")
    for flags in (0, S.SDFDDGI_FLAG_RECORD_RAYS):   # (one that keeps records never overlaps)
        ctx = context(S, w, form, flags=flags)
        target = torch.zeros(ctx.irr_shape, device="cuda:0")
        reads, frame = [], 0
        for k, op in enumerate(SEQUENCES[form]):
            if op in "ber":
                torch.mm(busy, busy)
            fr = w.frames[frame % len(w.frames)]
            args = (fr.dir_to_light, fr.radiance_rgb, fr.rotation_seed)
            if op == "f":
                frame += 1
                if form == "learned":
                    S.sdfddgi_update_frame_learned(ctx, den, *args)
                else:
                    S.sdfddgi_update_frame(ctx, *args)
            elif op == "m":
                reads += [m.clone() for m in S.sdfddgi_get_maps(ctx)]
            elif op == "b":
                S.sdfddgi_blend(ctx, payload, 1000 + k)
            elif op == "e":
                reads += [t.clone() for t in S.sdfddgi_learned_examples(
                    ctx, den, fr.dir_to_light, fr.radiance_rgb, 1000 + k, target, 0.05)]
            elif op == "r":
                S.sdfddgi_relocate_probes(ctx, 0.6, 0.25, 8, 0.1 + 0.01 * k)
            else:
                S.sdfddgi_reset_history(ctx)
        torch.cuda.synchronize()
        got.append(reads)
        S.sdfddgi_destroy(ctx)
    assert len(got[0]) == len(got[1]) > 0
    for k, (a, b) in enumerate(zip(*got)):
        assert torch.equal(a, b), k


# Two frames and their maps read, captured once and replayed between frames that the caller
# runs directly (in pairs, as the graph reads and writes fixed map buffers).
@pytest.mark.parametrize("form", FORMS)
def test_frames_around_captured_ones(S, scene, form):
    import torch
    announce(f"{form}: captured frames")
    w, den, got = scene, denoiser(S), []
    busy = torch.rand(6144, 6144, device="cuda:0")
    for capture in (True, False):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            ctx = context(S, w, form, flags=0 if capture else S.SDFDDGI_FLAG_RECORD_RAYS)
            bufs = [(torch.zeros(ctx.irr_shape, device="cuda:0"),
                     torch.zeros(ctx.depth_shape, device="cuda:0")) for _ in range(2)]
            reads = []

            def frame(k):
                fr = w.frames[k]
                args = (fr.dir_to_light, fr.radiance_rgb, fr.rotation_seed)
                if form == "learned":
                    S.sdfddgi_update_frame_learned(ctx, den, *args)
                else:
                    S.sdfddgi_update_frame(ctx, *args)

            def pair():
                for k, (irr, dep) in enumerate(bufs):
                    frame(2 + k)
                    S.sdfddgi_get_maps(ctx, irr, dep)

            frame(0)
            frame(1)
            graph = torch.cuda.CUDAGraph()
            if capture:
                with torch.cuda.graph(graph, stream=stream):
                    pair()
            for k, op in enumerate("!ffmfmfm!mfmfmffm!!ffmfmfm!"):
                if op == "!":
                    torch.mm(busy, busy)   # the replay waits while the host goes on
                    if capture:
                        graph.replay()
                    else:
                        pair()
                    reads += [m.clone() for pair_of in bufs for m in pair_of]
                elif op == "f":
                    frame(4 + k % 16)
                else:
                    reads += [m.clone() for m in S.sdfddgi_get_maps(ctx)]
            torch.cuda.synchronize()
            got.append(reads)
            S.sdfddgi_destroy(ctx)
    assert len(got[0]) == len(got[1]) > 0
    for k, (a, b) in enumerate(zip(*got)):
        assert torch.equal(a, b), k


# Maps read into memory that no kernel of the device may write (here the host's) are copied
# as into the device's own.
@pytest.mark.parametrize("batch", [False, True])
def test_maps_read_into_other_memory(S, batch):
    import ctypes
    import torch
    announce(f"maps to the host, batch={batch}")
    lib = S.load_library()
    if batch:
        specs, seeds = scenegen.batch_scene_specs(1, 2, frames=1, sdf_range=(20, 24),
                                                  probes_xz=(2, 4), probes_y=(2, 3), rays=(64, 64))
        h = S.batch_from_specs(specs)
        S.sdfddgi_batch_update_frame(h, [(sp.frames[0].dir_to_light, sp.frames[0].radiance_rgb)
                                         for sp in specs], seeds[0])
        ref = [m.cpu().numpy() for m in S.sdfddgi_batch_get_maps(h, 1)]
        read = lambda irr, dep: lib.sdfddgi_batch_get_maps(h.handle, 1, irr, dep)
    else:
        w = scenegen.small_cascade(2, probes=(3, 5, 3), rays=64)
        h = S.context_from_workload(w)
        fr = w.frames[0]
        S.sdfddgi_update_frame(h, fr.dir_to_light, fr.radiance_rgb, fr.rotation_seed)
        ref = [m.cpu().numpy() for m in S.sdfddgi_get_maps(h)]
        read = lambda irr, dep: lib.sdfddgi_get_maps(h.handle, irr, dep)
    for which in ((0, 1), (0,), (1,)):
        host = [np.full(m.size + 2, -1.0, np.float32) for m in ref]
        ptr = [ctypes.c_void_p(m.ctypes.data + 4) if k in which else None
               for k, m in enumerate(host)]
        assert read(*ptr) == S.SDFDDGI_OK
        torch.cuda.synchronize()
        for k, (m, r) in enumerate(zip(host, ref)):
            assert np.array_equal(m[1:-1], r.ravel()) if k in which else (m == -1.0).all()
            assert m[0] == m[-1] == -1.0
        # one to the host, one to the device
        mixed = torch.full(ref[1].shape, -1.0, device="cuda:0")
        assert read(ptr[0], ctypes.c_void_p(mixed.data_ptr())) == S.SDFDDGI_OK
        torch.cuda.synchronize()
        assert np.array_equal(mixed.cpu().numpy(), ref[1])
