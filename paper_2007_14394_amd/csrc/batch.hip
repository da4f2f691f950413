// gfx950 kernels of the batched form: many scenes of uneven size updated by one
// set of launches per frame (captured once in a graph and replayed).
//
//   batch_begin_kernel    zero the counters, stamp the frame start on the device clock
//   batch_primary_kernel  primary sphere trace of every scene's rays, one persistent
//                         wave-compacted grid over the concatenated ray space
//   batch_hits_kernel     first half of every scene's hit shading (normal, shadow ray, albedo)
//   batch_shade_kernel    second half (multi-bounce lookup, payload)
//   batch_blend_kernel    the precision-form blend of every scene's probes, one
//                         workgroup per 16 probes of a scene; stamps each scene's end
//
// Each ray runs the same binary32 sequence as the single-scene kernels with the
// scene's binary16 grid (one level: the grid box is the whole domain), so a scene's
// rays, payload and maps are bit-identical to a single-scene context in the
// precision form. A lane's scene comes from the ray's slot (binary search over the
// scenes' first slots) or from the hit-queue entry; the fields the sample loop needs
// are copied to registers when the lane takes the ray. The chunk sizes, refill
// threshold and grid sizes are chosen by the runtime's autotuner.
#include <algorithm>

#include "internal.h"
#include "octahedral.h"
#include "trace_common.h"
#include "blend_common.h"

#pragma clang fp contract(off)

namespace sdfddgi {

// The fields of a lane's scene that every sample reads.
struct LaneScene {
    LevelCells lv;
    float xlo0, xlo1, xlo2, xhi0, xhi1, xhi2;
    float eps, t_max, relax;
    int max_steps;
};

__device__ __forceinline__ LaneScene lane_scene(const BatchScene &s) {
    LaneScene d;
    d.lv = s.lv;
    d.xlo0 = s.xlo0; d.xlo1 = s.xlo1; d.xlo2 = s.xlo2;
    d.xhi0 = s.xhi0; d.xhi1 = s.xhi1; d.xhi2 = s.xhi2;
    d.eps = s.eps; d.t_max = s.t_max; d.relax = s.relax; d.max_steps = s.max_steps;
    return d;
}

// One sample of the fixed sphere-trace sequence for the lanes of `live` (as trace_step of
// the single-scene kernels with one level: a point inside the grid box is level 0, else
// the ray escapes); returns those whose ray goes on.
template <bool kWide>
__device__ __forceinline__ uint64_t batch_step(GlobalBytes cells, const LaneScene &d, uint64_t live,
                                               float o0, float o1, float o2, float w0, float w1,
                                               float w2, float &t, int &k, float &dist, int &level) {
    const float x0 = fmaf(t, w0, o0), x1 = fmaf(t, w1, o1), x2 = fmaf(t, w2, o2);
    const bool box = (x0 >= d.xlo0) & (x0 <= d.xhi0) & (x1 >= d.xlo1) & (x1 <= d.xhi1) &
                     (x2 >= d.xlo2) & (x2 <= d.xhi2);
    const uint64_t inside = live & __ballot(box) & ~__ballot(t > d.t_max);
    level = in_mask(live) ? (box ? 0 : -1) : level;
    if (in_mask(inside)) dist = distance_inside<true, kWide>(cells, d.lv, x0, x1, x2);
    const uint64_t go = inside & ~__ballot(dist < d.eps) & ~__ballot(k + 1 == d.max_steps);
    if (in_mask(go)) {
        t = fmaf(d.relax, dist, t);
        ++k;
    }
    return go;
}

__device__ __forceinline__ void load_scenes(const BatchArgs &a, BatchScene *s_sc, int *s_base) {
    for (int e = threadIdx.x; e < a.nscenes; e += blockDim.x) {
        s_sc[e] = a.scenes[e];
        s_base[e] = a.scenes[e].ray_base;
    }
    __syncthreads();
}

// Scene of a ray slot: the last scene whose first slot is <= slot.
__device__ __forceinline__ int scene_of(const int *s_base, int n, int slot) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_base[mid] <= slot) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__global__ __launch_bounds__(64) void batch_begin_kernel(int *counter,
                                                         unsigned long long *stamps, int n) {
    // stamps[0]: frame start; stamps[1 + s]: end of scene s's blend
    for (int e = threadIdx.x; e <= n; e += blockDim.x) stamps[e] = 0ull;
    for (int e = threadIdx.x; e < kBatchCounters; e += blockDim.x) counter[e] = 0;
    __syncthreads();
    if (threadIdx.x == 0) stamps[0] = wall_clock64();
}

__device__ __forceinline__ void batch_flush(const BatchArgs &a, int4 *buf, int count) {
    if (count == 0) return;
    int base = 0;
    if (__lane_id() == 0) base = atomicAdd(a.counter + 2, count);
    base = __builtin_amdgcn_readfirstlane(base);
    const int lane = (int)__lane_id();
    if (lane < count) a.hitq[base + lane] = buf[lane];
    __builtin_amdgcn_wave_barrier();
}

// Primary trace over the concatenated rays of all scenes (see primary_kernel).
template <bool kWide>
__global__ __launch_bounds__(256) void batch_primary_kernel(BatchArgs a, int chunk) {
    constexpr int kQueue = 128;
    __shared__ BatchScene s_sc[kMaxBatchScenes];
    __shared__ int s_base[kMaxBatchScenes];
    __shared__ int4 s_hits[4][64];
    __shared__ WaitingRay s_rays[4][kQueue];   // origin and scene, direction and ray
    load_scenes(a, s_sc, s_base);
    const GlobalBytes cells = (GlobalBytes)a.cells;
    const int lane = (int)__lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    // blocks of the concatenated rays dealt to the XCDs in turn (see BlockFeeder)
    BlockFeeder feed(chunk, kBatchBlockRays / chunk);
    uint64_t live = 0, ended = 0;
    int staged = 0, head = 0, waiting = 0, stage = 0, coming = 0;
    int ray = 0, k = 0, sc = 0, level = 0, n_ray = 0, n_probe = 0, n_sc = 0;
    float o0 = 0, o1 = 0, o2 = 0, w0 = 0, w1 = 0, w2 = 0, t = 0, dist = 0;
    float m0 = 0, m1 = 0, m2 = 0, v0 = 0, v1 = 0, v2 = 0;
    LaneScene d{};
    while (true) {
        if (stage == 2) {
            if (lane < coming) {
                WaitingRay &r = s_rays[wave][(head + waiting + lane) & (kQueue - 1)];
                r.from = make_float4(m0, m1, m2, __int_as_float(n_sc));
                r.dir = make_float4(v0, v1, v2, __int_as_float(n_ray));
            }
            __builtin_amdgcn_wave_barrier();
            waiting += coming;
            stage = 0;
        } else if (stage == 1) {
            if (lane < coming) {
                const BatchScene &s = s_sc[n_sc];
                n_ray += s.ray_base + n_probe * s.R;
                const int gp = s.probe_base + n_probe;
                m0 = a.probe_pos[3 * gp]; m1 = a.probe_pos[3 * gp + 1]; m2 = a.probe_pos[3 * gp + 2];
            }
            stage = 2;
        }
        if (__popcll(live) < a.refill) {
            if (ended) {
                bool hit = false;
                int4 entry = make_int4(0, 0, 0, 0);
                if (in_mask(ended)) {
                    const bool over = t > d.t_max, out = over || level < 0;
                    const bool inside = !out && k == 0 && dist < 0.0f;
                    if (out || inside) {
                        const BatchScene &s = s_sc[sc];
                        store_streamed(&a.payload[ray], inside ? make_float4(0.0f, 0.0f, 0.0f, 0.0f)
                                                : make_float4(s.sky0, s.sky1, s.sky2, s.t_max));
                    } else {
                        hit = true;
                        entry = make_int4(ray, __float_as_int(t),
                                          pack_hit(dist < d.eps ? kHit : kHitExhausted, 0, k + 1),
                                          sc);
                    }
                }
                ended = 0;
                const uint64_t hm = __ballot(hit);
                if (hm) {
                    const int n = __popcll(hm);
                    if (staged + n > 64) {
                        batch_flush(a, s_hits[wave], staged);
                        staged = 0;
                    }
                    if (hit) s_hits[wave][staged + __popcll(hm & below)] = entry;
                    __builtin_amdgcn_wave_barrier();
                    staged += n;
                }
            }
            if (waiting > 0) {
                const int rank = __popcll(~live & below);
                const uint64_t take = __ballot(in_mask(~live) && rank < waiting);
                if (in_mask(take)) {
                    const WaitingRay r = s_rays[wave][(head + rank) & (kQueue - 1)];
                    o0 = r.from.x; o1 = r.from.y; o2 = r.from.z;
                    w0 = r.dir.x; w1 = r.dir.y; w2 = r.dir.z;
                    sc = __float_as_int(r.from.w);
                    ray = __float_as_int(r.dir.w);
                    d = lane_scene(s_sc[sc]);
                    t = 0.0f;
                    k = 0;
                }
                __builtin_amdgcn_wave_barrier();
                live |= take;
                const int n = __popcll(take);
                head += n;
                waiting -= n;
            }
            if (stage == 0 && !feed.exhausted && waiting <= kQueue - 64 - 16) {
                coming = 0;
                while (coming < 64 && !feed.exhausted) {
                    int first = 0;
                    const int n = feed.claim(a.counter + kPartStride, a.total_rays, 64 - coming,
                                             first);
                    if (lane >= coming && lane < coming + n) {
                        const int slot = first + lane - coming;
                        n_sc = scene_of(s_base, a.nscenes, slot);
                        const BatchScene &s = s_sc[n_sc];
                        const int local = slot - s.ray_base;
                        const int q = local / s.R;
                        n_ray = local - q * s.R;
                        n_probe = a.probe_order[s.probe_base + q];
                        const int di = s.dir_base + n_ray;
                        v0 = a.dirs[3 * di]; v1 = a.dirs[3 * di + 1]; v2 = a.dirs[3 * di + 2];
                    }
                    coming += n;
                }
                stage = coming ? 1 : 0;
            }
            if (!live) {
                if (stage == 0 && feed.exhausted) {
                    batch_flush(a, s_hits[wave], staged);
                    break;
                }
                continue;
            }
        }
        const uint64_t go = batch_step<kWide>(cells, d, live, o0, o1, o2, w0, w1, w2, t, k, dist,
                                              level);
        ended |= live & ~go;
        live = go;
    }
}

__device__ __forceinline__ float3 batch_albedo(const BatchScene &s, float x0, float x1, float x2) {
    const LevelLds &d = s.lv;
    if (!d.alb) return make_float3(s.alb0, s.alb1, s.alb2);
    int i0, i1, i2;
    float f0, f1, f2;
    cell_of((x0 - d.org0) * d.inv, (float)d.cmax0, i0, f0);
    cell_of((x1 - d.org1) * d.inv, (float)d.cmax1, i1, f1);
    cell_of((x2 - d.org2) * d.inv, (float)d.cmax2, i2, f2);
    const uint32_t sy = d.arow, sz = d.aslice;
    const float *p = d.alb + 3u * ((uint32_t)i2 * sz + (uint32_t)i1 * sy + (uint32_t)i0);
    float out[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float v000 = p[c], v100 = p[3 + c], v010 = p[3 * sy + c], v110 = p[3 * (sy + 1) + c];
        const float v001 = p[3 * sz + c], v101 = p[3 * (sz + 1) + c];
        const float v011 = p[3 * (sz + sy) + c], v111 = p[3 * (sz + sy + 1) + c];
        const float c00 = fmaf(f0, v100 - v000, v000), c10 = fmaf(f0, v110 - v010, v010);
        const float c01 = fmaf(f0, v101 - v001, v001), c11 = fmaf(f0, v111 - v011, v011);
        const float c0 = fmaf(f1, c10 - c00, c00), c1 = fmaf(f1, c11 - c01, c01);
        out[c] = fmaf(f2, c1 - c0, c0);
    }
    return make_float3(out[0], out[1], out[2]);
}

// First half of hit shading for every scene's queued hits (see hits_kernel).
template <bool kWide>
__global__ __launch_bounds__(256) void batch_hits_kernel(BatchArgs a, int chunk) {
    constexpr int kQueue = 128;
    __shared__ BatchScene s_sc[kMaxBatchScenes];
    __shared__ int s_base[kMaxBatchScenes];
    __shared__ float4 s_rays[4][kQueue];   // shadow ray origins, hit-queue indices
    __shared__ int s_ray_sc[4][kQueue];    // their scenes
    load_scenes(a, s_sc, s_base);
    const GlobalBytes cells = (GlobalBytes)a.cells;
    const int lane = (int)__lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const int total = __builtin_amdgcn_readfirstlane(a.counter[2]);
    Feeder feed(chunk);
    uint64_t live = 0, ended = 0;
    int head = 0, waiting = 0, stage = 0, coming = 0;
    int qi = 0, k = 0, level = 0, n_qi = 0;
    float o0 = 0, o1 = 0, o2 = 0, t = 0, dist = 0, l0 = 0, l1 = 0, l2 = 0;
    int4 e = make_int4(0, 0, 0, 0);
    float p0 = 0, p1 = 0, p2 = 0, w0 = 0, w1 = 0, w2 = 0;
    LaneScene d{};
    while (true) {
        if (stage == 2) {
            bool lit = false;
            float4 from = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (lane < coming) {
                const BatchScene &s = s_sc[e.w];
                const float *lt = a.lights + 6 * e.w;
                const float ht = __int_as_float(e.y);
                const float x0 = fmaf(ht, w0, p0), x1 = fmaf(ht, w1, p1), x2 = fmaf(ht, w2, p2);
                const float3 alb = batch_albedo(s, x0, x1, x2);
                float n0, n1, n2;
                hit_normal<true>(cells, s.lv, kWide, x0, x1, x2, w0, w1, w2, n0, n1, n2);
                const float ndl = fmaf(n2, lt[2], fmaf(n1, lt[1], n0 * lt[0]));
                lit = ndl > 0.0f;
                const int64_t at = 2 * (int64_t)n_qi;
                a.geo[at] = make_float4(n0, n1, n2, lit ? ndl : 0.0f);
                a.geo[at + 1] = make_float4(alb.x, alb.y, alb.z, 0.0f);
                from = make_float4(fmaf(n0, s.bias, x0), fmaf(n1, s.bias, x1),
                                   fmaf(n2, s.bias, x2), __int_as_float(n_qi));
            }
            const uint64_t m = __ballot(lit);
            if (lit) {
                const int at = (head + waiting + __popcll(m & below)) & (kQueue - 1);
                s_rays[wave][at] = from;
                s_ray_sc[wave][at] = e.w;
            }
            order_wave_stores();   // the records; a lane of a blocked ray changes another's
            waiting += __popcll(m);
            stage = 0;
        } else if (stage == 1) {
            if (lane < coming) {
                const BatchScene &s = s_sc[e.w];
                const int local = e.x - s.ray_base;
                const int p = local / s.R, i = local - p * s.R;
                const int gp = s.probe_base + p, di = s.dir_base + i;
                p0 = a.probe_pos[3 * gp]; p1 = a.probe_pos[3 * gp + 1]; p2 = a.probe_pos[3 * gp + 2];
                w0 = a.dirs[3 * di]; w1 = a.dirs[3 * di + 1]; w2 = a.dirs[3 * di + 2];
            }
            stage = 2;
        }
        if (__popcll(live) < a.refill) {
            if (ended) {
                // stopped inside the grid before t_max: at a hit or out of steps
                if (in_mask(ended) && !(t > d.t_max) && level >= 0)
                    a.geo[2 * (int64_t)qi].w = 0.0f;
                ended = 0;
            }
            if (waiting > 0) {
                const int rank = __popcll(~live & below);
                const uint64_t take = __ballot(in_mask(~live) && rank < waiting);
                if (in_mask(take)) {
                    const int at = (head + rank) & (kQueue - 1);
                    const float4 r = s_rays[wave][at];
                    const int sc = s_ray_sc[wave][at];
                    o0 = r.x; o1 = r.y; o2 = r.z;
                    qi = __float_as_int(r.w);
                    const float *lt = a.lights + 6 * sc;
                    l0 = lt[0]; l1 = lt[1]; l2 = lt[2];
                    d = lane_scene(s_sc[sc]);
                    t = 0.0f;
                    k = 0;
                }
                __builtin_amdgcn_wave_barrier();
                live |= take;
                const int n = __popcll(take);
                head += n;
                waiting -= n;
            }
            if (stage == 0 && !feed.exhausted && waiting <= kQueue - 64 - 16) {
                coming = 0;
                while (coming < 64 && !feed.exhausted) {
                    int first = 0;
                    const int n = feed.claim(a.counter + 1, total, 64 - coming, first);
                    if (lane >= coming && lane < coming + n) {
                        n_qi = first + lane - coming;
                        e = a.hitq[n_qi];
                    }
                    coming += n;
                }
                stage = coming ? 1 : 0;
            }
            if (!live) {
                if (stage == 0 && feed.exhausted && waiting == 0) break;
                continue;
            }
        }
        const uint64_t go = batch_step<kWide>(cells, d, live, o0, o1, o2, l0, l1, l2, t, k, dist,
                                              level);
        ended |= live & ~go;
        live = go;
    }
}

// Second half of hit shading: the multi-bounce lookup and the payload of every scene's
// queued hits (see shade_kernel).
__global__ __launch_bounds__(256) void batch_shade_kernel(BatchArgs a) {
    __shared__ BatchScene s_sc[kMaxBatchScenes];
    __shared__ int s_base[kMaxBatchScenes];
    load_scenes(a, s_sc, s_base);
    const int total = a.counter[2];
    const int tile = 10 * 10 * 3;   // 8x8 irradiance tile with its border
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < total; q += gridDim.x * blockDim.x) {
        const int4 e = a.hitq[q];
        const float4 g0 = a.geo[2 * (int64_t)q], g1 = a.geo[2 * (int64_t)q + 1];
        const BatchScene &s = s_sc[e.w];
        const float *lt = a.lights + 6 * e.w;
        const float ht = __int_as_float(e.y);
        float3 ind = make_float3(0.0f, 0.0f, 0.0f);
        if (s.gain != 0.0f) {
            const int local = e.x - s.ray_base;
            const int p = local / s.R, i = local - p * s.R;
            const int gp = s.probe_base + p, di = s.dir_base + i;
            const float x0 = fmaf(ht, a.dirs[3 * di], a.probe_pos[3 * gp]);
            const float x1 = fmaf(ht, a.dirs[3 * di + 1], a.probe_pos[3 * gp + 1]);
            const float x2 = fmaf(ht, a.dirs[3 * di + 2], a.probe_pos[3 * gp + 2]);
            ind = interp_irradiance(a.prev_irr + (size_t)s.probe_base * tile, 8, s.pg, x0, x1, x2,
                                    g0.x, g0.y, g0.z);
        }
        const float inv_pi = 0.318309886183790671538f;
        float4 out;
        out.x = g1.x * inv_pi * (lt[3] * g0.w + s.gain * ind.x);
        out.y = g1.y * inv_pi * (lt[4] * g0.w + s.gain * ind.y);
        out.z = g1.z * inv_pi * (lt[5] * g0.w + s.gain * ind.z);
        out.w = ht;
        store_streamed(&a.payload[e.x], out);
    }
}

// One workgroup per kP probes of one scene (16 / kP workgroups per entry of the
// 16-probe block table): that scene's blend arguments, the shared precision-form
// blend body with the tile (kP, kChunk), then the scene's end stamp.
template <int kP, int kChunk>
__global__ __launch_bounds__(256, 4) void batch_blend_kernel(BatchBlendArgs b) {
    constexpr int kSub = kBlendProbes / kP;
    const int2 blk = b.blocks[blockIdx.x / kSub];
    const int pb = blk.y + (int)(blockIdx.x % kSub) * kP;
    const BatchScene &s = b.scenes[blk.x];
    const size_t ti = (size_t)s.probe_base * 10 * 10 * 3, td = (size_t)s.probe_base * 18 * 18 * 2;
    BlendArgs a{};
    a.P = s.P;
    a.R = s.R;
    a.irr_res = 8;
    a.depth_res = 16;
    a.hysteresis = s.hysteresis;
    a.payload = b.payload + s.ray_base;
    a.Rpad = s.R;
    a.w16_i = s.w16_i;
    a.w16_d = s.w16_d;
    a.norm_i = s.norm_i;
    a.norm_d = s.norm_d;
    a.prev_irr = b.prev_irr + ti;
    a.prev_depth = b.prev_depth + td;
    a.new_irr = b.new_irr + ti;
    a.new_depth = b.new_depth + td;
    a.reject = b.reject + s.probe_base;
    blend16_block<kStdMaps, kP, kChunk>(a, pb);
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        atomicMax(b.done + blk.x, (unsigned long long)wall_clock64());
    }
}

// ---------------------------------------------------------------- launchers --

bool batch_chunk_supported(int chunk, bool hits) {
    if (hits) return chunk == 16 || chunk == 32 || chunk == 64 || chunk == 128;
    return chunk == 64 || chunk == 128 || chunk == 256 || chunk == 512;
}

static int device_cus(int device) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess ||
        cus < 1)
        cus = 256;
    return cus;
}

int batch_max_blocks(int device, bool hits) { return (hits ? 4 : 8) * device_cus(device); }

int batch_resident_blocks(int device, bool hits) {
    int per_cu = 0;
    const void *k = hits ? (const void *)batch_hits_kernel<false>
                         : (const void *)batch_primary_kernel<false>;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, 256, 0) != hipSuccess || per_cu < 1)
        per_cu = 1;
    return std::min(per_cu * device_cus(device), batch_max_blocks(device, hits));
}

hipError_t launch_batch_begin(int *counter, unsigned long long *stamps, int n, hipStream_t s) {
    hipLaunchKernelGGL(batch_begin_kernel, dim3(1), dim3(64), 0, s, counter, stamps, n);
    return hipGetLastError();
}

hipError_t launch_batch_primary(const BatchArgs &a, const BatchTuning &t, hipStream_t s) {
    if (a.wide)
        hipLaunchKernelGGL(batch_primary_kernel<true>, dim3(t.primary_blocks), dim3(256), 0, s, a,
                           t.primary_chunk);
    else
        hipLaunchKernelGGL(batch_primary_kernel<false>, dim3(t.primary_blocks), dim3(256), 0, s, a,
                           t.primary_chunk);
    return hipGetLastError();
}

hipError_t launch_batch_hits(const BatchArgs &a, const BatchTuning &t, hipStream_t s) {
    if (a.wide)
        hipLaunchKernelGGL(batch_hits_kernel<true>, dim3(t.hits_blocks), dim3(256), 0, s, a,
                           t.hits_chunk);
    else
        hipLaunchKernelGGL(batch_hits_kernel<false>, dim3(t.hits_blocks), dim3(256), 0, s, a,
                           t.hits_chunk);
    return hipGetLastError();
}

hipError_t launch_batch_shade(const BatchArgs &a, hipStream_t s) {
    // four workgroups per CU of the 256-CU part, striding over the queue
    const int64_t blocks = ((int64_t)a.total_rays + 255) / 256;
    hipLaunchKernelGGL(batch_shade_kernel, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(256),
                       0, s, a);
    return hipGetLastError();
}

template <int kP, int kChunk>
static hipError_t launch_blend_tile(const BatchBlendArgs &a, int nblocks16, hipStream_t s) {
    hipLaunchKernelGGL(HIP_KERNEL_NAME(batch_blend_kernel<kP, kChunk>),
                       dim3(nblocks16 * (kBlendProbes / kP)), dim3(256), 0, s, a);
    return hipGetLastError();
}

bool batch_blend_tile_supported(int probes, int chunk) {
    return (probes == 16 || probes == 8) && (chunk == 32 || chunk == 64 || chunk == 128);
}

hipError_t launch_batch_blend(const BatchBlendArgs &a, int nblocks16, const BatchTuning &t,
                              hipStream_t s) {
    if (nblocks16 <= 0) return hipSuccess;
    const int key = t.blend_probes * 1000 + t.blend_chunk;
    switch (key) {
        case 16032: return launch_blend_tile<16, 32>(a, nblocks16, s);
        case 16064: return launch_blend_tile<16, 64>(a, nblocks16, s);
        case 16128: return launch_blend_tile<16, 128>(a, nblocks16, s);
        case 8032: return launch_blend_tile<8, 32>(a, nblocks16, s);
        case 8064: return launch_blend_tile<8, 64>(a, nblocks16, s);
        case 8128: return launch_blend_tile<8, 128>(a, nblocks16, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sdfddgi
