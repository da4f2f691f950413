// gfx950 kernels of the SDFDDGI per-frame probe update (paper Sec. 3.3).
//
//   tables_kernel   frame ray directions (binary64 rotation of the fixed
//                   spherical-Fibonacci set, rounded once) and the Eq. 3 texel-by-
//                   ray weight matrices w_ti = max(0, n_t . w_i) and w_ti^s with
//                   their reciprocal row sums
//   primary_kernel  per ray: primary sphere trace; payload of misses, hit records
//   hits_kernel     per hit: normal, SDF shadow ray, albedo
//   shade_kernel    per hit: multi-bounce lookup into the previous atlas, payload (R,G,B,t)
//   blend_kernel    per probe: Eq. 3 ratio estimate for every texel, depth
//                   moments, temporal mix, octahedral border
//   sample_kernel   probe interpolation at arbitrary points and normals
//
// The geometric part of the trace (everything that decides an integer) follows
// one fixed binary32 operation sequence, spelled out with fmaf; contraction of
// any other multiply-add is disabled for this file.
#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "octahedral.h"
#include "trace_common.h"
#include "blend_common.h"
#include "analytic_common.h"

#pragma clang fp contract(off)

namespace sdfddgi {

// ------------------------------------------------------------- geometry -----

__device__ __forceinline__ void load_levels(const TraceArgs &a, LevelLds *s_lv) {
    if (threadIdx.x < kMaxLevels && (int)threadIdx.x < a.nl) {
        const DevLevel &d = a.lv[threadIdx.x];
        LevelLds v;
        v.line0 = d.line0; v.nb0 = d.nb0; v.nb1 = d.nb1; v.alb = d.alb;
        v.org0 = d.org0; v.org1 = d.org1; v.org2 = d.org2; v.inv = d.inv;
        v.cmax0 = d.n0 - 2; v.cmax1 = d.n1 - 2; v.cmax2 = d.n2 - 2;
        v.half = d.half;
        v.arow = (uint32_t)d.n0; v.aslice = (uint32_t)d.n0 * (uint32_t)d.n1;
        s_lv[threadIdx.x] = v;
    }
    __syncthreads();
}

// Finest level whose box, shrunk by one voxel (the coarsest level: its full box),
// holds x; -1 outside the coarsest box. The test "grid coordinate within [lo, hi]"
// is made on x itself against per-level bounds: u = (x - org) * inv is monotone in x,
// so the host finds the exact binary32 thresholds once and the result is the same.
// Nested levels (`nested`, the usual cascade): no lane of the wave in a level's box, none
// in the finer ones'.
__device__ __forceinline__ int select_level(const TraceArgs &a, float x0, float x1, float x2) {
    int L = -1;
#pragma unroll
    for (int l = kMaxLevels - 1; l >= 0; --l) {
        const DevLevel &d = a.lv[l];   // absent levels hold no point (an empty box)
        const bool in = (x0 >= d.xlo0) & (x0 <= d.xhi0) & (x1 >= d.xlo1) & (x1 <= d.xhi1) &
                        (x2 >= d.xlo2) & (x2 <= d.xhi2);
        const uint64_t any = __ballot(in);
        L = in ? l : L;
        if (l > 0 && l < kMaxLevels - 1 && !any && a.nested >= l) break;
    }
    return L;
}

// Distance backends of the trace kernels: the cascade of grids with binary32 or
// binary16 values, or the scene's analytic primitives (Sec. 3.1) through their candidate
// cells, which answer the cluster-culled query of Sec. 3.3. The per-workgroup LDS state of
// each:
enum : int { kSdfGrid32 = 0, kSdfGrid16 = 1, kSdfAnalytic = 2 };
template <int kSdf> struct SdfLds { LevelLds lv[kMaxLevels]; };
template <> struct SdfLds<kSdfAnalytic> { float4 lv[kMaxCellLevels]; };  // and lds_prims()

template <int kSdf>
__device__ __forceinline__ void load_sdf(const TraceArgs &a, SdfLds<kSdf> &s) {
    if constexpr (kSdf == kSdfAnalytic) load_prims(a.an, s.lv);
    else load_levels(a, s.lv);
}

// Kernel arguments that only rare branches of a trace loop need, read where they are
// used: hoisted out of the loop like other uniform values they would take the scalar
// registers that every sample's level bounds need. The struct has to be the only argument
// of the calling kernel, whose type `Kernel` is: it then starts the argument segment.
typedef const __attribute__((address_space(4))) TraceArgs RareArgs;
template <typename Kernel>
__device__ __forceinline__ RareArgs *rare_args() {
    static_assert(std::is_same_v<Kernel, void(TraceArgs)>, "not this kernel's argument");
    RareArgs *p = (RareArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// The bricks' address, kept in scalar registers through a trace loop.
__device__ __forceinline__ GlobalBytes kept_cells(const TraceArgs &a) {
    GlobalBytes p = (GlobalBytes)a.cells;
    asm volatile("" : "+s"(p));
    return p;
}

// One sample of the fixed sphere-trace sequence, at sample k of rays o + t w, for the
// lanes of `live`; returns those whose ray goes on. There t and k are advanced; where a
// ray stops they stay, and stop_kind names the outcome from them, the sample's distance
// and its level (-1 outside every level). Other lanes' values stay as they are.
// Analytic backend: no grid box, so a ray misses only past t_max; the distance is
// the minimum over the cell's primitives, starting from `bound` (the previous
// sample's bound, +inf at a ray's first sample), and a primary ray's sample names
// its nearest primitive in `slot` (level is 0).
template <bool kPrimary, int kSdf, bool kWide>
__device__ __forceinline__ uint64_t trace_step(const TraceArgs &a, GlobalBytes cells,
                                               const SdfLds<kSdf> &s, uint64_t live, float o0,
                                               float o1, float o2, float w0, float w1, float w2,
                                               float &t, int &k, float &dist, int &level,
                                               float &bound, int &slot) {
    const float x0 = fmaf(t, w0, o0), x1 = fmaf(t, w1, o1), x2 = fmaf(t, w2, o2);
    uint64_t inside = live & ~__ballot(t > a.t_max);
    if constexpr (kSdf == kSdfAnalytic) {
        level = 0;
        if (in_mask(inside))
            dist = analytic_distance<kPrimary>(a.an, s.lv, x0, x1, x2, bound, slot);
    } else {
        constexpr bool kHalf = kSdf == kSdfGrid16;
        const int found = select_level(a, x0, x1, x2);
        inside &= __ballot(found >= 0);
        level = in_mask(live) ? found : level;
        if (in_mask(inside))
            dist = distance_inside<kHalf, kWide>(cells, s.lv[found], x0, x1, x2);
    }
    const uint64_t go = inside & ~__ballot(dist < a.eps) & ~__ballot(k + 1 == a.max_steps);
    if (in_mask(go)) {
        t = fmaf(a.relax, dist, t);
        ++k;
        if (kSdf == kSdfAnalytic) bound = next_bound(a.relax, dist);
    }
    return go;
}

// The outcome of a ray that stopped, and its number of samples.
template <bool kPrimary>
__device__ __forceinline__ int stop_kind(const TraceArgs &a, float t, int k, float dist, int level,
                                         int &steps) {
    const bool over = t > a.t_max;
    steps = over || level < 0 ? k : k + 1;
    if (over) return kMissTmax;
    if (level < 0) return kMissExit;
    if (kPrimary && k == 0 && dist < 0.0f) return kInside;
    return dist < a.eps ? kHit : kHitExhausted;
}

// ----------------------------------------------------------- radiometry -----

template <typename Args>
__device__ __forceinline__ float3 albedo_at(const Args &a, const LevelLds &d, float x0,
                                            float x1, float x2) {
    if (!d.alb) return make_float3(a.alb0, a.alb1, a.alb2);
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

// ------------------------------------------------------------- kernels ------

template <typename Args>
__device__ __forceinline__ void write_record(const Args &a, int ray, float t, int kind,
                                             int level, int steps, int vis, int shadow_steps,
                                             float n0, float n1, float n2) {
    if (a.records) {
        int4 *rec = reinterpret_cast<int4 *>(a.records) + 2 * (int64_t)ray;
        rec[0] = make_int4(kind | (level << 8), steps, vis, shadow_steps);
        rec[1] = make_int4(__float_as_int(t), __float_as_int(n0), __float_as_int(n1),
                           __float_as_int(n2));
    }
}

template <typename Args>
__device__ __forceinline__ void write_ray(const Args &a, int ray, float4 out, int kind,
                                          int level, int steps, int vis, int shadow_steps,
                                          float n0, float n1, float n2) {
    store_streamed(&a.payload[ray], out);
    write_record(a, ray, out.w, kind, level, steps, vis, shadow_steps, n0, n1, n2);
}

// Payload of a hit: (albedo / pi) (sun radiance x n.l-or-0 + gain x multi-bounce), t.
__device__ __forceinline__ float4 shade_hit(const TraceArgs &a, float3 alb, float lit, float3 ind,
                                            float t) {
    const float inv_pi = 0.318309886183790671538f;
    float4 out;
    out.x = alb.x * inv_pi * (a.rad0 * lit + a.gain * ind.x);
    out.y = alb.y * inv_pi * (a.rad1 * lit + a.gain * ind.y);
    out.z = alb.z * inv_pi * (a.rad2 * lit + a.gain * ind.z);
    out.w = t;
    return out;
}

// Per-wave staging of hit-queue entries (ray, bits of t, packed info, 0) in LDS;
// flushed to the global queue 64 at a time with one atomic.
__device__ __forceinline__ void flush_hits(RareArgs &a, int4 *buf, int count) {
    if (count == 0) return;
    int base = 0;
    if (__lane_id() == 0) base = atomicAdd(a.counter + 2, count);
    base = __builtin_amdgcn_readfirstlane(base);
    const int lane = (int)__lane_id();
    if (lane < count) a.hitq[base + lane] = buf[lane];
    __builtin_amdgcn_wave_barrier();
}

constexpr int kChunk = 256;       // primary rays claimed from a counter at a time
constexpr int kChunkSpread = 256; // ... while every wave of the grid gets this many
constexpr int kHitChunk = 64;     // queued hits claimed at a time (spreads them over all waves)
// Rays per block of the XCD interleave (BlockFeeder): blocks of 65536 rays keep
// the 8 XCDs on neighbouring blocks of the Morton order (one compact window for the
// shared Infinity Cache and HBM) with a compact region per L2. Measured at 16384 x 256
// (frame time, FP32 / FP16): one shared counter 0.862 / 0.758 ms; blocks of 1, 16,
// 64, 256, 512 probes 0.844, 0.833, 0.823, 0.799, 0.802 / -, -, 0.669, 0.652, 0.666;
// one contiguous part per XCD (blocks of 2048) was 1.6x slower than one counter.
constexpr int kXcdBlockRays = 65536;
constexpr int kEndBatch = 16;     // idle lanes at which a wave records ended rays and goes on
constexpr int kFetchAt = 48;      // a wave fetches 64 more rays when no more than these wait

// Primary sphere trace, persistent and wave-compacted: each lane owns one ray and takes
// one sample per iteration. Once kEndBatch lanes are idle the wave records the rays that
// ended and gives those lanes the next rays of its queue, which it fills 64 at a time
// ahead of need: runs of consecutive slots per atomic (rays of one probe, probes visited
// in Morton order of their grid cell, blocks of that order dealt to the XCDs in turn --
// see BlockFeeder), fetched in stages, one per iteration (the probe's index and the
// direction; its position and first sample; into the queue), whose loads return beside
// the iterations' own samples. Misses and probes inside geometry write their payload
// here; hits are appended to a compact queue (ray, t, outcome, level, steps) for
// hits_kernel, staged per wave in LDS. Each ray's arithmetic is the fixed sequence of
// trace_step, whatever lane or wave runs it. Every wave exits once the counters have
// passed the last ray and its lanes are idle, after flushing its staged hits.
// Alone at 16384 x 256 (open scene): 431 us in binary32 and 353 us in binary16, 99 M and
// 116 M vector instructions at 80 % of the lanes; taking rays straight into idle lanes
// once half of a wave's had stopped, over corner quads: 530 and 467 us, 159 M and 168 M
// at 57 %. More or fewer resident waves, direction-major ray orders over 64 to 16384
// probes (each direction's rays side by side) and a lane-by-lane look-ahead in registers
// (478 / 419 us) were no faster.
template <int kSdf, bool kWide = false>
__global__ __launch_bounds__(256) void primary_kernel(TraceArgs a) {
    using Self = decltype(primary_kernel<kSdf, kWide>);
    __shared__ SdfLds<kSdf> s_sdf;
    __shared__ int4 s_hits[4][64];
    constexpr int kRayQueue = 128;
    // origin and the distance of the first sample (0: not taken), direction and index
    __shared__ WaitingRay s_rays[4][kRayQueue];
    load_sdf<kSdf>(a, s_sdf);
    const GlobalBytes cells = kept_cells(a);
    const int lane = (int)__lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const int total =
        __builtin_amdgcn_readfirstlane((a.probe_count ? *a.probe_count : a.P) * a.R);
    // whole probes per claim, and rays queued ahead, while that still gives every wave
    // several; else few rays spread over all waves. Likewise the XCDs' blocks
    const bool plenty = total / kChunkSpread >= (int)gridDim.x * 4;
    const int chunk = plenty ? kChunk : 64;
    BlockFeeder feed(chunk, max(1, min(kXcdBlockRays, total / (4 * kXcds)) / chunk));
    // lanes that are stepping; that stopped and are not recorded
    uint64_t live = 0, ended = 0;
    int staged = 0;                 // hits in s_hits[wave]
    int head = 0, waiting = 0;      // first and number of the rays in s_rays[wave]
    int stage = 0, coming = 0;      // a fetch's stage (0: none), lanes 0 .. coming-1 have a ray
    int ray = 0, k = 0, level = 0, slot = -1, n_ray = 0, n_probe = 0;
    float o0 = 0, o1 = 0, o2 = 0, w0 = 0, w1 = 0, w2 = 0, t = 0, dist = 0, bound = INFINITY;
    float m0 = 0, m1 = 0, m2 = 0, v0 = 0, v1 = 0, v2 = 0;
    int2 n_first = make_int2(0, -1);
    while (true) {
        if (stage == 2) {
            RareArgs &f = *rare_args<Self>();
            if (lane < coming) {
                // the first sample sits at the probe (fma(0, w, o) = o) for every
                // ray of it: where that sample only steps on (a level holds the
                // probe, or the primitives are traced; distance >= eps), take
                // the step from the probe's precomputed sample; otherwise the
                // first trace_step samples
                const float d0 = __int_as_float(n_first.x);
                const bool known = f.probe_first && a.max_steps > 1 &&
                                   (kSdf == kSdfAnalytic || n_first.y >= 0) && !(d0 < a.eps);
                WaitingRay &r = s_rays[wave][(head + waiting + lane) & (kRayQueue - 1)];
                r.from = make_float4(m0, m1, m2, known ? d0 : 0.0f);
                r.dir = make_float4(v0, v1, v2, __int_as_float(n_probe * f.R + n_ray));
            }
            __builtin_amdgcn_wave_barrier();
            waiting += coming;
            stage = 0;
        } else if (stage == 1) {
            RareArgs &f = *rare_args<Self>();
            if (lane < coming) {
                m0 = f.probe_pos[3 * n_probe];
                m1 = f.probe_pos[3 * n_probe + 1];
                m2 = f.probe_pos[3 * n_probe + 2];
                if (f.probe_first) n_first = f.probe_first[n_probe];
            }
            stage = 2;
        }
        if (__popcll(live) <= 64 - kEndBatch) {
            if (ended) {
                RareArgs &f = *rare_args<Self>();
                bool hit = false;
                int4 entry = make_int4(0, 0, 0, 0);
                if (in_mask(ended)) {
                    int steps;
                    const int kind = stop_kind<true>(a, t, k, dist, level, steps);
                    if (kind == kHit || kind == kHitExhausted) {
                        hit = true;
                        entry = make_int4(ray, __float_as_int(t), pack_hit(kind, level, steps),
                                          kSdf == kSdfAnalytic ? slot : 0);
                    } else {
                        const float4 out = kind == kInside
                                               ? make_float4(0.0f, 0.0f, 0.0f, 0.0f)
                                               : make_float4(f.sky0, f.sky1, f.sky2, a.t_max);
                        write_ray(f, ray, out, kind, 0, steps, -1, 0, 0.0f, 0.0f, 0.0f);
                    }
                }
                ended = 0;
                const uint64_t hm = __ballot(hit);
                if (hm) {
                    const int n = __popcll(hm);
                    if (staged + n > 64) {
                        flush_hits(*rare_args<Self>(), s_hits[wave], staged);
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
                    const WaitingRay r = s_rays[wave][(head + rank) & (kRayQueue - 1)];
                    o0 = r.from.x; o1 = r.from.y; o2 = r.from.z;
                    w0 = r.dir.x; w1 = r.dir.y; w2 = r.dir.z;
                    ray = __float_as_int(r.dir.w);
                    const float d0 = r.from.w;
                    t = fmaf(a.relax, d0, 0.0f);
                    k = d0 != 0.0f ? 1 : 0;
                    if constexpr (kSdf == kSdfAnalytic)
                        bound = d0 != 0.0f ? next_bound(a.relax, d0) : INFINITY;
                }
                __builtin_amdgcn_wave_barrier();
                live |= take;
                const int n = __popcll(take);
                head += n;
                waiting -= n;
            }
            if (stage == 0 && !feed.exhausted &&
                (plenty ? waiting <= kFetchAt : __popcll(live) <= 32)) {
                RareArgs &f = *rare_args<Self>();
                coming = 0;
                while (coming < 64 && !feed.exhausted) {
                    int first = 0;
                    const int n = feed.claim(f.parts, total, 64 - coming, first);
                    if (lane >= coming && lane < coming + n) {
                        // slot -> (probe in Morton order, ray): neighbouring slots trace
                        // neighbouring probes, so the rays in flight share cache lines
                        const int sid = first + lane - coming;
                        // sid / R: at most one too large (sid < 2^31, R <= 2^10)
                        int q = (int)__umulhi((uint32_t)sid, f.r_magic);
                        int i = sid - q * f.R;
                        if (i < 0) { --q; i += f.R; }
                        n_probe = f.probe_order[q];
                        v0 = f.dirs[3 * i]; v1 = f.dirs[3 * i + 1]; v2 = f.dirs[3 * i + 2];
                        n_ray = i;
                    }
                    coming += n;
                }
                stage = coming ? 1 : 0;
            }
            if (!live) {  // then no ray waits either
                if (stage == 0 && feed.exhausted) {
                    flush_hits(*rare_args<Self>(), s_hits[wave], staged);
                    break;
                }
                continue;
            }
        }
        const uint64_t go = trace_step<true, kSdf, kWide>(a, cells, s_sdf, live, o0, o1, o2, w0, w1, w2,
                                                   t, k, dist, level, bound, slot);
        ended |= live & ~go;
        live = go;
    }
}

// First half of hit shading, what does not depend on the previous atlas, for the queue
// the primary trace built; persistent and wave-compacted like primary_kernel. A wave
// claims 64 hits at a time and fetches them in stages (queue entry; probe position and
// direction), then, all lanes at once, computes their points, normals and albedos and
// stores their records (geo) as if lit, and queues in LDS the shadow rays of those that
// face the light; its lanes step shadow rays from that queue, and a blocked one clears
// its hit's sun term. shade_kernel adds the multi-bounce lookup. Every wave exits once
// the queue's claims have passed its end and its lanes are idle.
// Alone on the open scene's hits (16384 x 256): 144 us in either precision, bound by the
// 64-step chains of its last shadow rays; with points, normals and shading done by
// whichever lanes were due, beside the stepping ones, 202 and 216 us at 42 % of the lanes.
template <int kSdf, bool kWide = false>
__global__ __launch_bounds__(256) void hits_kernel(TraceArgs a) {
    using Self = decltype(hits_kernel<kSdf, kWide>);
    constexpr int kQueue = 128;
    __shared__ SdfLds<kSdf> s_sdf;
    __shared__ float4 s_rays[4][kQueue];   // origin, hit-queue index
    load_sdf<kSdf>(a, s_sdf);
    const GlobalBytes cells = kept_cells(a);
    const int lane = (int)__lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    // queue length, final once primary_kernel has finished
    const int total = __builtin_amdgcn_readfirstlane(a.counter[2]);
    const bool plenty = total / kChunk >= (int)gridDim.x * 4;
    bool exhausted = false;
    uint64_t live = 0, ended = 0;   // lanes that are stepping; that stopped, not recorded
    int head = 0, waiting = 0;      // first and number of the rays in s_rays[wave]
    int stage = 0, first = 0, coming = 0;   // hits first .. first+coming-1 are being fetched
    int qi = 0, k = 0, level = 0, unused = 0;
    float o0 = 0, o1 = 0, o2 = 0, t = 0, dist = 0, bound = INFINITY;
    int4 e = make_int4(0, 0, 0, 0);
    float p0 = 0, p1 = 0, p2 = 0, w0 = 0, w1 = 0, w2 = 0;
    while (true) {
        if (stage == 2) {
            RareArgs &f = *rare_args<Self>();
            bool lit = false;
            float4 from = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (lane < coming) {
                const float ht = __int_as_float(e.y);
                const float x0 = fmaf(ht, w0, p0), x1 = fmaf(ht, w1, p1), x2 = fmaf(ht, w2, p2);
                float n0, n1, n2;
                float3 alb;
                if constexpr (kSdf == kSdfAnalytic) {
                    analytic_normal(e.w, x0, x1, x2, w0, w1, w2, n0, n1, n2);
                    alb = make_float3(f.prim_alb[3 * e.w], f.prim_alb[3 * e.w + 1],
                                      f.prim_alb[3 * e.w + 2]);
                } else {
                    const LevelLds &d = s_sdf.lv[(e.z >> 4) & 15];
                    alb = albedo_at(f, d, x0, x1, x2);
                    hit_normal<kSdf == kSdfGrid16>(cells, d, kWide, x0, x1, x2, w0, w1, w2, n0, n1,
                                                   n2);
                }
                const float ndl = fmaf(n2, a.l2, fmaf(n1, a.l1, n0 * a.l0));
                lit = ndl > 0.0f;
                const int64_t at = 2 * (int64_t)(first + lane);   // passes INT_MAX from 2^30 hits
                f.geo[at] = make_float4(n0, n1, n2, lit ? ndl : 0.0f);
                f.geo[at + 1] = make_float4(alb.x, alb.y, alb.z, 0.0f);
                write_record(f, e.x, ht, e.z & 15, (e.z >> 4) & 15, e.z >> 8, lit ? 1 : -1, 0, n0,
                             n1, n2);
                from = make_float4(fmaf(n0, a.bias, x0), fmaf(n1, a.bias, x1),
                                   fmaf(n2, a.bias, x2), __int_as_float(first + lane));
            }
            const uint64_t m = __ballot(lit);
            if (lit) s_rays[wave][(head + waiting + __popcll(m & below)) & (kQueue - 1)] = from;
            order_wave_stores();   // the records; a lane of a blocked ray changes another's
            waiting += __popcll(m);
            stage = 0;
        } else if (stage == 1) {
            RareArgs &f = *rare_args<Self>();
            if (lane < coming) {
                const int p = e.x / f.R, i = e.x - p * f.R;
                p0 = f.probe_pos[3 * p]; p1 = f.probe_pos[3 * p + 1]; p2 = f.probe_pos[3 * p + 2];
                w0 = f.dirs[3 * i]; w1 = f.dirs[3 * i + 1]; w2 = f.dirs[3 * i + 2];
            }
            stage = 2;
        }
        if (__popcll(live) <= 64 - kEndBatch) {
            RareArgs &f = *rare_args<Self>();
            if (ended) {
                if (in_mask(ended)) {
                    int steps;
                    const int kind = stop_kind<false>(a, t, k, dist, level, steps);
                    const bool blocked = kind == kHit || kind == kHitExhausted;
                    if (blocked) f.geo[2 * (int64_t)qi].w = 0.0f;
                    if (f.records) {
                        int *rec = f.records + 8 * (int64_t)f.hitq[qi].x;
                        rec[2] = blocked ? 0 : 1;
                        rec[3] = steps;
                    }
                }
                ended = 0;
            }
            if (waiting > 0) {
                const int rank = __popcll(~live & below);
                const uint64_t take = __ballot(in_mask(~live) && rank < waiting);
                if (in_mask(take)) {
                    const float4 r = s_rays[wave][(head + rank) & (kQueue - 1)];
                    o0 = r.x; o1 = r.y; o2 = r.z;
                    qi = __float_as_int(r.w);
                    t = 0.0f;
                    k = 0;
                    bound = INFINITY;
                }
                __builtin_amdgcn_wave_barrier();
                live |= take;
                const int n = __popcll(take);
                head += n;
                waiting -= n;
            }
            if (stage == 0 && !exhausted &&
                (plenty ? waiting <= kFetchAt : __popcll(live) + waiting <= 32)) {
                if (lane == 0) first = atomicAdd(f.counter + 1, kHitChunk);
                first = __builtin_amdgcn_readfirstlane(first);
                coming = min(kHitChunk, total - first);
                if (coming > 0) {
                    if (lane < coming) e = f.hitq[first + lane];
                    stage = 1;
                } else {
                    exhausted = true;
                }
            }
            if (!live) {
                if (stage == 0 && exhausted && waiting == 0) break;
                continue;
            }
        }
        const uint64_t go = trace_step<false, kSdf, kWide>(a, cells, s_sdf, live, o0, o1, o2, a.l0,
                                                           a.l1, a.l2, t, k, dist, level, bound,
                                                           unused);
        ended |= live & ~go;
        live = go;
    }
}

// Second half of hit shading: per hit-queue entry, the hit point again (the
// same operations as hits_kernel), the multi-bounce lookup into the previous atlas
// and the payload. Grid-stride over the queue, whose length the primary trace left
// in counter[2].
__global__ __launch_bounds__(256) void shade_kernel(TraceArgs a) {
    const int total = a.counter[2];
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < total; q += gridDim.x * blockDim.x) {
        const int4 e = a.hitq[q];
        const float4 g0 = a.geo[2 * (int64_t)q], g1 = a.geo[2 * (int64_t)q + 1];
        const int ray = e.x;
        const float ht = __int_as_float(e.y);
        float3 ind = make_float3(0.0f, 0.0f, 0.0f);
        if (a.gain != 0.0f) {
            const int p = ray / a.R, i = ray - (ray / a.R) * a.R;
            const float hx0 = fmaf(ht, a.dirs[3 * i], a.probe_pos[3 * p]);
            const float hx1 = fmaf(ht, a.dirs[3 * i + 1], a.probe_pos[3 * p + 1]);
            const float hx2 = fmaf(ht, a.dirs[3 * i + 2], a.probe_pos[3 * p + 2]);
            ind = interp_irradiance(a.prev_irr, a.irr_res, a.pg, hx0, hx1, hx2, g0.x, g0.y, g0.z);
        }
        store_streamed(&a.payload[ray], shade_hit(a, make_float3(g1.x, g1.y, g1.z), g0.w, ind, ht));
    }
}

// One block per texel row of the weight matrices (irradiance rows, then depth
// rows), plus one block that writes the binary32 directions.
__global__ __launch_bounds__(256) void tables_kernel(TableArgs a) {
    __shared__ double red[256];
    const int row = blockIdx.x + a.row0;
    const int tid = threadIdx.x;
    const bool is_dirs = row == a.Ti + a.Td;
    const bool is_depth = row >= a.Ti && !is_dirs;
    const int t = is_depth ? row - a.Ti : row;
    double q[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) q[k] = a.q_dev ? a.q_dev[k] : a.q[k];
    double nt0 = 0, nt1 = 0, nt2 = 0;
    if (!is_dirs) {
        const double *nt = is_depth ? a.texel_d + 3 * t : a.texel_i + 3 * t;
        nt0 = nt[0]; nt1 = nt[1]; nt2 = nt[2];
    }
    double part = 0.0;
    for (int i = tid; i < a.R; i += 256) {
        const double s0 = a.base[3 * i], s1 = a.base[3 * i + 1], s2 = a.base[3 * i + 2];
        const double w0 = q[0] * s0 + q[1] * s1 + q[2] * s2;
        const double w1 = q[3] * s0 + q[4] * s1 + q[5] * s2;
        const double w2 = q[6] * s0 + q[7] * s1 + q[8] * s2;
        if (is_dirs) {
            a.dirs[3 * i] = (float)w0;
            a.dirs[3 * i + 1] = (float)w1;
            a.dirs[3 * i + 2] = (float)w2;
            continue;
        }
        double c = nt0 * w0 + nt1 * w1 + nt2 * w2;
        double w = c > 0.0 ? c : 0.0;
        if (is_depth) {
            w = pow(w, a.sharp);
            if (a.w16_d) {  // precision form: BF16 depth weights, sums of the rounded values
                const __bf16 b = (__bf16)(float)w;
                a.w16_d[weight_index<32>(t, i, a.Rpad)] = b;
                w = (double)(float)b;
            } else {
                a.wt_d[weight_index<16>(t, i, a.Rpad)] = (float)w;
            }
        } else {
            if (a.w16_i) {  // precision form: FP16 irradiance weights
                const _Float16 h = (_Float16)w;
                a.w16_i[weight_index<32>(t, i, a.Rpad)] = h;
                w = (double)(float)h;
            } else {
                a.wt_i[weight_index<16>(t, i, a.Rpad)] = (float)w;
            }
        }
        part += w;
    }
    if (is_dirs) {
        if (a.counter)  // trace (and fallback) counters
            for (int e = tid; e < a.ncounter; e += blockDim.x) a.counter[e] = 0;
        return;
    }
    red[tid] = part;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) red[tid] += red[tid + s];
        __syncthreads();
    }
    if (tid == 0) {
        const double sum = red[0];
        const double pi = 3.14159265358979323846;
        if (is_depth) a.norm_d[t] = sum > 0.0 ? (float)(1.0 / sum) : -1.0f;
        else a.norm_i[t] = sum > 0.0 ? (float)(pi / sum) : -1.0f;
    }
}

template <int kMaps, int kP>
__global__ __launch_bounds__(256, 4) void blend16_kernel(BlendArgs a) {
    blend16_block<kMaps, kP>(a, blockIdx.x * kP);
}

// One workgroup's share (probe slots pb .. pb+kP-1) of the FP32 blend. Sixteen rays make
// four products: lane group g takes rays 4 g .. 4 g + 3 of both operands, one ray per
// product, so that a lane's operands for all four are 16 bytes side by side -- the
// weights' in their table (a step's read while the one before is multiplied), the
// payload's in its LDS column. The next 64 rays' payload is read while the present ones
// are multiplied.
// At 16384 x 256 and 8x8 + 16x16 maps: 81 us, of which 37.5 are the matrix cores' (they
// reach 151 TFLOP/s of binary32 at best) and some 20 the reading and writing of the maps,
// which the workgroups of a CU come to at about the same time. One dword per operand and
// product from tables of one row per ray, and an epilogue through three passes over LDS:
// 114 us. Raising the waves' priority by their slot, to pull the workgroups of a CU apart,
// gave nothing.
template <int kMaps, int kP>
__device__ __forceinline__ void blend32_block(const BlendArgs &a, int pb) {
    constexpr bool kStd = kMaps == kStdMaps;
    constexpr int kIS = kStd ? kIrrSlots : kIrrSlotsAny, kSlots = kIS + kDepthSlots;
    constexpr int kPitch = kBlendChunk + 4;   // a column's rays; +4 spreads the banks
    constexpr int kNi = (3 * kP + 15) / 16, kNd = (2 * kP + 15) / 16;
    // payload of kP probes x 4 channels, plus one zero column for absent probes; the
    // epilogue through LDS reuses the buffer
    constexpr int kStage = (kP * 4 + 1) * kPitch, kBuf = kP * (kStd ? kProbeFloatsStd : kProbeFloatsAny);
    __shared__ __attribute__((aligned(16))) float sbuf[kStage > kBuf ? kStage : kBuf];
    __shared__ float s_h[kP];
    __shared__ int s_pid[kP];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, krow = lane >> 4;
    const int count = a.probe_list ? min(*a.probe_count, a.P) : a.P;
    if (pb >= count) return;
    const int np = min(kP, count - pb);
    const int Ti = a.irr_res * a.irr_res, Td = a.depth_res * a.depth_res;
    const int mti = (Ti + 15) >> 4, mtd = (Td + 15) >> 4;
    load_blend_probes<kP>(a, pb, np, s_pid, s_h);
    for (int e = tid; e < kPitch; e += 256) sbuf[kP * 4 * kPitch + e] = 0.0f;

    // B-operand columns of this lane: irradiance (q, c), depth (q, m)
    int bi_off[kNi], bd_off[kNd];
#pragma unroll
    for (int n = 0; n < kNi; ++n) {
        const int col = n * 16 + row, q = col / 3, c = col - 3 * q;
        bi_off[n] = (q < np ? q * 4 + c : kP * 4) * kPitch + 4 * krow;
    }
#pragma unroll
    for (int n = 0; n < kNd; ++n) {
        const int q = (n * 16 + row) >> 1;
        bd_off[n] = (q < np ? q * 4 + 3 : kP * 4) * kPitch + 4 * krow;
    }
    const bool square = (row & 1) != 0;

    // this thread's rays of a chunk (absent probes and rays read a present one and are
    // zeroed)
    constexpr int kLoads = kP * kBlendChunk / 256;
    float4 pv[kLoads];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int b = 0; b < kLoads; ++b) {
            const int e = tid + 256 * b, q = e / kBlendChunk, kk = e - q * kBlendChunk;
            pv[b] = load_streamed(a.payload + (size_t)s_pid[min(q, np - 1)] * a.R +
                                  min(k0 + kk, a.R - 1));
        }
    };
    const int passes = kMaps == kLargeMaps ? blend_passes(a.irr_res, a.depth_res) : 1;
    for (int pass = 0; pass < passes; ++pass) {
        floatx4 ai[kIS][kNi], ad[kDepthSlots][kNd];
        // the slots' weights (irradiance tiles, then depth tiles) for a step and the next
        GlobalBytes w[kSlots];
        floatx4 a0[kSlots], a1[kSlots];
        const int ti = pass * 4 * kIS + wave, td = pass * 4 * kDepthSlots + wave;
        auto load_weights = [&](floatx4 (&av)[kSlots], int k) {
            const uint32_t at = (uint32_t)(64 * min(k, a.R - 16) + 16 * lane);
#pragma unroll
            for (int s = 0; s < kSlots; ++s)
                av[s] = *(const __attribute__((address_space(1))) floatx4 *)(w[s] + at);
        };
        auto multiply = [&](const floatx4 (&av)[kSlots], int kk) {
            floatx4 bi[kNi], bd[kNd];
#pragma unroll
            for (int n = 0; n < kNi; ++n)
                bi[n] = *reinterpret_cast<const floatx4 *>(&sbuf[bi_off[n] + kk]);
#pragma unroll
            for (int n = 0; n < kNd; ++n) {
                const floatx4 t = *reinterpret_cast<const floatx4 *>(&sbuf[bd_off[n] + kk]);
                bd[n] = square ? t * t : t;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
#pragma unroll
                for (int s = 0; s < kIS; ++s)
                    if (kStd || ti + 4 * s < mti)
#pragma unroll
                        for (int n = 0; n < kNi; ++n)
                            ai[s][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s][k], bi[n][k],
                                                                            ai[s][n], 0, 0, 0);
#pragma unroll
                for (int s = 0; s < kDepthSlots; ++s)
                    if (kStd || td + 4 * s < mtd)
#pragma unroll
                        for (int n = 0; n < kNd; ++n)
                            ad[s][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[kIS + s][k], bd[n][k],
                                                                            ad[s][n], 0, 0, 0);
            }
        };
        __syncthreads();
        fetch(0);
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
            // (slots past a map's last tile read that one's weights, unused)
            const int tile = s < kIS ? min(ti + 4 * s, mti - 1) : min(td + 4 * (s - kIS), mtd - 1);
            w[s] = (GlobalBytes)((s < kIS ? a.wt_i : a.wt_d) + (size_t)(16 * tile) * a.Rpad);
        }
        load_weights(a0, 0);
#pragma unroll
        for (int n = 0; n < kNi; ++n)
#pragma unroll
            for (int s = 0; s < kIS; ++s) ai[s][n] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int n = 0; n < kNd; ++n)
#pragma unroll
            for (int s = 0; s < kDepthSlots; ++s) ad[s][n] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        for (int k0 = 0; k0 < a.R; k0 += kBlendChunk) {
            const int kc = min(kBlendChunk, a.R - k0);
            if (k0) __syncthreads();
#pragma unroll
            for (int b = 0; b < kLoads; ++b) {
                const int e = tid + 256 * b, q = e / kBlendChunk, kk = e - q * kBlendChunk;
                const float4 v = (q < np && kk < kc) ? pv[b] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                float *d = sbuf + q * 4 * kPitch + kk;
                d[0] = v.x; d[kPitch] = v.y; d[2 * kPitch] = v.z; d[3 * kPitch] = v.w;
            }
            __syncthreads();
            load_weights(a1, k0 + 16);
            if (k0 + kBlendChunk < a.R) fetch(k0 + kBlendChunk);
            for (int kk = 0; kk < kc; kk += 32) {
                if (kk) load_weights(a1, k0 + kk + 16);
                __builtin_amdgcn_sched_barrier(0);   // the reads go out before the products
                multiply(a0, kk);
                if (kk + 16 >= kc) break;
                load_weights(a0, k0 + kk + 32);
                __builtin_amdgcn_sched_barrier(0);
                multiply(a1, kk + 16);
            }
        }
        if constexpr (kMaps == kLargeMaps)
            blend_epilogue_direct<false>(a, s_h, s_pid, np, ti, td, row, krow, ai, ad);
        else
            blend_epilogue_lds<kStd, false>(a, s_h, s_pid, np, ti, td, row, krow, ai, ad, sbuf);
    }
    __syncthreads();
    if (tid < np && a.reject) a.reject[s_pid[tid]] = 0;
}

// (four workgroups per CU: 128 registers)
template <int kMaps, int kP>
__global__ __launch_bounds__(256, kMaps == kLargeMaps ? 2 : 4) void blend_kernel(BlendArgs a) {
    blend32_block<kMaps, kP>(a, blockIdx.x * kP);
}

// Alg. 1 per probe: from the grid position, while the distance is below t1 (at most
// `iterations` times) take a Newton step t1 - d along the normalised distance
// gradient (the hit-normal rule; +y where it vanishes), each coordinate kept within
// the offset of the grid position; stop outside every level. Then compare with the
// last position and reject the history of a probe that moved more than t2.
template <bool kHalf>
__global__ __launch_bounds__(256) void relocate_kernel(TraceArgs a, RelocateArgs r) {
    __shared__ LevelLds s_lv[kMaxLevels];
    load_levels(a, s_lv);
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.P) return;
    const float g0 = r.grid_pos[3 * p], g1 = r.grid_pos[3 * p + 1], g2 = r.grid_pos[3 * p + 2];
    const float lo0 = g0 - r.off0, lo1 = g1 - r.off1, lo2 = g2 - r.off2;
    const float hi0 = g0 + r.off0, hi1 = g1 + r.off1, hi2 = g2 + r.off2;
    float x0 = g0, x1 = g1, x2 = g2;
    for (int it = 0; it < r.iterations; ++it) {
        const int L = select_level(a, x0, x1, x2);
        if (L < 0) break;
        const float d = sample_at<kHalf>((GlobalBytes)a.cells, s_lv[L], a.wide, x0, x1, x2);
        if (!(d < r.t1)) break;
        float n0, n1, n2;
        hit_normal<kHalf>((GlobalBytes)a.cells, s_lv[L], a.wide, x0, x1, x2, 0.0f, -1.0f, 0.0f, n0, n1, n2);
        const float step = r.t1 - d;
        x0 = fminf(fmaxf(fmaf(step, n0, x0), lo0), hi0);
        x1 = fminf(fmaxf(fmaf(step, n1, x1), lo1), hi1);
        x2 = fminf(fmaxf(fmaf(step, n2, x2), lo2), hi2);
    }
    const float dx = x0 - r.pos[3 * p], dy = x1 - r.pos[3 * p + 1], dz = x2 - r.pos[3 * p + 2];
    const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
    if (d2 > r.t2 * r.t2) r.reject[p] = 1;
    r.pos[3 * p] = x0;
    r.pos[3 * p + 1] = x1;
    r.pos[3 * p + 2] = x2;
}

// Signed distance at each probe position: the trace's own level choice and sampler.
template <bool kHalf>
__global__ __launch_bounds__(256) void probe_sdf_kernel(TraceArgs a, float *out) {
    __shared__ LevelLds s_lv[kMaxLevels];
    load_levels(a, s_lv);
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.P) return;
    const float x0 = a.probe_pos[3 * p], x1 = a.probe_pos[3 * p + 1], x2 = a.probe_pos[3 * p + 2];
    const int L = select_level(a, x0, x1, x2);
    out[p] = L < 0 ? 1e30f : sample_at<kHalf>((GlobalBytes)a.cells, s_lv[L], a.wide, x0, x1, x2);
}

// Each probe's first sample: the level its position selects and the distance there,
// by the same sequence as a ray's sample at t = 0.
template <bool kHalf>
__global__ __launch_bounds__(256) void probe_first_kernel(TraceArgs a, int2 *out) {
    __shared__ LevelLds s_lv[kMaxLevels];
    load_levels(a, s_lv);
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.P) return;
    const float x0 = a.probe_pos[3 * p], x1 = a.probe_pos[3 * p + 1], x2 = a.probe_pos[3 * p + 2];
    const int L = select_level(a, x0, x1, x2);
    const float d = L < 0 ? 0.0f : sample_at<kHalf>((GlobalBytes)a.cells, s_lv[L], a.wide, x0, x1, x2);
    out[p] = make_int2(__float_as_int(d), L);
}

// The same for the analytic backend: the culled query's distance at the probe from an
// unbounded start, and the nearest primitive's slot.
__global__ __launch_bounds__(256) void probe_first_analytic_kernel(TraceArgs a, int2 *out) {
    __shared__ float4 s_lv[kMaxCellLevels];
    load_prims(a.an, s_lv);
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.P) return;
    int slot;
    const float d = analytic_distance<true>(a.an, s_lv, a.probe_pos[3 * p], a.probe_pos[3 * p + 1],
                                            a.probe_pos[3 * p + 2], INFINITY, slot);
    out[p] = make_int2(__float_as_int(d), slot);
}

__global__ __launch_bounds__(256) void sample_kernel(SampleArgs a) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= a.n) return;
    float3 e = interp_irradiance(a.atlas, a.irr_res, a.pg, a.points[3 * q], a.points[3 * q + 1],
                                 a.points[3 * q + 2], a.normals[3 * q], a.normals[3 * q + 1],
                                 a.normals[3 * q + 2]);
    a.out[3 * q] = e.x;
    a.out[3 * q + 1] = e.y;
    a.out[3 * q + 2] = e.z;
}

// Cell bricks of one grid level (see load_corners), one thread per vertex column of a
// brick; past the grid's last vertex a column repeats it (no cell reads those). The
// binary16 form clamps each value to +-65504 and rounds it to nearest even.
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ _Float16 to_half(float v) {
    return (_Float16)fminf(fmaxf(v, -65504.0f), 65504.0f);
}

template <bool kHalf>
__global__ __launch_bounds__(256) void pack_cells_kernel(const float *__restrict__ g, int n0, int n1,
                                                         int n2, CellShape sh,
                                                         char *__restrict__ cells) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t line = e >> 4;
    if (line >= sh.lines()) return;
    const int col = (int)(e & 15);
    const int64_t row = line / sh.nb0;
    const int64_t b0 = line - row * sh.nb0, b2 = row / sh.nb1, b1 = row - b2 * sh.nb1;
    const int64_t i = min(3 * b0 + (col & 3), (int64_t)n0 - 1);
    const int64_t j = min(3 * b1 + (col >> 2), (int64_t)n1 - 1);
    const auto at = [&](int64_t k) {
        return g[(min(k, (int64_t)n2 - 1) * n1 + j) * n0 + i];
    };
    char *out = cells + line * kLineBytes + col * 8;
    if (kHalf) {
        half4_t h;
        h.x = to_half(at(3 * b2)); h.y = to_half(at(3 * b2 + 1));
        h.z = to_half(at(3 * b2 + 2)); h.w = to_half(at(3 * b2 + 3));
        *reinterpret_cast<half4_t *>(out) = h;
    } else {
        *reinterpret_cast<float2 *>(out) = make_float2(at(b2), at(b2 + 1));
    }
}

__global__ __launch_bounds__(256) void fill_u8_kernel(uint8_t *dst, uint8_t value, int64_t n) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) dst[k] = value;
}

// Two float arrays copied in one launch (a context's or a scene's pair of maps), 16
// bytes per lane where both ends are aligned for it (kVec), else 4. Bound by memory
// bandwidth at large maps and by the launch at small ones, where one launch replaces
// two device-to-device copies (a blend of 1001 probes x 80 rays and its maps read back:
// 37.7 us with the copies, 36.3 with this).
template <bool kVec>
__global__ __launch_bounds__(256) void copy_pair_kernel(float *d0, const float *s0, int64_t n0,
                                                        float *d1, const float *s1, int64_t n1) {
    constexpr int kW = kVec ? 4 : 1;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t m0 = n0 / kW, m1 = n1 / kW;
    for (int64_t e = first; e < m0 + m1; e += stride) {
        const bool one = e >= m0;
        float *d = one ? d1 : d0;
        const float *s = one ? s1 : s0;
        const int64_t k = one ? e - m0 : e;
        if (kVec) reinterpret_cast<float4 *>(d)[k] = reinterpret_cast<const float4 *>(s)[k];
        else d[k] = s[k];
    }
    if (kVec && first < 8) {    // up to three floats past the last whole vector of each
        const int64_t k = first & 3;
        if (first < 4 && 4 * m0 + k < n0) d0[4 * m0 + k] = s0[4 * m0 + k];
        if (first >= 4 && 4 * m1 + k < n1) d1[4 * m1 + k] = s1[4 * m1 + k];
    }
}

// ------------------------------------------------------------ launchers -----

static unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

hipError_t launch_tables(const TableArgs &a, hipStream_t s) {
    TableArgs t = a;
    t.row0 = 0;
    hipLaunchKernelGGL(tables_kernel, dim3(t.Ti + t.Td + 1), dim3(256), 0, s, t);
    return hipGetLastError();
}

hipError_t launch_tables_dirs(TableArgs a, hipStream_t s) {
    a.row0 = a.Ti + a.Td;
    hipLaunchKernelGGL(tables_kernel, dim3(1), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_tables_weights(TableArgs a, hipStream_t s) {
    a.row0 = 0;
    hipLaunchKernelGGL(tables_kernel, dim3(a.Ti + a.Td), dim3(256), 0, s, a);
    return hipGetLastError();
}

// Persistent grids: as many 256-thread blocks as fit on the device at once, at most
// max_per_cu per compute unit (fewer when there are fewer rays). A block is one wave
// per SIMD.
static int persistent_blocks(const void *kernel, int device, int64_t rays, int max_per_cu,
                             size_t lds) {
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, lds) != hipSuccess)
        per_cu = 1;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess)
        cus = 1;
    per_cu = std::max(1, std::min(per_cu, max_per_cu));
    const int64_t resident = (int64_t)per_cu * (cus > 0 ? cus : 1);
    const int64_t needed = blocks_for(rays, 256);
    return (int)(needed < resident ? needed : resident);
}

// The trace kernels are bound by how often the SDF lines of the rays in flight are
// found in the L2 (each XCD's 4 MB serves its own CUs): more resident waves hide more
// latency but evict each other's lines. Measured on the open scene at 16384 x 256
// rays, alone: the primary trace with 2, 3, 4, 5, 6, 7 blocks per CU 493, 436, 432, 468,
// 494, 502 us in binary32 and 481, 379, 358, 374, 394, 413 in binary16; the hit shading
// with 1, 2, 3, 4 162, 144, 155, 166 us. Beside the other frames' work (four frames and
// their maps): primary 3 and 4 blocks 2.65 and 2.77 ms in binary32, 2.23 and 2.23 in
// binary16; hit shading 1, 2, 3 blocks 2.77, 2.79, 2.93 ms. The trace of primitives needs
// no lines: 2, 3, 4, 5 blocks 388, 372, 341, 337 us a frame (16384 x 64).
constexpr int kPrimaryBlocksPerCu = 4;
constexpr int kPrimaryBlocksPerCuOverlapped[2] = {3, 4};  // binary32 SDF; binary16, primitives
constexpr int kHitsBlocksPerCu = 2;
constexpr int kHitsBlocksPerCuOverlapped = 1;

TraceGrid trace_grid(int device, int64_t rays, bool half, int analytic_prims) {
    TraceGrid g;
    const bool analytic = analytic_prims > 0;
    const size_t lds = analytic_prims * sizeof(AnalyticPrim);
    const void *pk = analytic ? (const void *)primary_kernel<kSdfAnalytic>
                     : half   ? (const void *)primary_kernel<kSdfGrid16>
                              : (const void *)primary_kernel<kSdfGrid32>;
    g.primary_blocks = persistent_blocks(pk, device, rays, kPrimaryBlocksPerCu, lds);
    g.primary_blocks_overlapped =
        persistent_blocks(pk, device, rays, kPrimaryBlocksPerCuOverlapped[half || analytic ? 1 : 0], lds);
    const void *hk = analytic ? (const void *)hits_kernel<kSdfAnalytic>
                     : half   ? (const void *)hits_kernel<kSdfGrid16>
                              : (const void *)hits_kernel<kSdfGrid32>;
    g.hits_blocks = persistent_blocks(hk, device, rays, kHitsBlocksPerCu, lds);
    g.hits_blocks_overlapped = persistent_blocks(hk, device, rays, kHitsBlocksPerCuOverlapped, lds);
    return g;
}

// The kernel of a context's distance backend.
#define SDFDDGI_LAUNCH_TRACE(kernel, blocks)                                                       \
    do {                                                                                           \
        if (a.analytic)                                                                            \
            hipLaunchKernelGGL(kernel<kSdfAnalytic>, dim3(blocks), dim3(256),                      \
                               a.an.nprims * sizeof(AnalyticPrim), s, a);                          \
        else if (a.half_sdf && a.wide)                                                             \
            hipLaunchKernelGGL(HIP_KERNEL_NAME(kernel<kSdfGrid16, true>), dim3(blocks), dim3(256), \
                               0, s, a);                                                           \
        else if (a.half_sdf)                                                                       \
            hipLaunchKernelGGL(kernel<kSdfGrid16>, dim3(blocks), dim3(256), 0, s, a);              \
        else if (a.wide)                                                                           \
            hipLaunchKernelGGL(HIP_KERNEL_NAME(kernel<kSdfGrid32, true>), dim3(blocks), dim3(256), \
                               0, s, a);                                                           \
        else                                                                                       \
            hipLaunchKernelGGL(kernel<kSdfGrid32>, dim3(blocks), dim3(256), 0, s, a);              \
    } while (0)

hipError_t launch_primary(const TraceArgs &a, const TraceGrid &g, hipStream_t s) {
    if ((int64_t)a.P * a.R == 0) return hipSuccess;
    SDFDDGI_LAUNCH_TRACE(primary_kernel, g.primary_blocks);
    return hipGetLastError();
}

hipError_t launch_hits(const TraceArgs &a, const TraceGrid &g, hipStream_t s) {
    if ((int64_t)a.P * a.R == 0) return hipSuccess;
    SDFDDGI_LAUNCH_TRACE(hits_kernel, g.hits_blocks);
    return hipGetLastError();
}

hipError_t launch_shade(const TraceArgs &a, hipStream_t s) {
    if ((int64_t)a.P * a.R == 0) return hipSuccess;
    const int64_t threads = (int64_t)a.P * a.R;
    // four workgroups per CU of the 256-CU part, striding over the queue
    const int blocks = (int)std::min<int64_t>((threads + 255) / 256, 1024);
    hipLaunchKernelGGL(shade_kernel, dim3(blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <int kMaps, int kP>
static hipError_t launch_blend_tile(const BlendArgs &a, hipStream_t s) {
    const dim3 grid(blocks_for(a.P, kP)), block(256);
    if (a.w16_i)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(blend16_kernel<kMaps, kP>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(blend_kernel<kMaps, kP>), grid, block, 0, s, a);
    return hipGetLastError();
}

// Probes per workgroup: 8, or 4 while 8 leave CUs of the 256-CU part without work. Tables,
// blend and a copy of the maps, FP32 / precision form, with 16, 8 and 4 probes: at 1001
// probes of 6x6 + 12x12 texels and 80 rays 23.9, 20.1, 17.7 / 25.3, 22.2, 20.1 us; 8x8 +
// 16x16, 144 rays at 1000 probes 29.2, 22.5, 20.7 / 28.9, 20.4, 20.7 and at 4096 36.2, 31.0,
// 35.3; 256 rays at 8192 60.1, 59.0, 82.7 / 51.6, 38.7, 54.5 and at 16384 104, 108, 144 /
// 97.4, 70.7, 84.8 (a workgroup of 4 wastes 1/4 of its irradiance and half of its depth
// products; one of 16 leaves fewer to overlap).
hipError_t launch_blend(const BlendArgs &a, hipStream_t s) {
    const bool small = a.P < 8 * 256;
    if (blend_passes(a.irr_res, a.depth_res) > 1) return launch_blend_tile<kLargeMaps, 8>(a, s);
    if (a.irr_res == 8 && a.depth_res == 16)
        return small ? launch_blend_tile<kStdMaps, 4>(a, s) : launch_blend_tile<kStdMaps, 8>(a, s);
    return small ? launch_blend_tile<kSmallMaps, 4>(a, s) : launch_blend_tile<kSmallMaps, 8>(a, s);
}

hipError_t launch_relocate(const TraceArgs &a, const RelocateArgs &r, hipStream_t s) {
    if (a.half_sdf)
        hipLaunchKernelGGL(relocate_kernel<true>, dim3(blocks_for(a.P, 256)), dim3(256), 0, s, a, r);
    else
        hipLaunchKernelGGL(relocate_kernel<false>, dim3(blocks_for(a.P, 256)), dim3(256), 0, s, a, r);
    return hipGetLastError();
}

hipError_t launch_probe_sdf(const TraceArgs &a, float *out, hipStream_t s) {
    if (a.half_sdf)
        hipLaunchKernelGGL(probe_sdf_kernel<true>, dim3(blocks_for(a.P, 256)), dim3(256), 0, s, a, out);
    else
        hipLaunchKernelGGL(probe_sdf_kernel<false>, dim3(blocks_for(a.P, 256)), dim3(256), 0, s, a, out);
    return hipGetLastError();
}

hipError_t launch_probe_first(const TraceArgs &a, int2 *out, hipStream_t s) {
    if (a.analytic)
        hipLaunchKernelGGL(probe_first_analytic_kernel, dim3(blocks_for(a.P, 256)), dim3(256),
                           a.an.nprims * sizeof(AnalyticPrim), s, a, out);
    else if (a.half_sdf)
        hipLaunchKernelGGL(probe_first_kernel<true>, dim3(blocks_for(a.P, 256)), dim3(256), 0, s, a,
                           out);
    else
        hipLaunchKernelGGL(probe_first_kernel<false>, dim3(blocks_for(a.P, 256)), dim3(256), 0, s,
                           a, out);
    return hipGetLastError();
}

hipError_t launch_sample(const SampleArgs &a, hipStream_t s) {
    if (a.n == 0) return hipSuccess;
    hipLaunchKernelGGL(sample_kernel, dim3(blocks_for(a.n, 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

CellShape cell_shape(int n0, int n1, int n2, bool half) {
    CellShape s{};
    s.nb0 = (uint32_t)(n0 - 1 + 2) / 3;
    s.nb1 = (uint32_t)(n1 - 1 + 2) / 3;
    s.nb2 = half ? (uint32_t)(n2 - 1 + 2) / 3 : (uint32_t)(n2 - 1);
    s.wide = n0 > 65536 || n1 > 65536 || n2 > 65536 || (int64_t)s.nb2 * s.nb1 >= (int64_t)1 << 24;
    return s;
}

hipError_t launch_pack_cells(const float *g, int n0, int n1, int n2, bool half, char *cells,
                             hipStream_t s) {
    const CellShape sh = cell_shape(n0, n1, n2, half);
    const unsigned blocks = blocks_for(sh.lines() * 16, 256);
    if (half)
        hipLaunchKernelGGL(pack_cells_kernel<true>, dim3(blocks), dim3(256), 0, s, g, n0, n1, n2, sh,
                           cells);
    else
        hipLaunchKernelGGL(pack_cells_kernel<false>, dim3(blocks), dim3(256), 0, s, g, n0, n1, n2,
                           sh, cells);
    return hipGetLastError();
}

hipError_t launch_fill_u8(uint8_t *dst, uint8_t value, int64_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u8_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, dst, value, n);
    return hipGetLastError();
}

hipError_t launch_copy_pair(float *d0, const float *s0, int64_t n0, float *d1, const float *s1,
                            int64_t n1, hipStream_t s) {
    if (n0 + n1 <= 0) return hipSuccess;
    const auto bits = [](const void *p, int64_t n) { return n > 0 ? (uintptr_t)p : (uintptr_t)0; };
    const bool vec = ((bits(d0, n0) | bits(s0, n0) | bits(d1, n1) | bits(s1, n1)) & 15) == 0;
    const int64_t work = vec ? (n0 + n1 + 3) / 4 : n0 + n1;
    // eight blocks per CU of the 256-CU part, striding
    const unsigned blocks = (unsigned)std::min<int64_t>((work + 255) / 256, 2048);
    if (vec)
        hipLaunchKernelGGL(copy_pair_kernel<true>, dim3(blocks), dim3(256), 0, s, d0, s0, n0, d1,
                           s1, n1);
    else
        hipLaunchKernelGGL(copy_pair_kernel<false>, dim3(blocks), dim3(256), 0, s, d0, s0, n0, d1,
                           s1, n1);
    return hipGetLastError();
}

}  // namespace sdfddgi
