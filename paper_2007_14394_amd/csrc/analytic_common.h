// Device code of the analytic-primitive SDF query of Sec. 3.3: the cluster walk of the
// standalone query and trace kernels (cluster.hip), and the candidate cells that answer it
// in the probe update's trace kernels when a context traces the primitives instead of a
// grid (kernels.hip).
// Primitives are packed into clusters; a cluster's primitives are visited only
// when the signed distance to its bounding box is below the best distance so far,
// and along a sphere-traced ray the best distance starts from the bound the
// previous sample gives (the paper's 2 lastSDF) instead of infinity. Distances are
// binary32 in one fixed sequence; the culled minimum equals the minimum over every
// primitive bit for bit (a minimum is exact, and every culling test compares a
// lower bound of a cluster's distances, widened beyond rounding, against an upper
// bound of the scene's).
#pragma once

#include "internal.h"
#include "trace_common.h"

namespace sdfddgi {

__device__ __forceinline__ float prim_distance32(int kind, const float *c, const float *h,
                                                 float x0, float x1, float x2) {
    const float dx = x0 - c[0], dy = x1 - c[1], dz = x2 - c[2];
    if (kind == 0) return sqrtf(fmaf(dz, dz, fmaf(dy, dy, dx * dx))) - h[0];
    const float qx = fabsf(dx) - h[0], qy = fabsf(dy) - h[1], qz = fabsf(dz) - h[2];
    const float ox = fmaxf(qx, 0.0f), oy = fmaxf(qy, 0.0f), oz = fmaxf(qz, 0.0f);
    const float outside = sqrtf(fmaf(oz, oz, fmaf(oy, oy, ox * ox)));
    const float inside = fminf(fmaxf(qx, fmaxf(qy, qz)), 0.0f);
    return outside + inside;
}

// Signed distance to an axis-aligned box given by its corners.
__device__ __forceinline__ float box_distance32(const float *lo, const float *hi, float x0,
                                                float x1, float x2) {
    const float qx = fmaxf(lo[0] - x0, x0 - hi[0]);
    const float qy = fmaxf(lo[1] - x1, x1 - hi[1]);
    const float qz = fmaxf(lo[2] - x2, x2 - hi[2]);
    const float ox = fmaxf(qx, 0.0f), oy = fmaxf(qy, 0.0f), oz = fmaxf(qz, 0.0f);
    return sqrtf(fmaf(oz, oz, fmaf(oy, oy, ox * ox))) + fminf(fmaxf(qx, fmaxf(qy, qz)), 0.0f);
}

struct ClusterLds {
    int kind[kMaxAnalyticPrims];
    float cen[kMaxAnalyticPrims][3], hal[kMaxAnalyticPrims][3];
    float lo[kMaxClusters][3], hi[kMaxClusters][3];
    int first[kMaxClusters + 1];
};

__device__ __forceinline__ void load_clusters(const AnalyticArgs &a, ClusterLds &s) {
    for (int e = threadIdx.x; e < a.nprims; e += blockDim.x) {
        s.kind[e] = a.kind[e];
        for (int c = 0; c < 3; ++c) {
            s.cen[e][c] = a.center[3 * e + c];
            s.hal[e][c] = a.half[3 * e + c];
        }
    }
    for (int e = threadIdx.x; e < a.nclusters; e += blockDim.x)
        for (int c = 0; c < 3; ++c) {
            s.lo[e][c] = a.lo[3 * e + c];
            s.hi[e][c] = a.hi[3 * e + c];
        }
    for (int e = threadIdx.x; e <= a.nclusters; e += blockDim.x) s.first[e] = a.first[e];
    __syncthreads();
}

// The scene distance at x: mode 0 every primitive; otherwise the cluster walk from
// the bound d_init (+inf, or the previous sample's bound along a ray).
__device__ __forceinline__ float scene_distance(const AnalyticArgs &a, const ClusterLds &s,
                                                int mode, float x0, float x1, float x2,
                                                float d_init, uint32_t &evals) {
    if (mode == 0) {
        float best = INFINITY;
        for (int m = 0; m < a.nprims; ++m)
            best = fminf(best, prim_distance32(s.kind[m], s.cen[m], s.hal[m], x0, x1, x2));
        evals += (uint32_t)a.nprims;
        return best;
    }
    float D = d_init;
    for (int c = 0; c < a.nclusters; ++c) {
        if (!(box_distance32(s.lo[c], s.hi[c], x0, x1, x2) < D)) continue;
        for (int m = s.first[c]; m < s.first[c + 1]; ++m)
            D = fminf(D, prim_distance32(s.kind[m], s.cen[m], s.hal[m], x0, x1, x2));
        evals += (uint32_t)(s.first[c + 1] - s.first[c]);
    }
    return D;
}

// The same operations on a packed primitive, one sequence for both kinds: a sphere is a
// box of no extent, whose terms reproduce sqrt(|x - c|^2) bit for bit, less its radius.
__device__ __forceinline__ float prim_distance(const AnalyticPrim &p, float x0, float x1,
                                               float x2) {
    const float qx = fabsf(x0 - p.c.x) - p.h.x, qy = fabsf(x1 - p.c.y) - p.h.y;
    const float qz = fabsf(x2 - p.c.z) - p.h.z;
    const float ox = fmaxf(qx, 0.0f), oy = fmaxf(qy, 0.0f), oz = fmaxf(qz, 0.0f);
    const float outside = sqrtf(fmaf(oz, oz, fmaf(oy, oy, ox * ox)));
    const float inside = fminf(fmaxf(qx, fmaxf(qy, qz)), 0.0f);
    return (outside + inside) - p.c.w;
}

// The primitives of a trace kernel's scene, in its dynamic LDS.
__device__ __forceinline__ AnalyticPrim *lds_prims() {
    extern __shared__ AnalyticPrim s_prims[];
    return s_prims;
}

__device__ __forceinline__ void load_prims(const AnalyticScene &a, float4 *s_lv) {
    AnalyticPrim *s = lds_prims();
    for (int e = threadIdx.x; e < a.nprims; e += blockDim.x) s[e] = a.prims[e];
    if ((int)threadIdx.x < a.nlevels) s_lv[threadIdx.x] = a.lv[threadIdx.x];
    __syncthreads();
}

// The minimum D so far and, when kName, the primitive at it (as 32 x its slot): of those
// at the minimum the one of lowest caller index.
struct Nearest {
    float D;
    int key;
    uint32_t at;
};

template <bool kName>
__device__ __forceinline__ void visit(Nearest &b, uint32_t at, float x0, float x1, float x2) {
    const AnalyticPrim p = *(const AnalyticPrim *)((const char *)lds_prims() + at);
    const float d = prim_distance(p, x0, x1, x2);
    if (kName) {
        const int key = __float_as_int(p.h.w);
        const bool nearer = (d < b.D) | ((d == b.D) & (key < b.key));
        b.key = nearer ? key : b.key;
        b.at = nearer ? at : b.at;
    }
    b.D = fminf(b.D, d);
}

// Eight candidates, each in 16 bits as 32 x its slot (flags in the low bits of the first),
// the last one repeated to the end of the list.
template <bool kName>
__device__ __forceinline__ void visit8(Nearest &b, const uint4 &w, float x0, float x1, float x2) {
    const uint32_t v[4] = {w.x, w.y, w.z, w.w};
    uint32_t last = v[0] & 0xffe0u;
    visit<kName>(b, last, x0, x1, x2);
#pragma unroll
    for (int j = 1; j < 8; ++j) {
        const uint32_t at = j & 1 ? v[j / 2] >> 16 : v[j / 2] & 0xffffu;
        if (!__ballot(at != last)) break;   // every lane's list has ended
        visit<kName>(b, at, x0, x1, x2);
        last = at;
    }
}

// The scene distance at x, from an upper bound of it (+inf, or the previous sample's
// along a ray), and the nearest primitive's slot when kName. x's cell lists every
// primitive that can be the nearest somewhere in it, so the minimum over the list is the
// minimum over the scene, bit for bit, and holds every primitive at that minimum. Points
// outside the levels and cells of more than kCellPrims candidates walk the clusters
// against the best distance so far (their boxes are widened, so that a primitive at the
// minimum lies in a cluster strictly below it).
// Bound by the vector instructions of the candidates' distances and the latency of the
// list's read: at 16384 x 64 rays among 400 primitives (1.6 to 2.3 candidates a cell on
// average, three visits a wave) the primary trace takes 252 us and the hits' shadow rays
// 106, where walking 50 clusters per sample took 9.8 and 2.35 ms. Probe by probe a wave's
// lanes read few lines; 64 probes' rays of one direction side by side, which the cluster
// walk preferred, took 495 us. Reading a candidate while the last is evaluated: no gain.
template <bool kName>
__device__ __forceinline__ float analytic_distance(const AnalyticScene &a, const float4 *s_lv,
                                                   float x0, float x1, float x2, float bound,
                                                   int &slot) {
    const float u0 = (x0 - a.mid0) * a.inv, u1 = (x1 - a.mid1) * a.inv;
    const float u2 = (x2 - a.mid2) * a.inv;
    // how far x lies beyond level 0's box: level l's margin is kCellMargin 2^l
    const float e = fmaxf(fabsf(u0) - a.half0, fmaxf(fabsf(u1) - a.half1, fabsf(u2) - a.half2));
    const bool listed = e < a.beyond;
    const int out = max(__builtin_amdgcn_frexp_expf(e * (1.0f / kCellMargin)), 1);
    const int l = listed && e >= 0.0f ? out : 0;
    const float4 d = s_lv[l];
    const float i0 = floorf(ldexpf(u0, -l) + d.x), i1 = floorf(ldexpf(u1, -l) + d.y);
    const float i2 = floorf(ldexpf(u2, -l) + d.z);
    // exact: below 2^24 cells
    const float in_level = fmaf(fmaf(i2, d.y + d.y, i1), d.x + d.x, i0);
    const uint32_t line = listed ? (uint32_t)in_level + __float_as_uint(d.w) : 0u;
    const auto *list = (const __attribute__((address_space(1))) uint4 *)(
        (GlobalBytes)a.cells + line * (uint32_t)kCellPrims);
    const uint4 w = {list->x, list->y, list->z, list->w};
    Nearest b{bound, 0x7fffffff, 0u};
    visit8<kName>(b, w, x0, x1, x2);
    if (w.x & 1u) {
        const auto *rest = list + (uint32_t)a.ncells;
        const uint4 v = {rest->x, rest->y, rest->z, rest->w};
        visit8<kName>(b, v, x0, x1, x2);
    }
    if ((w.x & 2u) || !listed) {
        for (int c = 0; c < a.nclusters; ++c) {
            if (!(box_distance32(a.lo + 3 * c, a.hi + 3 * c, x0, x1, x2) < b.D)) continue;
            for (int k = a.first[c]; k < a.first[c + 1]; ++k)
                visit<kName>(b, 32u * (uint32_t)k, x0, x1, x2);
        }
    }
    slot = (int)(b.at >> 5);
    return b.D;
}

// The bound on the next sample's distance from the previous one d: the scene
// distance is 1-Lipschitz and the ray moved relax * d, so it is at most
// (1 + relax) d (the paper's 2 lastSDF for relax = 1); widened by 2^-10
// relative and 1e-4 m so that it stays a bound under binary32 rounding.
__device__ __forceinline__ float next_bound(float relax, float d) {
    return fmaf((1.0f + relax) * d, 1.0009765625f, 1.0e-4f);
}

// Normal at x from the gradient of the distance of primitive slot m: a sphere's
// radial direction x - c; outside a box the offset from its nearest point, inside
// it the signed axis of the face nearest to x (the largest q, lowest axis on a
// tie); normalised like the grid normal, -w where the gradient vanishes.
__device__ __forceinline__ void analytic_normal(int m, float x0, float x1, float x2, float w0,
                                                float w1, float w2, float &n0, float &n1,
                                                float &n2) {
    const AnalyticPrim p = lds_prims()[m];
    const float d[3] = {x0 - p.c.x, x1 - p.c.y, x2 - p.c.z}, hal[3] = {p.h.x, p.h.y, p.h.z};
    float g[3] = {0.0f, 0.0f, 0.0f};
    if (!(__float_as_int(p.h.w) & 1)) {
        g[0] = d[0]; g[1] = d[1]; g[2] = d[2];
    } else {
        float q[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) q[k] = fabsf(d[k]) - hal[k];
        const float qm = fmaxf(q[0], fmaxf(q[1], q[2]));
        if (qm > 0.0f) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const float o = fmaxf(q[k], 0.0f);
                g[k] = d[k] >= 0.0f ? o : -o;
            }
        } else {
            const int ax = q[0] >= q[1] ? (q[0] >= q[2] ? 0 : 2) : (q[1] >= q[2] ? 1 : 2);
            g[ax] = d[ax] >= 0.0f ? 1.0f : -1.0f;
        }
    }
    const float len2 = fmaf(g[2], g[2], fmaf(g[1], g[1], g[0] * g[0]));
    if (!(len2 >= 1e-24f)) { n0 = -w0; n1 = -w1; n2 = -w2; return; }
    const float inv = 1.0f / sqrtf(len2);
    n0 = g[0] * inv; n1 = g[1] * inv; n2 = g[2] * inv;
}

}  // namespace sdfddgi
