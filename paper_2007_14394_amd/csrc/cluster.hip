// gfx950 kernels of the analytic-primitive SDF query of Sec. 3.3 on their own
// (the cluster walk itself is in analytic_common.h):
//
//   cluster_query_kernel  one distance per point
//   cluster_trace_kernel  one sphere-traced ray per thread
//
// and the set-up of the probe update's candidate cells:
//
//   candidate_cells_kernel  the primitives that can be the nearest within each cell
#include "internal.h"
#include "analytic_common.h"

#pragma clang fp contract(off)

namespace sdfddgi {

__global__ __launch_bounds__(256) void cluster_query_kernel(AnalyticArgs a, const float *pts,
                                                            int n, int mode, float *out,
                                                            unsigned long long *evals) {
    __shared__ ClusterLds s;
    load_clusters(a, s);
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t ev = 0;
    if (q < n)
        out[q] = scene_distance(a, s, mode, pts[3 * q], pts[3 * q + 1], pts[3 * q + 2], INFINITY,
                                ev);
    if (evals && ev) atomicAdd(evals, (unsigned long long)ev);
}

__global__ __launch_bounds__(256) void cluster_trace_kernel(AnalyticArgs a, AnalyticTrace r) {
    __shared__ ClusterLds s;
    load_clusters(a, s);
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t ev = 0;
    if (q < r.n) {
        const float o0 = r.o[3 * q], o1 = r.o[3 * q + 1], o2 = r.o[3 * q + 2];
        const float w0 = r.w[3 * q], w1 = r.w[3 * q + 1], w2 = r.w[3 * q + 2];
        float t = 0.0f, bound = INFINITY;
        int k = 0, kind = -1, steps = 0;
        while (kind < 0) {
            if (t > r.t_max) { kind = 0; steps = k; break; }
            const float x0 = fmaf(t, w0, o0), x1 = fmaf(t, w1, o1), x2 = fmaf(t, w2, o2);
            const float d = scene_distance(a, s, r.mode, x0, x1, x2, r.mode == 2 ? bound : INFINITY,
                                           ev);
            if (k == 0 && d < 0.0f) { kind = 4; steps = 1; break; }
            if (d < r.eps) { kind = 2; steps = k + 1; break; }
            t = fmaf(r.relax, d, t);
            bound = next_bound(r.relax, d);
            ++k;
            if (k == r.max_steps) { kind = 3; steps = k; break; }
        }
        r.t_out[q] = t;
        r.steps_out[q] = steps;
        r.kind_out[q] = kind;
    }
    if (r.evals && ev) atomicAdd(r.evals, (unsigned long long)ev);
}

// A packed primitive's distance at x, and its direction: the unit gradient outside its
// core (a sphere's centre, a box), at distance `out` of it.
struct Slope {
    float d, out, g0, g1, g2;
};
__device__ __forceinline__ Slope slope_at(const AnalyticPrim &p, float x0, float x1, float x2) {
    const float d0 = x0 - p.c.x, d1 = x1 - p.c.y, d2 = x2 - p.c.z;
    const float o0 = copysignf(fmaxf(fabsf(d0) - p.h.x, 0.0f), d0);
    const float o1 = copysignf(fmaxf(fabsf(d1) - p.h.y, 0.0f), d1);
    const float o2 = copysignf(fmaxf(fabsf(d2) - p.h.z, 0.0f), d2);
    Slope s;
    s.d = prim_distance(p, x0, x1, x2);
    s.out = sqrtf(fmaf(o2, o2, fmaf(o1, o1, o0 * o0)));
    const float inv = 1.0f / fmaxf(s.out, 1e-30f);
    s.g0 = o0 * inv; s.g1 = o1 * inv; s.g2 = o2 * inv;
    return s;
}

// One wave per cell. Within a ball of radius r about q a primitive m can be nearer than b
// only if d_m(q) - d_b(q) <= r L, L a Lipschitz constant of d_m - d_b there: 2 always, as
// each distance has slope 1; and, outside both cores, |g_m - g_b| at q plus what either
// direction turns over the ball, at most r / (its core's distance - r). With b the nearest
// at q, the cell's own ball (L = 2) selects a first list from all primitives, and the
// balls of its 4 x 4 x 4 parts, one per lane, the candidates from that list. Far from the
// scene the directions are what tells the primitives apart: at 400 primitives the cells of
// levels 0, 1, 3 and 5 hold 1.8, 1.7, 1.9 and 2.8 candidates on average; with L = 2 alone
// 1.9, 2.4, 8.8 and 71. Radii and thresholds are widened by 1e-5 of the largest coordinate
// in reach, some 40 roundings of a binary32 distance or lookup.
__global__ __launch_bounds__(256) void candidate_cells_kernel(AnalyticScene a, uint16_t *out) {
    __shared__ uint16_t s_list[4][kMaxAnalyticPrims];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int id = blockIdx.x * 4 + wave;
    if (id >= a.ncells) return;
    uint16_t *list = s_list[wave];
    int l = 0;
    while (l + 1 < a.nlevels && id >= __float_as_int(a.lv[l + 1].w)) ++l;
    const float4 lv = a.lv[l];
    const int n0 = 2 * (int)lv.x, n1 = 2 * (int)lv.y;
    int c = id - __float_as_int(lv.w);
    const int i0 = c % n0; c /= n0;
    const int i1 = c % n1, i2 = c / n1;
    const float side = ldexpf(a.cell, l), quarter = 0.25f * side;
    const float far = fmaxf(fabsf(a.mid0), fmaxf(fabsf(a.mid1), fabsf(a.mid2))) +
                      side * fmaxf(lv.x, fmaxf(lv.y, lv.z));
    const float slack = 1e-5f * (far + a.reach);
    const float x0 = fmaf((float)i0 - lv.x, side, a.mid0);   // lowest corner
    const float x1 = fmaf((float)i1 - lv.y, side, a.mid1);
    const float x2 = fmaf((float)i2 - lv.z, side, a.mid2);
    // radii of the cell and of its parts; half the diagonal of a unit cube is below 0.8661
    const float r = fmaf(0.8661f, side, slack), rp = fmaf(0.8661f, quarter, slack);

    const float h = 0.5f * side;
    float best = INFINITY;
    for (int m = lane; m < a.nprims; m += 64)
        best = fminf(best, prim_distance(a.prims[m], x0 + h, x1 + h, x2 + h));
    for (int o = 32; o > 0; o >>= 1) best = fminf(best, __shfl_xor(best, o));
    int count = 0;
    for (int base = 0; base < a.nprims; base += 64) {
        const int m = base + lane;
        const bool near = m < a.nprims && prim_distance(a.prims[m], x0 + h, x1 + h, x2 + h) <=
                                              best + (2.0f * r + slack);
        const uint64_t any = __ballot(near);
        if (near) list[count + __popcll(any & ((1ull << lane) - 1))] = (uint16_t)m;
        count += __popcll(any);
    }
    __builtin_amdgcn_wave_barrier();

    const float q0 = fmaf((float)(lane & 3) + 0.5f, quarter, x0);
    const float q1 = fmaf((float)((lane >> 2) & 3) + 0.5f, quarter, x1);
    const float q2 = fmaf((float)(lane >> 4) + 0.5f, quarter, x2);
    float nearest = INFINITY;
    int at = -1;
    for (int j = 0; j < count; ++j) {
        const float d = prim_distance(a.prims[list[j]], q0, q1, q2);
        if (d < nearest) { nearest = d; at = list[j]; }
    }
    Slope b;
    b.d = INFINITY; b.out = 0.0f; b.g0 = b.g1 = b.g2 = 0.0f;
    if (at >= 0) b = slope_at(a.prims[at], q0, q1, q2);
    int n = 0;
    uint32_t entry = 0;
    for (int j = 0; j < count; ++j) {
        const int m = list[j];
        const Slope s = slope_at(a.prims[m], q0, q1, q2);
        float L = 2.0f;
        if (fminf(s.out, b.out) > 1.01f * rp) {
            const float e0 = s.g0 - b.g0, e1 = s.g1 - b.g1, e2 = s.g2 - b.g2;
            const float apart = sqrtf(fmaf(e2, e2, fmaf(e1, e1, e0 * e0)));
            // and the rounding of the directions
            const float turn = rp / (s.out - rp) + rp / (b.out - rp) + 0.1f * slack / rp + 1e-3f;
            L = fminf(L, apart + turn);
        }
        // (not "<=": what is undefined stays listed)
        if (!__ballot(!(s.d > b.d + (L * rp + slack)))) continue;
        if (lane == n) entry = 32u * (uint32_t)m;
        if (++n > kCellPrims) break;   // (the cell walks the clusters)
    }
    entry = __shfl(entry, min(lane, max(min(n, kCellPrims) - 1, 0)));
    if (lane == 0) entry |= (n > 8 ? 1u : 0u) | (n > kCellPrims || n == 0 ? 2u : 0u);
    // the first halves of all lists before the second: few cells have more than eight
    if (lane < kCellPrims)
        out[((size_t)(lane >> 3) * a.ncells + id) * 8 + (lane & 7)] = (uint16_t)entry;
}

hipError_t launch_candidate_cells(const AnalyticScene &a, uint16_t *cells, hipStream_t s) {
    hipLaunchKernelGGL(candidate_cells_kernel, dim3((unsigned)((a.ncells + 3) / 4)), dim3(256), 0,
                       s, a, cells);
    return hipGetLastError();
}

hipError_t launch_cluster_query(const AnalyticArgs &a, const float *pts, int n, int mode,
                                float *out, unsigned long long *evals, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(cluster_query_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a,
                       pts, n, mode, out, evals);
    return hipGetLastError();
}

hipError_t launch_cluster_trace(const AnalyticArgs &a, const AnalyticTrace &r, hipStream_t s) {
    if (r.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(cluster_trace_kernel, dim3((unsigned)((r.n + 255) / 256)), dim3(256), 0, s,
                       a, r);
    return hipGetLastError();
}

}  // namespace sdfddgi
