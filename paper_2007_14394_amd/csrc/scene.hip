// Device baker of scene distance grids: the exact signed distance of a union of
// spheres and axis-aligned boxes at the vertices of a vertex-centred grid, with the
// albedo of the nearest primitive. Input preparation (the probe update consumes
// a baked grid); it lets the learned form's training generate thousands of scenes
// on the GPU. Distances are evaluated in binary64 and rounded once to binary32,
// ties in the nearest primitive go to the lower index.
#include <algorithm>

#include "internal.h"

#pragma clang fp contract(off)

namespace sdfddgi {

constexpr int kPrimChunk = 256;   // primitives staged in LDS at a time

__device__ __forceinline__ double prim_distance(int kind, const double *c, const double *h,
                                                double px, double py, double pz) {
    const double dx = px - c[0], dy = py - c[1], dz = pz - c[2];
    if (kind == 0) return sqrt(dx * dx + dy * dy + dz * dz) - h[0];
    // box: Euclidean distance outside plus the (negative) largest axis excess inside
    const double qx = fabs(dx) - h[0], qy = fabs(dy) - h[1], qz = fabs(dz) - h[2];
    const double ox = qx > 0 ? qx : 0, oy = qy > 0 ? qy : 0, oz = qz > 0 ? qz : 0;
    const double outside = sqrt(ox * ox + oy * oy + oz * oz);
    double m = qx > qy ? qx : qy;
    m = m > qz ? m : qz;
    const double inside = m < 0 ? m : 0;
    return outside + inside;
}

// One workgroup per brick of 256 vertices (2^s0 x 2^s1 x 2^s2), one thread per vertex.
// Distances are 1-Lipschitz, so with r the distance from the brick's centre to
// its corners a primitive at d from the centre is within [d - r, d + r] at every vertex:
// the workgroup first takes the least d + r over the primitives, then stages only the
// primitives whose d - r does not exceed it, in index order, and every vertex evaluates
// those. Both bounds are widened far beyond binary64 rounding (and a primitive whose
// distance is not a finite number is always staged), so the values and the nearest
// primitive are those of evaluating every primitive. The kernel is bound by binary64
// arithmetic: 128^3 vertices x 400 primitives took 1050 us with every primitive
// evaluated at every vertex, 66 us so. A brick is 16 x 4 x 4 (16 in x for whole 64-byte
// stores) unless the grid is thinner than that.

// A primitive's distance from the brick's centre and the slack of both its bounds.
__device__ __forceinline__ double brick_distance(const BakeArgs &a, int m, const double *bc,
                                                 double &slack) {
    const double *c = a.center + 3 * (size_t)m, *h = a.half + 3 * (size_t)m;
    slack = 1e-150;
    for (int k = 0; k < 3; ++k) slack += 1e-10 * (fabs(bc[k]) + fabs(c[k]) + fabs(h[k]));
    return prim_distance(a.kind[m], c, h, bc[0], bc[1], bc[2]);
}

__global__ __launch_bounds__(256) void bake_kernel(BakeArgs a, int s0, int s1, int64_t bricks) {
    __shared__ double s_c[kPrimChunk][3], s_h[kPrimChunk][3];
    __shared__ int s_k[kPrimChunk], s_m[kPrimChunk];
    __shared__ double s_red[4];
    __shared__ int s_cnt[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int s2 = 8 - s0 - s1;
    const int nb0 = (a.n0 + (1 << s0) - 1) >> s0, nb1 = (a.n1 + (1 << s1) - 1) >> s1;
    const double hx = 0.5 * ((1 << s0) - 1), hy = 0.5 * ((1 << s1) - 1), hz = 0.5 * ((1 << s2) - 1);
    const double r = a.spacing * sqrt(hx * hx + hy * hy + hz * hz) * (1.0 + 1e-10);
    for (int64_t brick = blockIdx.x; brick < bricks; brick += gridDim.x) {
        const int b0 = (int)(brick % nb0) << s0, b1 = (int)(brick / nb0 % nb1) << s1;
        const int b2 = (int)(brick / nb0 / nb1) << s2;
        const int i = b0 + (tid & ((1 << s0) - 1)), j = b1 + ((tid >> s0) & ((1 << s1) - 1));
        const int k = b2 + (tid >> (s0 + s1));
        const double px = a.org0 + a.spacing * i;
        const double py = a.org1 + a.spacing * j;
        const double pz = a.org2 + a.spacing * k;
        const double bc[3] = {a.org0 + a.spacing * (b0 + hx), a.org1 + a.spacing * (b1 + hy),
                              a.org2 + a.spacing * (b2 + hz)};
        // the least upper bound over the primitives
        double bound = INFINITY;
        for (int m = tid; m < a.nprims; m += 256) {
            double slack;
            const double d = brick_distance(a, m, bc, slack);
            bound = fmin(bound, d + r + slack);   // fmin passes over NaN
        }
        for (int off = 32; off > 0; off >>= 1) bound = fmin(bound, __shfl_xor(bound, off));
        if (lane == 0) s_red[wave] = bound;
        __syncthreads();
        bound = fmin(fmin(s_red[0], s_red[1]), fmin(s_red[2], s_red[3]));
        double best = INFINITY;
        int arg = -1;
        for (int m0 = 0; m0 < a.nprims; m0 += kPrimChunk) {
            const int m = m0 + tid;
            bool keep = false;
            if (m < a.nprims) {
                double slack;
                const double d = brick_distance(a, m, bc, slack);
                keep = !(d - r - slack > bound) || !isfinite(d);
            }
            const uint64_t kept = __ballot(keep);
            if (lane == 0) s_cnt[wave] = __popcll(kept);
            __syncthreads();   // and the previous chunk's primitives have been read
            int at = 0, cnt = 0;
            for (int w = 0; w < 4; ++w) {
                if (w == wave) at = cnt;
                cnt += s_cnt[w];
            }
            if (keep) {
                at += __popcll(kept & ((1ull << lane) - 1));
                s_k[at] = a.kind[m];
                s_m[at] = m;
                for (int c = 0; c < 3; ++c) {
                    s_c[at][c] = a.center[3 * (size_t)m + c];
                    s_h[at][c] = a.half[3 * (size_t)m + c];
                }
            }
            __syncthreads();
            for (int e = 0; e < cnt; ++e) {
                const double d = prim_distance(s_k[e], s_c[e], s_h[e], px, py, pz);
                if (d < best) { best = d; arg = s_m[e]; }
            }
        }
        __syncthreads();   // the staged primitives have been read
        if (i >= a.n0 || j >= a.n1 || k >= a.n2) continue;
        const int64_t v = ((int64_t)k * a.n1 + j) * a.n0 + i;
        a.sdf[v] = arg < 0 ? a.empty_value : (float)best;
        if (a.alb)
            for (int c = 0; c < 3; ++c)
                a.alb[3 * v + c] = arg < 0 ? 0.0f : (float)a.albedo[3 * (size_t)arg + c];
    }
}

hipError_t launch_bake(const BakeArgs &a, hipStream_t s) {
    // 16 x 4 x 4, an axis no longer than the grid's next power of two, what that leaves
    // to the others
    const int n[3] = {a.n0, a.n1, a.n2}, want[3] = {4, 2, 2};
    int cap[3], sh[3], left = 8;
    for (int c = 0; c < 3; ++c) {
        for (cap[c] = 0; cap[c] < 8 && (1 << cap[c]) < n[c];) ++cap[c];
        sh[c] = std::min(want[c], cap[c]);
        left -= sh[c];
    }
    for (int c = 0; c < 3; ++c) {
        const int add = std::min(left, cap[c] - sh[c]);
        sh[c] += add;
        left -= add;
    }
    sh[2] += left;
    int64_t bricks = 1;
    for (int c = 0; c < 3; ++c) bricks *= ((int64_t)n[c] + (1 << sh[c]) - 1) >> sh[c];
    const int64_t blocks = std::min<int64_t>(bricks, 1 << 22);  // x 256 threads < 2^32
    hipLaunchKernelGGL(bake_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a, sh[0], sh[1],
                       bricks);
    return hipGetLastError();
}

}  // namespace sdfddgi
