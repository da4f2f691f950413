// The Eq. 3 blend of one workgroup's probes, shared by the single-scene kernels
// (kernels.hip) and the batched ones (batch.hip).
#pragma once

#include <algorithm>

#include "internal.h"
#include "octahedral.h"

namespace sdfddgi {

constexpr int kBlendProbes = 16;  // probes per workgroup: the N extent of a tile row
typedef float floatx4 __attribute__((ext_vector_type(4)));

// The probes of one blend workgroup of kP (slots pb .. pb+np-1 of the probe list, or
// of 0..P-1) and their hysteresis: none where the history is rejected. The first
// __syncthreads of the caller's ray loop publishes them.
template <int kP = kBlendProbes>
__device__ __forceinline__ void load_blend_probes(const BlendArgs &a, int pb, int np, int *s_pid,
                                                  float *s_h) {
    const int tid = threadIdx.x;
    if (tid < kP) {
        const int pid = tid < np ? (a.probe_list ? a.probe_list[pb + tid] : pb + tid) : 0;
        s_pid[tid] = pid;
        s_h[tid] = (tid < np && !(a.reject && a.reject[pid])) ? a.hysteresis : 0.0f;
    }
}

constexpr int kBlendChunk = 64;   // rays staged in LDS at a time
// 16-texel M-tiles per wave per pass: of the irradiance map (one covers 8x8, two, for
// other resolutions, 11x11), and of the depth map (16x16)
constexpr int kIrrSlots = 1, kIrrSlotsAny = 2, kDepthSlots = 4;

// The map layouts that the blend kernels are compiled for: 8x8 irradiance and 16x16 depth
// (4 + 16 M-tiles, which fill one pass); others of one pass, whose epilogue goes through
// LDS; larger ones, pass by pass and texel by texel.
enum : int { kStdMaps = 0, kSmallMaps = 1, kLargeMaps = 2 };

// LDS floats of an epilogue through LDS: per probe and map one row of updates, of one texel
// more than the map has (which spreads the rows over the banks).
__host__ __device__ constexpr int update_row(int texels, int comps) { return (texels + 1) * comps; }
// ... of both maps per probe: 8x8 and 16x16, and the largest of one pass
constexpr int kProbeFloatsStd = update_row(64, 3) + update_row(256, 2);
constexpr int kProbeFloatsAny = update_row(121, 3) + update_row(256, 2);

// Eq. 3 for up to 16 probes as a matrix product on MFMA (v_mfma_f32_16x16x4f32):
//   irradiance  U_i[t][(q,c)] = sum_k w_tk   * L[q][k][c]      (M = texels, N = 16 x RGB)
//   depth       U_d[t][(q,m)] = sum_k w_tk^s * t[q][k]^(m+1)   (M = texels, N = 16 x 2)
// with K = rays. The weights (shared by every probe of the frame) are the A operand,
// read from the tables in operand order (weight_index); the probes' payload is the B
// operand, staged in LDS 64 rays at a time. Each map's M-tiles are dealt round-robin to
// the 4 waves. The epilogue normalises, mixes with the previous interior (hysteresis, or
// none for rejected probes) and writes interior and border texels.
// Epilogue of both blend kernels for one 16x16 accumulator tile: lane holds
// D[4*krow + r][row]. Normalises, mixes with the previous interior (hysteresis, or
// none for rejected probes) and writes interior and border texels.
// kClamp (precision form): the depth map's second moment is raised to the square of
// its first where rounding left it below (the moments of any set of depths satisfy
// E[t^2] >= E[t]^2); the two moments of a probe sit in neighbouring lanes.
template <bool kClamp = false>
__device__ __forceinline__ void blend_epilogue(const BlendArgs &a, const float *s_h, const int *s_pid, int np,
                                               bool irr, int mtile, int n, int row, int krow,
                                               floatx4 acc) {
    const int res = irr ? a.irr_res : a.depth_res;
    const int T = res * res, comps = irr ? 3 : 2, side = res + 2;
    const int m0 = mtile * 16 + 4 * krow;
    const float *norm = irr ? a.norm_i : a.norm_d;
    const int col = n * 16 + row;
    const int q = irr ? col / 3 : col >> 1;
    const int c = irr ? col - 3 * q : col & 1;
    if (q >= np) return;
    const size_t tile_floats = (size_t)side * side * comps;
    const float *old_tile = (irr ? a.prev_irr : a.prev_depth) + (size_t)s_pid[q] * tile_floats;
    float *new_tile = (irr ? a.new_irr : a.new_depth) + (size_t)s_pid[q] * tile_floats;
    const float h = s_h[q];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int t = m0 + r;
        if (t >= T) continue;
        const int i = t % res, j = t / res;
        const float nrm = norm[t];
        const float old = old_tile[((j + 1) * side + (i + 1)) * comps + c];
        const float u = acc[r] * nrm;
        float v = nrm < 0.0f ? old : fmaf(h, old - u, u);
        if (kClamp && !irr) {
            const float first = __shfl_xor(v, 1);  // lane pairs (row, row ^ 1) hold (E[t], E[t^2])
            if (c == 1) v = fmaxf(v, first * first);
        }
        store_with_border(new_tile, res, comps, i, j, c, v);
    }
}

// The quotient of small integers by a runtime divisor n, inv = 1 / n: exact for
// e < 2^20, as (e + 1/2) / n lies at least 1 / (2 n) from an integer.
__device__ __forceinline__ int small_div(int e, float inv) { return (int)(((float)e + 0.5f) * inv); }

// One map's accumulator tiles into its rows of buf, times the texels' weight norms.
// tile0: the M-tile of slot 0.
template <int kComps, int kS, int kN>
__device__ __forceinline__ void store_updates(const float *norm, int T, int np, int tile0, int row,
                                              int krow, const floatx4 (&acc)[kS][kN], float *buf) {
#pragma unroll
    for (int s = 0; s < kS; ++s) {
        const int t0 = (tile0 + 4 * s) * 16 + 4 * krow;
        if (t0 >= T) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool in = t0 + r < T;
            const float nrm = norm[in ? t0 + r : 0];
#pragma unroll
            for (int n = 0; n < kN; ++n) {
                const int col = n * 16 + row, q = col / kComps, c = col - kComps * q;
                if (q < np && in) buf[q * update_row(T, kComps) + (t0 + r) * kComps + c] = acc[s][n][r] * nrm;
            }
        }
    }
}

// One map's padded tiles from the updates in buf: a wave takes whole probes, its lanes
// padded texels in order. Each lane finds the interior texels behind its positions once;
// per probe it reads their previous values (every read issued before the first use), mixes
// in the updates (hysteresis, or none where the history is rejected; the previous value
// where all weights vanish) and writes interior and border in order, whole texels at a time.
// A border texel repeats its source's arithmetic, so the two agree bit for bit. Per texel
// some 10 vector instructions, where deriving every element's place took 30 and the blend
// of 16384 x 256 rays 103 us for 86.
// kN: the resolution (0: `res`). kClamp: as for blend_epilogue.
template <int kN, int kComps, bool kClamp>
__device__ __forceinline__ void mix_map(int res, const float *prev, float *next, const float *norm,
                                        const float *s_h, const int *s_pid, int np,
                                        const float *buf) {
    struct Texel { float v[kComps]; };
    constexpr int kMaxSide = kN ? kN + 2 : kComps == 3 ? 13 : 18;
    constexpr int kIters = (kMaxSide * kMaxSide + 63) / 64;
    const int n = kN ? kN : res, side = n + 2, positions = side * side;
    const int lane = (int)__lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const float inv_side = 1.0f / (float)side;
    int from[kIters], old_at[kIters];
    bool keep[kIters];
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
        const int p = min(it * 64 + lane, positions - 1);
        const int y = kN ? p / side : small_div(p, inv_side), x = p - y * side;
        int i, j;
        padded_source(n, x, y, i, j);
        from[it] = (j * n + i) * kComps;
        old_at[it] = (j + 1) * side + (i + 1);
        keep[it] = norm[j * n + i] < 0.0f;
    }
    for (int q = wave; q < np; q += 4) {
        const int pid = __builtin_amdgcn_readfirstlane(s_pid[q]);
        const float h = s_h[q];
        const Texel *old_tile = reinterpret_cast<const Texel *>(prev) + (size_t)pid * positions;
        Texel *new_tile = reinterpret_cast<Texel *>(next) + (size_t)pid * positions;
        const float *u_row = buf + q * update_row(n * n, kComps);
        Texel old[kIters];
#pragma unroll
        for (int it = 0; it < kIters; ++it)
            if (kN || it * 64 < positions) old[it] = old_tile[old_at[it]];
#pragma unroll
        for (int it = 0; it < kIters; ++it) {
            const int p = it * 64 + lane;
            if (p >= positions) continue;
            Texel out;
#pragma unroll
            for (int c = 0; c < kComps; ++c) {
                const float u = u_row[from[it] + c];
                out.v[c] = keep[it] ? old[it].v[c] : fmaf(h, old[it].v[c] - u, u);
            }
            if (kClamp) out.v[1] = fmaxf(out.v[1], out.v[0] * out.v[0]);
            new_tile[p] = out;
        }
    }
}

// The epilogue through LDS, for maps of one pass. ti, td: the M-tiles of the wave's slots 0.
template <bool kStd, bool kClamp, int kIS, int kNi, int kNd>
__device__ __forceinline__ void blend_epilogue_lds(const BlendArgs &a, const float *s_h,
                                                   const int *s_pid, int np, int ti, int td,
                                                   int row, int krow, const floatx4 (&ai)[kIS][kNi],
                                                   const floatx4 (&ad)[kDepthSlots][kNd],
                                                   float *buf) {
    const int Ti = kStd ? 64 : a.irr_res * a.irr_res, Td = kStd ? 256 : a.depth_res * a.depth_res;
    float *buf_d = buf + np * update_row(Ti, 3);
    __syncthreads();  // every wave is done with what buf held before
    store_updates<3>(a.norm_i, Ti, np, ti, row, krow, ai, buf);
    store_updates<2>(a.norm_d, Td, np, td, row, krow, ad, buf_d);
    __syncthreads();
    mix_map<kStd ? 8 : 0, 3, false>(a.irr_res, a.prev_irr, a.new_irr, a.norm_i, s_h, s_pid, np, buf);
    mix_map<kStd ? 16 : 0, 2, kClamp>(a.depth_res, a.prev_depth, a.new_depth, a.norm_d, s_h, s_pid,
                                      np, buf_d);
}

// Epilogue of larger maps, texel by texel.
template <bool kClamp, int kIS, int kNi, int kNd>
__device__ __forceinline__ void blend_epilogue_direct(const BlendArgs &a, const float *s_h,
                                                      const int *s_pid, int np, int ti, int td,
                                                      int row, int krow,
                                                      const floatx4 (&ai)[kIS][kNi],
                                                      const floatx4 (&ad)[kDepthSlots][kNd]) {
    const int mti = (a.irr_res * a.irr_res + 15) >> 4, mtd = (a.depth_res * a.depth_res + 15) >> 4;
#pragma unroll
    for (int s = 0; s < kIS; ++s)
#pragma unroll
        for (int n = 0; n < kNi; ++n)
            if (ti + 4 * s < mti)
                blend_epilogue<kClamp>(a, s_h, s_pid, np, true, ti + 4 * s, n, row, krow, ai[s][n]);
#pragma unroll
    for (int s = 0; s < kDepthSlots; ++s)
#pragma unroll
        for (int n = 0; n < kNd; ++n)
            if (td + 4 * s < mtd)
                blend_epilogue<kClamp>(a, s_h, s_pid, np, false, td + 4 * s, n, row, krow, ad[s][n]);
}

// Passes that the maps' M-tiles take.
__host__ __device__ __forceinline__ int blend_passes(int irr_res, int depth_res) {
    const int mti = (irr_res * irr_res + 15) >> 4, mtd = (depth_res * depth_res + 15) >> 4;
    return std::max((mti + 4 * kIrrSlotsAny - 1) / (4 * kIrrSlotsAny),
               (mtd + 4 * kDepthSlots - 1) / (4 * kDepthSlots));
}

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// Precision form of the blend: the same tiling as blend_kernel, with the weights as
// FP16 (irradiance) / BF16 (depth) tables and the payload staged in LDS as
// FP16 radiance and BF16 (t, t^2) columns, contracted 32 rays at a time on
// v_mfma_f32_16x16x32_{f16,bf16} with FP32 accumulation.
// One workgroup's share (probe slots pb .. pb+kP-1) of the precision-form blend; also
// the body of the batched blend, which passes each scene's arguments. The tile: kP
// probes per workgroup (16: 3 irradiance and 2 depth N-tiles of 16 columns; 8: 2 and
// 1, the last irradiance tile a third empty) and kChunk rays staged in LDS at a time
// (a multiple of 32 that divides Rpad).
template <int kMaps, int kP = kBlendProbes, int kChunk = kBlendChunk>
__device__ __forceinline__ void blend16_block(const BlendArgs &a, int pb) {
    constexpr bool kStd = kMaps == kStdMaps;
    constexpr int kIS = kStd ? kIrrSlots : kIrrSlotsAny;
    constexpr int kPitch = kChunk + 8;  // halves per LDS column (+8 spreads the banks)
    constexpr int kNi = (3 * kP + 15) / 16, kNd = (2 * kP + 15) / 16;
    // payload staging (FP16 radiance, BF16 moments); the standard layout's epilogue
    // reuses the buffer
    constexpr int kSi = (kP * 3 + 1) * kPitch, kSd = (kP * 2 + 1) * kPitch;
    static_assert(kP <= kBlendProbes && kChunk % 32 == 0, "tile within the buffers");
    static_assert(kSi % 8 == 0, "16-byte aligned depth staging");
    constexpr int kStage = (kSi + kSd + 1) / 2, kBuf = kP * (kStd ? kProbeFloatsStd : kProbeFloatsAny);
    __shared__ __attribute__((aligned(16))) float sbuf[kStage > kBuf ? kStage : kBuf];
    _Float16 *si = reinterpret_cast<_Float16 *>(sbuf);
    __bf16 *sd = reinterpret_cast<__bf16 *>(si + kSi);
    __shared__ float s_h[kP];
    __shared__ int s_pid[kP];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kgrp = lane >> 4;
    const int count = a.probe_list ? min(*a.probe_count, a.P) : a.P;
    if (pb >= count) return;
    const int np = min(kP, count - pb);
    const int Ti = a.irr_res * a.irr_res, Td = a.depth_res * a.depth_res;
    const int mti = (Ti + 15) >> 4, mtd = (Td + 15) >> 4;
    load_blend_probes<kP>(a, pb, np, s_pid, s_h);
    for (int e = tid; e < kPitch; e += 256) {
        si[kP * 3 * kPitch + e] = (_Float16)0.0f;
        sd[kP * 2 * kPitch + e] = (__bf16)0.0f;
    }
    int bi_off[kNi], bd_off[kNd];
#pragma unroll
    for (int n = 0; n < kNi; ++n) {
        const int col = n * 16 + row;
        bi_off[n] = (col / 3 < np ? col : kP * 3) * kPitch;
    }
#pragma unroll
    for (int n = 0; n < kNd; ++n) {
        const int col = n * 16 + row;
        bd_off[n] = ((col >> 1) < np ? col : kP * 2) * kPitch;
    }
    // this thread's rays of a chunk, the next one's read while the present are multiplied
    // (absent probes and rays read a present one and are zeroed)
    constexpr int kLoads = (kP * kChunk + 255) / 256;
    float4 pv[kLoads];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int b = 0; b < kLoads; ++b) {
            const int e = tid + 256 * b, q = e / kChunk, kk = e - q * kChunk;
            pv[b] = load_streamed(a.payload + (size_t)s_pid[min(q, np - 1)] * a.R +
                                  min(k0 + kk, a.R - 1));
        }
    };
    const int passes = kMaps == kLargeMaps ? blend_passes(a.irr_res, a.depth_res) : 1;
    for (int pass = 0; pass < passes; ++pass) {
        floatx4 ai[kIS][kNi], ad[kDepthSlots][kNd];
        const _Float16 *wi[kIS];
        const __bf16 *wd[kDepthSlots];
        const int ti = pass * 4 * kIS + wave, td = pass * 4 * kDepthSlots + wave;  // M-tiles of
#pragma unroll                                                                     // slots 0
        for (int s = 0; s < kIS; ++s) {
            wi[s] = a.w16_i + (size_t)((ti + 4 * s) * 16) * a.Rpad + 8 * lane;
#pragma unroll
            for (int n = 0; n < kNi; ++n) ai[s][n] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        }
#pragma unroll
        for (int s = 0; s < kDepthSlots; ++s) {
            wd[s] = a.w16_d + (size_t)((td + 4 * s) * 16) * a.Rpad + 8 * lane;
#pragma unroll
            for (int n = 0; n < kNd; ++n) ad[s][n] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        __syncthreads();
        fetch(0);
        for (int k0 = 0; k0 < a.Rpad; k0 += kChunk) {
            if (k0) __syncthreads();
            const int kc = min(kChunk, a.R - k0);  // rays present in this chunk
#pragma unroll
            for (int b = 0; b < kLoads; ++b) {
                const int e = tid + 256 * b, q = e / kChunk, kk = e - q * kChunk;
                if (kP * kChunk % 256 && q >= kP) break;
                const float4 v = (q < np && kk < kc) ? pv[b] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                si[(q * 3 + 0) * kPitch + kk] = (_Float16)v.x;
                si[(q * 3 + 1) * kPitch + kk] = (_Float16)v.y;
                si[(q * 3 + 2) * kPitch + kk] = (_Float16)v.z;
                sd[(q * 2 + 0) * kPitch + kk] = (__bf16)v.w;
                sd[(q * 2 + 1) * kPitch + kk] = (__bf16)(v.w * v.w);
            }
            __syncthreads();
            if (k0 + kChunk < a.Rpad) fetch(k0 + kChunk);
#pragma unroll
            for (int kk = 0; kk < kChunk; kk += 32) {
                const int kl = kk + 8 * kgrp;  // this lane's 8 rays within the chunk
                half8_t bi[kNi];
                bf16x8_t bd[kNd];
#pragma unroll
                for (int n = 0; n < kNi; ++n)
                    bi[n] = *reinterpret_cast<const half8_t *>(&si[bi_off[n] + kl]);
#pragma unroll
                for (int n = 0; n < kNd; ++n)
                    bd[n] = *reinterpret_cast<const bf16x8_t *>(&sd[bd_off[n] + kl]);
#pragma unroll
                for (int s = 0; s < kIS; ++s)
                    if (kStd || ti + 4 * s < mti) {
                        const half8_t av = *reinterpret_cast<const half8_t *>(wi[s] + 16 * (k0 + kk));
#pragma unroll
                        for (int n = 0; n < kNi; ++n)
                            ai[s][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bi[n], ai[s][n], 0, 0, 0);
                    }
#pragma unroll
                for (int s = 0; s < kDepthSlots; ++s)
                    if (kStd || td + 4 * s < mtd) {
                        const bf16x8_t av = *reinterpret_cast<const bf16x8_t *>(wd[s] + 16 * (k0 + kk));
#pragma unroll
                        for (int n = 0; n < kNd; ++n)
                            ad[s][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bd[n], ad[s][n], 0, 0, 0);
                    }
            }
        }
        if constexpr (kMaps == kLargeMaps)
            blend_epilogue_direct<true>(a, s_h, s_pid, np, ti, td, row, kgrp, ai, ad);
        else
            blend_epilogue_lds<kStd, true>(a, s_h, s_pid, np, ti, td, row, kgrp, ai, ad, sbuf);
    }
    __syncthreads();
    if (tid < np && a.reject) a.reject[s_pid[tid]] = 0;
}

}  // namespace sdfddgi
