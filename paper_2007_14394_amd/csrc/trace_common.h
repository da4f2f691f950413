// Device code shared by the trace kernels of one scene (kernels.hip) and of a
// batch of scenes (batch.hip): the cascade level as the loops read it, the
// trilinear sampler and its fixed binary32 lerp sequence, the hit normal, the
// probe interpolation, and the wave-level work feeder.
#pragma once

#include "internal.h"

namespace sdfddgi {

enum : int { kMissTmax = 0, kMissExit = 1, kHit = 2, kHitExhausted = 3, kInside = 4 };

__device__ __forceinline__ float clampf(float v, float lo, float hi) { return fminf(fmaxf(v, lo), hi); }

// Cell and fraction of grid coordinate u along one axis (cell clamped to [0, cmax],
// cmax = vertices - 2), for any u.
__device__ __forceinline__ void cell_of(float u, float cmax, int &i, float &f) {
    const float fl = clampf(floorf(u), 0.0f, cmax);
    i = (int)fl;
    f = clampf(u - fl, 0.0f, 1.0f);
}

// The same for a coordinate known to lie in the level's box, 0 <= u <= cmax + 1, without
// the clamps that cannot act there (u - floor(u) is in [0, 1), and 1 at u = cmax + 1).
__device__ __forceinline__ void cell_inside(float u, uint32_t cmax, uint32_t &i, float &f) {
    i = min((uint32_t)u, cmax);
    f = u - (float)i;
}

// The grid is stored as cell bricks, one 128-byte line each, so that the eight corners of
// any cell sit in one line and are read with two 16-byte loads. Neighbouring bricks share
// their boundary vertices:
//   binary32: 4 x 4 vertex columns of two z each (z, z+1): 3 x 3 x 1 cells. Column (a, b)
//     at byte 8 (4 b + a); corners of cell (a, b): columns a, a+1 of rows b and b+1.
//   binary16: 4 x 4 x 4 vertices, column (a, b) = its four z at byte 8 (4 b + a): 3 x 3 x 3
//     cells; the pair (z, z+1) of a cell is picked from each column.
// The trace is bound by its scattered reads: two requests per sample to the L1, and fills
// of the lines its L2 misses. Against corner quads in x order (8 or 16 cells in a row per
// line, a cell crossing two lines in 1 of 8 or 16), one primary trace of the open scene
// (16384 x 256) fills 16.9 M lines instead of 20.1 M in binary32 and 9.6 M instead of
// 14.2 M in binary16, whose bricks also take 4.7 bytes a cell instead of 8.
typedef float float4_a8 __attribute__((ext_vector_type(4), aligned(8)));
typedef uint32_t uint4_a8 __attribute__((ext_vector_type(4), aligned(8)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

// a * b + c on the low 24 bits of a and b (the compiler turns the plain expressions into
// 64-bit multiply-adds, at four times the cost); `s` in a scalar register.
__device__ __forceinline__ uint32_t mad_u24(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ uint32_t mul_u24_s(uint32_t a, uint32_t s) {
    uint32_t r;
    asm("v_mul_u32_u24 %0, %1, %2" : "=v"(r) : "s"(s), "v"(a));
    return r;
}
__device__ __forceinline__ uint32_t mad_i24_s(uint32_t a, int32_t s, uint32_t c) {
    uint32_t r;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(s), "v"(c));
    return r;
}

// Device memory as such (a generic address would also count as an LDS access).
typedef const __attribute__((address_space(1))) char *GlobalBytes;

struct Corners { float v000, v100, v010, v110, v001, v101, v011, v111; };

// kWide: the general 32-bit division and products and 64-bit offsets; else every cell
// index is below 2^16, every row of bricks below 2^24 and all bricks within 4 GiB, for
// which the 24-bit products are exact (43691 / 2^17 exceeds 1/3 by less than
// 1 / (3 * 2^16)) and cost a quarter, and an offset is one register.
template <bool kHalf, bool kWide>
__device__ __forceinline__ Corners load_corners(GlobalBytes cells, const LevelCells &d, uint32_t i0,
                                                uint32_t i1, uint32_t i2) {
    uint32_t a2;
    GlobalBytes p;
    if (kWide) {
        const uint32_t b0 = i0 / 3u, b1 = i1 / 3u, b2 = kHalf ? i2 / 3u : i2;
        a2 = i2 - 3u * b2;
        const uint32_t line = (b2 * d.nb1 + b1) * d.nb0 + (b0 + d.line0);
        p = cells + (((uint64_t)line << 7) + ((i1 - 3u * b1) * 32u + (i0 - 3u * b0) * 8u));
    } else {
        const uint32_t b0 = mul_u24_s(i0, 43691u) >> 17, b1 = mul_u24_s(i1, 43691u) >> 17;
        const uint32_t b2 = kHalf ? mul_u24_s(i2, 43691u) >> 17 : i2;
        a2 = mad_i24_s(b2, -3, i2);
        const uint32_t line = mad_u24(mad_u24(b2, d.nb1, b1), d.nb0, b0 + d.line0);
        p = cells + ((line << 7) |
                     mad_i24_s(b1, -96, mad_i24_s(b0, -24, (i1 << 5) + (i0 << 3))));
    }
    Corners c;
    if (kHalf) {
        const uint4_a8 r0 = *(const __attribute__((address_space(1))) uint4_a8 *)p;
        const uint4_a8 r1 = *(const __attribute__((address_space(1))) uint4_a8 *)(p + 32);
        // bytes 2 a2 .. 2 a2 + 3 of a column
        const uint32_t sel = __builtin_amdgcn_perm(a2 + a2, a2 + a2, 0u) + 0x03020100u;
        const half2_t c00 = __builtin_bit_cast(half2_t, __builtin_amdgcn_perm(r0.y, r0.x, sel));
        const half2_t c10 = __builtin_bit_cast(half2_t, __builtin_amdgcn_perm(r0.w, r0.z, sel));
        const half2_t c01 = __builtin_bit_cast(half2_t, __builtin_amdgcn_perm(r1.y, r1.x, sel));
        const half2_t c11 = __builtin_bit_cast(half2_t, __builtin_amdgcn_perm(r1.w, r1.z, sel));
        c.v000 = (float)c00.x; c.v001 = (float)c00.y;
        c.v100 = (float)c10.x; c.v101 = (float)c10.y;
        c.v010 = (float)c01.x; c.v011 = (float)c01.y;
        c.v110 = (float)c11.x; c.v111 = (float)c11.y;
    } else {
        const float4_a8 r0 = *(const __attribute__((address_space(1))) float4_a8 *)p;
        const float4_a8 r1 = *(const __attribute__((address_space(1))) float4_a8 *)(p + 32);
        c.v000 = r0.x; c.v001 = r0.y; c.v100 = r0.z; c.v101 = r0.w;
        c.v010 = r1.x; c.v011 = r1.y; c.v110 = r1.z; c.v111 = r1.w;
    }
    return c;
}

// Trilinear interpolation: lerps along x, then y, then z.
__device__ __forceinline__ float lerp_corners(const Corners &c, float f0, float f1, float f2) {
    const float c00 = fmaf(f0, c.v100 - c.v000, c.v000);
    const float c10 = fmaf(f0, c.v110 - c.v010, c.v010);
    const float c01 = fmaf(f0, c.v101 - c.v001, c.v001);
    const float c11 = fmaf(f0, c.v111 - c.v011, c.v011);
    const float c0 = fmaf(f1, c10 - c00, c00);
    const float c1 = fmaf(f1, c11 - c01, c01);
    return fmaf(f2, c1 - c0, c0);
}

// Trilinear sample at any grid coordinates (u0,u1,u2). `wide`: see CellShape.
template <bool kHalf>
__device__ __forceinline__ float trilinear(GlobalBytes cells, const LevelCells &d, int wide,
                                           float u0, float u1, float u2) {
    int i0, i1, i2;
    float f0, f1, f2;
    cell_of(u0, (float)d.cmax0, i0, f0);
    cell_of(u1, (float)d.cmax1, i1, f1);
    cell_of(u2, (float)d.cmax2, i2, f2);
    return lerp_corners(wide ? load_corners<kHalf, true>(cells, d, i0, i1, i2)
                             : load_corners<kHalf, false>(cells, d, i0, i1, i2),
                        f0, f1, f2);
}

template <bool kHalf>
__device__ __forceinline__ float sample_at(GlobalBytes cells, const LevelCells &d, int wide, float p0,
                                           float p1, float p2) {
    return trilinear<kHalf>(cells, d, wide, (p0 - d.org0) * d.inv, (p1 - d.org1) * d.inv, (p2 - d.org2) * d.inv);
}

// The distance at a point of the level's box (elsewhere, a value between a cell's
// corners or beyond them).
template <bool kHalf, bool kWide>
__device__ __forceinline__ float distance_inside(GlobalBytes cells, const LevelCells &level,
                                                 float x0, float x1, float x2) {
    const LevelCells d = level;
    uint32_t i0, i1, i2;
    float f0, f1, f2;
    cell_inside((x0 - d.org0) * d.inv, d.cmax0, i0, f0);
    cell_inside((x1 - d.org1) * d.inv, d.cmax1, i1, f1);
    cell_inside((x2 - d.org2) * d.inv, d.cmax2, i2, f2);
    return lerp_corners(load_corners<kHalf, kWide>(cells, d, i0, i1, i2), f0, f1, f2);
}

// Central differences at +-spacing/2 on the hit's level, normalised. Half a cell either way,
// one of an axis's two samples lies in x's own cell (but for rounding, and at the level's
// borders, where both may or neither), whose corners are read once for all three: four
// cells' reads instead of six, and fewer places to find. Of the frames of 24 scenes, bound by
// the lines that their hits and traces draw through the L1, 6.58 -> 6.41 ms for four; one
// axis at a time, in fewer registers, 6.49.
template <bool kHalf>
__device__ __forceinline__ void hit_normal(GlobalBytes cells, const LevelCells &d, int wide, float x0,
                                           float x1, float x2, float w0, float w1, float w2,
                                           float &n0, float &n1, float &n2) {
    const float h = d.half;
    float g0 = 0.0f, g1 = 0.0f, g2 = 0.0f;
    int i0, i1, i2;
    float f0, f1, f2;
    cell_of((x0 - d.org0) * d.inv, (float)d.cmax0, i0, f0);
    cell_of((x1 - d.org1) * d.inv, (float)d.cmax1, i1, f1);
    cell_of((x2 - d.org2) * d.inv, (float)d.cmax2, i2, f2);
    auto corners = [&](int c0, int c1, int c2) {
        return wide ? load_corners<kHalf, true>(cells, d, c0, c1, c2)
                    : load_corners<kHalf, false>(cells, d, c0, c1, c2);
    };
    const Corners own = corners(i0, i1, i2);
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const float x = ax == 0 ? x0 : ax == 1 ? x1 : x2;
        const float org = ax == 0 ? d.org0 : ax == 1 ? d.org1 : d.org2;
        const float cmax = (float)(ax == 0 ? d.cmax0 : ax == 1 ? d.cmax1 : d.cmax2);
        const int i = ax == 0 ? i0 : ax == 1 ? i1 : i2;
        int ip, im;
        float fp, fm;
        cell_of((x + h - org) * d.inv, cmax, ip, fp);
        cell_of((x - h - org) * d.inv, cmax, im, fm);
        // the sample in x's own cell (the minus one if neither is) and the other
        const bool plus = ip == i;
        const int far = plus ? im : ip;
        auto along = [&](int c) {
            return corners(ax == 0 ? c : i0, ax == 1 ? c : i1, ax == 2 ? c : i2);
        };
        const Corners other = along(far);
        Corners near = own;
        if (!plus && im != i) near = along(im);
        auto at = [&](const Corners &c, float f) {
            return lerp_corners(c, ax == 0 ? f : f0, ax == 1 ? f : f1, ax == 2 ? f : f2);
        };
        const float a = at(near, plus ? fp : fm), b = at(other, plus ? fm : fp);
        const float g = plus ? a - b : b - a;
        g0 = ax == 0 ? g : g0;
        g1 = ax == 1 ? g : g1;
        g2 = ax == 2 ? g : g2;
    }
    const float len2 = fmaf(g2, g2, fmaf(g1, g1, g0 * g0));
    if (!(len2 >= 1e-24f)) { n0 = -w0; n1 = -w1; n2 = -w2; return; }
    const float inv = 1.0f / sqrtf(len2);
    n0 = g0 * inv; n1 = g1 * inv; n2 = g2 * inv;
}

__device__ __forceinline__ float sgnf(float v) { return v >= 0.0f ? 1.0f : -1.0f; }

// Probe interpolation: trilinear over the 8 probes of x's cell, bilinear in each
// probe's padded octahedral tile at direction n.
__device__ __forceinline__ float3 interp_irradiance(const float *__restrict__ atlas, int res,
                                                   const ProbeGridDev &pg, float x0, float x1,
                                                   float x2, float n0, float n1, float n2) {
    int b0, b1, b2;
    float f0, f1, f2;
    cell_of((x0 - pg.org0) * pg.inv0, (float)(pg.n0 - 2), b0, f0);
    cell_of((x1 - pg.org1) * pg.inv1, (float)(pg.n1 - 2), b1, f1);
    cell_of((x2 - pg.org2) * pg.inv2, (float)(pg.n2 - 2), b2, f2);
    float l1 = fabsf(n0) + fabsf(n1) + fabsf(n2);
    float u = n0 / l1, v = n1 / l1;
    if (n2 < 0.0f) {
        float fu = (1.0f - fabsf(v)) * sgnf(u);
        float fv = (1.0f - fabsf(u)) * sgnf(v);
        u = fu; v = fv;
    }
    const float fres = (float)res;
    float su = (fres * (u + 1.0f) + 1.0f) * 0.5f;
    float sv = (fres * (v + 1.0f) + 1.0f) * 0.5f;
    float au = clampf(floorf(su), 0.0f, fres), av = clampf(floorf(sv), 0.0f, fres);
    float fu = clampf(su - au, 0.0f, 1.0f), fv = clampf(sv - av, 0.0f, 1.0f);
    const int side = res + 2;
    const int t00 = ((int)av * side + (int)au) * 3;
    const int tile = side * side * 3;
    // the first probe's texel, and the same texel's distance (uniform) in the others
    const float *t0 = atlas + ((size_t)(b0 + pg.n0 * (b1 + pg.n1 * b2)) * tile + t00);
    const float w00 = (1.0f - fu) * (1.0f - fv), w10 = fu * (1.0f - fv);
    const float w01 = (1.0f - fu) * fv, w11 = fu * fv;
    float3 acc = make_float3(0.0f, 0.0f, 0.0f);
    // four probes per iteration: 48 values in flight, half the registers of a full unroll.
    // Addresses of the probes from one lane address and uniform strides, and fused
    // multiply-adds: half the vector instructions. Samples of a coherent image (2 M points) are
    // bound by the L1's lookups (43 us, 45 before); the hit shading of 24 scenes,
    // which shares the CUs with other kernels, gains more (6.80 -> 6.66 ms for four frames).
#pragma unroll 4
    for (int c8 = 0; c8 < 8; ++c8) {
        const int dx = c8 & 1, dy = (c8 >> 1) & 1, dz = c8 >> 2;
        const float wp = (dx ? f0 : 1.0f - f0) * (dy ? f1 : 1.0f - f1) * (dz ? f2 : 1.0f - f2);
        const float *tx = t0 + (size_t)(dx + pg.n0 * (dy + pg.n1 * dz)) * tile;
        const float *ty = tx + side * 3;
        float e[3];
#pragma unroll
        for (int c = 0; c < 3; ++c)
            e[c] = fmaf(w11, ty[3 + c], fmaf(w01, ty[c], fmaf(w10, tx[3 + c], w00 * tx[c])));
        acc.x = fmaf(wp, e[0], acc.x);
        acc.y = fmaf(wp, e[1], acc.y);
        acc.z = fmaf(wp, e[2], acc.z);
    }
    return acc;
}

// Primary-ray hit record packing: outcome | level << 4 | steps << 8.
__device__ __forceinline__ int pack_hit(int kind, int level, int steps) {
    return kind | (level << 4) | (steps << 8);
}

// Wave-level work feeder: claims `chunk` consecutive items per atomic and hands them
// to idle lanes in order. All members are wave-uniform.
struct Feeder {
    int next = 0, end = 0, chunk;
    bool exhausted = false;
    __device__ __forceinline__ explicit Feeder(int chunk_items) : chunk(chunk_items) {}
    // Returns the number of items given out; the rank-th idle lane takes first + rank.
    __device__ __forceinline__ int claim(int *counter, int total, int want, int &first) {
        if (next >= end) {
            int base = 0;
            if (__lane_id() == 0) base = atomicAdd(counter, chunk);
            base = __builtin_amdgcn_readfirstlane(base);
            if (base >= total) { exhausted = true; return 0; }
            next = base;
            end = min(base + chunk, total);
        }
        const int n = min(want, end - next);
        first = next;
        next += n;
        return n;
    }
};

// Whatever lanes of the wave store before this point reaches memory before what others of
// its lanes store after it. The memory model gives a wave's operations in the order of the
// program, so the fence is for the compiler and no instruction.
__device__ __forceinline__ void order_wave_stores() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Whether the calling lane is in a wave-uniform mask.
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// A ray waiting in LDS to be traced.
struct WaitingRay { float4 from, dir; };

// The XCD (accelerator complex die) the calling wave runs on, from the hardware
// register that holds it; each XCD has its own L2.
__device__ __forceinline__ int xcd_id() {
    return __builtin_amdgcn_s_getreg((3 << 11) | 20) & (kXcds - 1);  // HW_REG_XCC_ID, 4 bits
}

// Work handed out so that every XCD walks the same region of the item order at the
// same time (the order is coherent in space, so the device-wide working set stays
// small) while each XCD's L2 sees runs of neighbouring items: the order is cut into
// blocks of `block` chunks of `chunk` items, block b belongs to XCD b mod kXcds,
// and each XCD claims the chunks of its blocks in order from a counter of its own
// (parts[x * kPartStride]). A wave starts on its XCD's counter and moves on to the
// next XCD's once that one is used up; a counter, once used up, stays so, so a wave
// that has found kXcds used up in a row has seen them all and reports exhausted.
struct BlockFeeder {
    int next = 0, end = 0, part = 0, misses = 0, chunk, block;
    bool exhausted = false;
    __device__ __forceinline__ BlockFeeder(int chunk_items, int block_chunks)
        : part(xcd_id()), chunk(chunk_items), block(block_chunks) {}
    // Returns the number of items given out; the rank-th idle lane takes first + rank.
    __device__ __forceinline__ int claim(int *parts, int total, int want, int &first) {
        while (next >= end) {
            if (misses == kXcds) { exhausted = true; return 0; }
            int s = 0;
            if (__lane_id() == 0) s = atomicAdd(parts + part * kPartStride, 1);
            s = __builtin_amdgcn_readfirstlane(s);
            const int64_t base = (((int64_t)(s / block) * kXcds + part) * block + s % block) * chunk;
            if (base >= total) {
                part = part + 1 == kXcds ? 0 : part + 1;
                ++misses;
                continue;
            }
            next = (int)base;
            end = (int)min(base + chunk, (int64_t)total);
        }
        const int n = min(want, end - next);
        first = next;
        next += n;
        return n;
    }
};

}  // namespace sdfddgi
