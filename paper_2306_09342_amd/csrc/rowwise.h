// Helpers shared by the kernels that give one wavefront one row at a time: 4-element vector access
// for float and bf16 rows, and the choice of how many such chunks a lane holds.
#pragma once
#include "common.h"

namespace rev {

// ---- 4-element vector access for float and bf16 -------------------------------
struct f4 { float x, y, z, w; };

__device__ __forceinline__ f4 load4(const float* p) {
    float4 v = *reinterpret_cast<const float4*>(p);
    return {v.x, v.y, v.z, v.w};
}
__device__ __forceinline__ f4 load4(const bf16* p) {
    uint2 u = *reinterpret_cast<const uint2*>(p);
    f4 r;
    r.x = __uint_as_float(u.x << 16);
    r.y = __uint_as_float(u.x & 0xFFFF0000u);
    r.z = __uint_as_float(u.y << 16);
    r.w = __uint_as_float(u.y & 0xFFFF0000u);
    return r;
}
__device__ __forceinline__ void store4(float* p, f4 v) {
    *reinterpret_cast<float4*>(p) = make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    bf16 a = __float2bfloat16(lo), b = __float2bfloat16(hi);
    uint16_t ua = *reinterpret_cast<uint16_t*>(&a), ub = *reinterpret_cast<uint16_t*>(&b);
    return (uint32_t)ua | ((uint32_t)ub << 16);
}
__device__ __forceinline__ void store4(bf16* p, f4 v) {
    uint2 u;
    u.x = pack_bf16x2(v.x, v.y);
    u.y = pack_bf16x2(v.z, v.w);
    *reinterpret_cast<uint2*>(p) = u;
}

// Register chunks (of 4 floats) each lane holds of a row: the smallest instantiated count that covers
// D / 4 / 64.  Intermediate sizes matter: the kernels keep several row-long arrays in registers, so a
// width of 768 (3 chunks) or 1280 (5) should not pay for 4 or 8.
inline int pick_maxj(int D) {
    const int nch = D / 4, need = (nch + 63) / 64;
    static const int sizes[] = {2, 3, 4, 5, 6, 8, 12, 16, 24, 32};
    for (int j : sizes)
        if (j >= need) return j;
    return 64;   // D > 8192: no instantiation
}

// How the LayerNorm kernels lay out a row: lpr lanes with maxj chunks of 4 floats each.  Rows of up to 256 floats may share a
// wavefront; row_sum adds the chunks of a row in the same order either way, so the layout is free to follow the clock.
struct RowSplit { int lpr, maxj; };
#define ROW_SPLITS_WIDE(X) X(64, 2) X(64, 3) X(64, 4) X(64, 5) X(64, 6) X(64, 8) X(64, 12) X(64, 16) X(64, 24) X(64, 32)
#define ROW_SPLITS_8(X) X(8, 1) X(8, 2) X(8, 3)
#define ROW_SPLITS_FWD(X) X(8, 4) X(16, 3) X(16, 4)              // the forward kernel only
inline RowSplit pick_row(int D, bool shared) {
    const int nch = D / 4;
    if (shared && nch <= 32) return {8, (nch + 7) / 8};
    if (shared && nch <= 64) return {16, nch <= 48 ? 3 : 4};
    return {64, pick_maxj(D)};
}
// Sum of a row from each lane's chunk sums p, the same value in all of its lanes: chunks c and c ^ 8 first, then c ^ 4, c ^ 2, c ^ 1
// within each run of 16 chunks, then the runs (wave_sum's order).
template <int LPR, int MAXJ> __device__ __forceinline__ float row_sum(const float (&p)[MAXJ]) {
    if constexpr (LPR == 64) {
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < MAXJ; ++j) s += p[j];
        return wave_sum(s);
    } else if constexpr (LPR == 16) {
        float r[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < MAXJ; ++j) {
            float v = p[j];
            v += dpp_mov<0x128>(v);    // row_ror:8
            v += dpp_mov<0x124>(v);    // row_ror:4
            v += dpp_mov<0x122>(v);    // row_ror:2
            r[j] = v + dpp_mov<0x121>(v);    // row_ror:1
        }
        return (r[0] + r[1]) + (r[2] + r[3]);
    } else {
        static_assert(LPR == 8 && MAXJ <= 4, "row_sum");
        float r[2] = {0.f, 0.f};
#pragma unroll
        for (int k = 0; 2 * k < MAXJ; ++k) {
            float v = p[2 * k];
            if (2 * k + 1 < MAXJ) v += p[2 * k + 1];
            v += dpp_mov<0x141>(dpp_mov<0x1B>(v));    // lane ^ 4: quads reversed, then mirrored in the 8
            v += dpp_mov<0x4E>(v);     // quad_perm 2,3,0,1
            r[k] = v + dpp_mov<0xB1>(v);     // quad_perm 1,0,3,2
        }
        return r[0] + r[1];
    }
}

}  // namespace rev
