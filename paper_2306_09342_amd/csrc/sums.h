// Fixed-order sums that run in a launch of their own or in the last workgroups of another one: the second stages described by
// RedSeg, and column sums in one piece.  Workgroups of 256 threads.
#pragma once
#include "rowwise.h"

namespace rev {

// out[i] = sum over p (ascending) of partial[p * stride + i]; 4 elements per thread.
// Elements at or beyond `split4` (in units of 4) go to out2 instead (nullable: dropped).
__device__ __forceinline__ void reduce_store(float* out, float* out2, int64_t split4, int64_t i, float4 acc) {
    if (i < split4) *reinterpret_cast<float4*>(out + 4 * i) = acc;
    else if (out2) *reinterpret_cast<float4*>(out2 + 4 * (i - split4)) = acc;
}

struct RedSegDev { const float* partial; float* out; float* out2; int64_t stride, n4, split4; int P, first_block; };
struct RedArgs { RedSegDev seg[RED_MAX_SEGS]; int nseg; };

// Segments with many partial rows, or few columns and more than 8 rows, use 16 row-lanes per group of 16 column quads, folded
// in lane order through LDS; the others one thread per column quad.  Either way the order is fixed.  8 loads of a
// thread are in flight together: with few blocks the launch is a chain of memory round trips (two segments of 25 rows by 2304,
// one thread per quad, loads one by one: 4.4 us, now 2.6; 1024 rows: 4.7 -> 4.2).
__host__ __device__ __forceinline__ bool reduce_by_lanes(int P, int64_t n4) { return P > 32 || (P > 8 && n4 <= 16384); }

__device__ __forceinline__ void reduce_block(const RedArgs& a, int block, float4* sh) {
    int si = 0;
#pragma unroll
    for (int k = 1; k < RED_MAX_SEGS; ++k)
        if (k < a.nseg && block >= a.seg[k].first_block) si = k;
    const RedSegDev g = a.seg[si];
    const int lb = block - g.first_block;
    // adds rows p, p + step, ... of column quad i, ascending
    auto sum_rows = [&](int p, int step, int64_t i) {
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        const float* q = g.partial + 4 * i;
        for (; p + 7 * step < g.P; p += 8 * step) {
            float4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const float4*>(q + (int64_t)(p + u * step) * g.stride);
#pragma unroll
            for (int u = 0; u < 8; ++u) { acc.x += v[u].x; acc.y += v[u].y; acc.z += v[u].z; acc.w += v[u].w; }
        }
        if (p < g.P) {
            float4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (p + u * step < g.P) v[u] = *reinterpret_cast<const float4*>(q + (int64_t)(p + u * step) * g.stride);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (p + u * step < g.P) { acc.x += v[u].x; acc.y += v[u].y; acc.z += v[u].z; acc.w += v[u].w; }
        }
        return acc;
    };
    if (reduce_by_lanes(g.P, g.n4)) {
        const int cg = threadIdx.x & 15, pl = threadIdx.x >> 4;
        const int64_t i = (int64_t)lb * 16 + cg;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i < g.n4) acc = sum_rows(pl, 16, i);
        sh[threadIdx.x] = acc;
        __syncthreads();
        if (pl == 0 && i < g.n4) {
#pragma unroll
            for (int q = 1; q < 16; ++q) {
                float4 v = sh[q * 16 + cg];
                acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
            }
            reduce_store(g.out, g.out2, g.split4, i, acc);
        }
    } else {
        const int64_t i = (int64_t)lb * 256 + threadIdx.x;
        if (i >= g.n4) return;
        const float4 acc = sum_rows(0, 1, i);
        reduce_store(g.out, g.out2, g.split4, i, acc);
    }
}

// Fills the device description; the number of workgroups, or an error.  bytes: nullable
inline int reduce_args(const RedSeg* segs, int nseg, RedArgs* a, double* bytes) {
    if (nseg > RED_MAX_SEGS) { set_error("reduce_multi: too many segments"); return REV_EINVAL; }
    a->nseg = nseg;
    int blocks = 0;
    for (int k = 0; k < nseg; ++k) {
        const RedSeg& g = segs[k];
        if (g.n % 4 != 0 || g.split % 4 != 0) { set_error("reduce_multi: lengths must be multiples of 4"); return REV_EINVAL; }
        const int64_t n4 = g.n / 4;
        a->seg[k] = {g.partial, g.out, g.out2, g.stride, n4, g.split / 4, g.P, blocks};
        blocks += (int)(reduce_by_lanes(g.P, n4) ? (n4 + 15) / 16 : (n4 + 255) / 256);
        if (bytes) *bytes += (double)(g.P + 1) * g.n * 4;
    }
    return blocks;
}

// Column sums of an [M, N] matrix in one piece, 64 columns a workgroup: 16 (float) or 8 (bf16) lanes across, the other threads
// take every 16th or 32nd row with eight loads in flight, and are added in order through sh (4 or 8 KB).  For matrices of up to
// COLSUM_ROWS rows, where a second stage would cost a launch.
inline int colsum_blocks(int N) { return (N + 63) / 64; }
template <typename T>
__device__ __forceinline__ void colsum_block(const T* __restrict__ in, int64_t ld, int M, int N, float* __restrict__ out, int block, float* sh) {
    constexpr int PER = 16 / sizeof(T), ACROSS = 64 / PER, GROUPS = 256 / ACROSS;
    const int lane = threadIdx.x % ACROSS, grp = threadIdx.x / ACROSS, col = block * 64 + lane * PER;
    float s[PER] = {};
    auto add = [&](const T* p) {
        if constexpr (sizeof(T) == 4) {
            const f4 v = load4(p);
            s[0] += v.x; s[1] += v.y; s[2] += v.z; s[3] += v.w;
        } else {
            const f4 v = load4(p), w = load4(p + 4);
            s[0] += v.x; s[1] += v.y; s[2] += v.z; s[3] += v.w;
            s[4] += w.x; s[5] += w.y; s[6] += w.z; s[7] += w.w;
        }
    };
    if (col < N) {
        const T* src = in + col;
        int r = grp;
        for (; r + 7 * GROUPS < M; r += 8 * GROUPS) {
            uint4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const uint4*>(src + (int64_t)(r + u * GROUPS) * ld);
#pragma unroll
            for (int u = 0; u < 8; ++u) add(reinterpret_cast<const T*>(&v[u]));
        }
        uint4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (r + u * GROUPS < M) v[u] = *reinterpret_cast<const uint4*>(src + (int64_t)(r + u * GROUPS) * ld);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (r + u * GROUPS < M) add(reinterpret_cast<const T*>(&v[u]));
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) sh[grp * 64 + lane * PER + e] = s[e];
    __syncthreads();
    const int c = block * 64 + threadIdx.x;
    if (threadIdx.x < 64 && c < N) {
        float t = sh[threadIdx.x];
#pragma unroll
        for (int g = 1; g < GROUPS; ++g) t += sh[g * 64 + threadIdx.x];
        out[c] = t;
    }
}

}  // namespace rev
