// Softmax attention with float32 products on the float32 matrix cores (v_mfma_f32_32x32x2_f32): the float32 mode, and the
// backward of bf16 heads wider than 96 features (which the bf16 kernels do not take).
//
// A workgroup owns 32 query rows (forward, dQ) or 32 key rows (dK, dV) of one head; its four wavefronts split the other
// axis: wavefront w takes the 32-row tiles w, w + 4, ..., everything straight from global memory (a head's rows stay in
// the caches), and their results are combined in wavefront order through LDS.  The score tile has the owned index on the
// accumulator's lane axis, so its registers are directly the B operand of the next product, whose other operand is read
// one float per lane from two rows: nothing is transposed.  Both backward passes are one launch (blockIdx.z).
//
// Register layout of v_mfma_f32_32x32x2_f32, lane l, g = l / 32: A row l%32, k = g; B column l%32, k = g; D column l%32,
// rows 8*(v/4) + 4g + v%4.
#include "mfma.h"
#include "rowwise.h"
#include <algorithm>

namespace rev {

constexpr int AF_NW = 4;

// Rows r0 + l%32 (clamped) of a [rows, ld] matrix: f[4*q + e] = X[row][8q + 4g + e], 0 beyond dh
template <int DHP, typename T>
__device__ __forceinline__ void rows_frag(const T* __restrict__ base, int64_t ld, int r0, int rows, int dh, int lane, float (&f)[DHP / 2]) {
    const T* p = base + (int64_t)min(r0 + (lane & 31), rows - 1) * ld + 4 * (lane >> 5);
#pragma unroll
    for (int q = 0; q < DHP / 8; ++q) {
        f4 v = {0.f, 0.f, 0.f, 0.f};
        if (8 * q < dh) v = load4(p + 8 * q);
        f[4 * q] = v.x; f[4 * q + 1] = v.y; f[4 * q + 2] = v.z; f[4 * q + 3] = v.w;
    }
}
template <int DHP>
__device__ __forceinline__ f32x16_t rows_product(const float (&a)[DHP / 2], const float (&b)[DHP / 2]) {
    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
    for (int k = 0; k < DHP / 2; ++k) acc = mfma_f32(a[k], b[k], acc);
    return acc;
}
// acc[d, owned] += sum over the tile's rows r of X[r0 + r][32*dt + d] * p[r, owned]; p in accumulator order.  Rows from `rows`
// on count as zeros whatever they hold: their p is 0, but 0 times an infinity or a NaN would not be.  The columns are requested
// before the first product: left to the compiler, which of its loops wait for every element by itself changes from kernel to kernel.
// Four float32 blocks, both passes of the backward / the forward, us, left to it and this way: 54732 heads of one token, 32 features 4915 / 895 and
// 4500 / 825; 161 of 503 tokens, 32 features 1351 / 326 and 1261 / 332; 394 of 46, 80 features 438 / 114 and 395 / 110; three blocks, 80 of 100, 128
// features 259 / 139 and 202 / 80; 18 of 197, 64 features 84 / 47 and 79 / 40.
template <typename T>
__device__ __forceinline__ void cols_frag(const T* __restrict__ base, int64_t ld, int r0, int rows, int dh, int dt, int lane, T (&x)[16]) {
    const int c = min(dt * 32 + (lane & 31), dh - 1), g = lane >> 5;
#pragma unroll
    for (int v = 0; v < 16; ++v) x[v] = base[(int64_t)min(r0 + 8 * (v >> 2) + 4 * g + (v & 3), rows - 1) * ld + c];
    __builtin_amdgcn_sched_barrier(0);
}
template <typename T>
__device__ __forceinline__ f32x16_t cols_product(const T (&x)[16], int r0, int rows, int lane, const float (&p)[16], f32x16_t acc) {
    const int g = lane >> 5;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc = mfma_f32(r0 + 8 * (v >> 2) + 4 * g + (v & 3) < rows ? to_f(x[v]) : 0.f, p[v], acc);
    return acc;
}
template <typename T>
__device__ __forceinline__ f32x16_t cols_product(const T* __restrict__ base, int64_t ld, int r0, int rows, int dh, int dt, int lane,
                                                 const float (&p)[16], f32x16_t acc) {
    T x[16];
    cols_frag(base, ld, r0, rows, dh, dt, lane, x);
    return cols_product(x, r0, rows, lane, p, acc);
}
// Sum over the workgroup's wavefronts of an accumulator, in wavefront order: every wavefront puts its tile to LDS
// (lane-major, conflict-free), wavefront dt % AF_NW then owns tile dt.
constexpr int AF_SLOT = 16 * 64;
__device__ __forceinline__ void put_tile(float* slot, const f32x16_t& a, int lane) {
#pragma unroll
    for (int v = 0; v < 16; ++v) slot[v * 64 + lane] = a[v];
}
__device__ __forceinline__ f32x16_t sum_tiles(const float* slot, int stride, int lane) {
    f32x16_t s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = slot[v * 64 + lane];
#pragma unroll
    for (int w = 1; w < AF_NW; ++w)
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] += slot[w * stride + v * 64 + lane];
    return s;
}
// columns 8*v4 + 4g ... +3 of feature tile dt of row `row` (the lane's owned row)
template <typename T>
__device__ __forceinline__ void store_tile(T* row, int dt, int dh, int lane, const f32x16_t& a, float mul) {
    const int g = lane >> 5;
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4) {
        const int d = dt * 32 + 8 * v4 + 4 * g;
        if (d < dh) store4(row + d, f4{a[4 * v4] * mul, a[4 * v4 + 1] * mul, a[4 * v4 + 2] * mul, a[4 * v4 + 3] * mul});
    }
}

// the rows q0 .. q0 + 31 of head bh
template <int DHP> constexpr int AF_FWD_LDS = AF_NW * (DHP / 32 * AF_SLOT + 64) * 4;
template <int DHP>
__device__ __forceinline__ void fwd_rows_f32(const float* __restrict__ qkv, float* __restrict__ o, float* __restrict__ lse,
                                             const int* __restrict__ key_len, int T, int H, int dh, int q0, int bh, float* lds) {
    constexpr int DT = DHP / 32;
    float (*tiles)[DT][AF_SLOT] = reinterpret_cast<float (*)[DT][AF_SLOT]>(lds);
    float (*sm)[32] = reinterpret_cast<float (*)[32]>(lds + AF_NW * DT * AF_SLOT), (*sl)[32] = sm + AF_NW;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 5;
    const int b = bh / H, h = bh % H, D = H * dh;
    const int64_t ld = 3 * (int64_t)D;
    const float* base = qkv + (int64_t)b * T * ld + h * dh;
    const int q = q0 + (lane & 31);
    const float scale = rsqrtf((float)dh);
    const int Tk = key_len ? min(max(key_len[b], 1), T) : T;     // keys beyond take no part in the softmax

    float bq[DHP / 2];
    rows_frag<DHP>(base, ld, q0, T, dh, lane, bq);
    f32x16_t acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[dt][v] = 0.f;
    float m = -INFINITY, l = 0.f;
    for (int k0 = wave * 32; k0 < Tk; k0 += AF_NW * 32) {
        float ak[DHP / 2];
        rows_frag<DHP>(base + D, ld, k0, T, dh, lane, ak);
        float xv[16];
        constexpr bool EARLY = DT <= 2;                          // beyond 64 features a second workgroup needs the registers
        if (EARLY) cols_frag(base + 2 * D, ld, k0, Tk, dh, 0, lane, xv);
        const f32x16_t s = rows_product<DHP>(ak, bq);
        float p[16], mloc = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int key = k0 + 8 * (v >> 2) + 4 * g + (v & 3);
            p[v] = key < Tk ? s[v] * scale : -INFINITY;
            mloc = fmaxf(mloc, p[v]);
        }
        mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64));
        const float mn = fmaxf(m, mloc), ms = mn == -INFINITY ? 0.f : mn, corr = __expf(m - ms);    // (no finite score yet)
        float lsum = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            p[v] = __expf(p[v] - ms);
            lsum += p[v];
        }
        l = l * corr + lsum + __shfl_xor(lsum, 32, 64);
        m = mn;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[dt][v] *= corr;
            if (!EARLY || dt > 0) cols_frag(base + 2 * D, ld, k0, Tk, dh, dt, lane, xv);
            acc[dt] = cols_product(xv, k0, Tk, lane, p, acc[dt]);
        }
    }
    if (g == 0) { sm[wave][lane] = m; sl[wave][lane] = l; }
    __syncthreads();
    // common maximum and denominator, in wavefront order (a wavefront without keys has m = -inf, l = 0)
    float M = sm[0][lane & 31];
#pragma unroll
    for (int w = 1; w < AF_NW; ++w) M = fmaxf(M, sm[w][lane & 31]);
    float Lsum = 0.f;
#pragma unroll
    for (int w = 0; w < AF_NW; ++w) Lsum += sl[w][lane & 31] * __expf(sm[w][lane & 31] - M);
    const float mine = __expf(m - M);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[dt][v] *= mine;
        put_tile(tiles[wave][dt], acc[dt], lane);
    }
    __syncthreads();
    if (q < T) {
        float* row = o + ((int64_t)b * T + q) * D + h * dh;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
            if (dt % AF_NW == wave) store_tile(row, dt, dh, lane, sum_tiles(tiles[0][dt], DT * AF_SLOT, lane), 1.f / Lsum);
        if (wave == 0 && g == 0) lse[(int64_t)bh * T + q] = M + __logf(Lsum);
    }
}

template <int DHP>
__global__ __launch_bounds__(AF_NW * 64) void attn_fwd_f32(const float* __restrict__ qkv, float* __restrict__ o, float* __restrict__ lse,
                                                           const int* __restrict__ key_len, int T, int H, int dh) {
    __shared__ float lds[AF_FWD_LDS<DHP> / 4];
    fwd_rows_f32<DHP>(qkv, o, lse, key_len, T, H, dh, blockIdx.x * 32, blockIdx.y, lds);
}

// pass 0: dQ of the 32 query rows from r0 on, head bh;  1: dK and dV of 32 key rows.  tiles: [AF_NW][2 * DT][AF_SLOT]
template <int DHP, typename T>
__device__ __forceinline__ void bwd_rows_f32(const T* __restrict__ qkv, const T* __restrict__ o, const T* __restrict__ dout,
                                             const float* __restrict__ lse, T* __restrict__ dqkv, const int* __restrict__ key_len, int Tn,
                                             int H, int dh, int r0, int bh, int pass, float* tiles) {
    constexpr int DT = DHP / 32;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 5;
    const int b = bh / H, h = bh % H, D = H * dh;
    const int64_t ld = 3 * (int64_t)D;
    const T* base = qkv + (int64_t)b * Tn * ld + h * dh;
    const T* dob = dout + (int64_t)b * Tn * D + h * dh;
    const T* ob = o + (int64_t)b * Tn * D + h * dh;
    const float* lrow = lse + (int64_t)bh * Tn;
    const int own = r0 + (lane & 31);
    const float scale = rsqrtf((float)dh);
    const int Tk = key_len ? min(max(key_len[b], 1), Tn) : Tn;
    // delta of rows t0 + l%32: sum over features of dO * O; the two lane groups hold complementary features
    auto row_delta = [&](int t0, const float (&fdo)[DHP / 2]) {
        float fo[DHP / 2], dl = 0.f;
        rows_frag<DHP>(ob, D, t0, Tn, dh, lane, fo);
#pragma unroll
        for (int k = 0; k < DHP / 2; ++k) dl += fdo[k] * fo[k];
        return dl + __shfl_xor(dl, 32, 64);
    };
    f32x16_t acc[2 * DT];
#pragma unroll
    for (int t = 0; t < 2 * DT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;

    if (pass == 0) {
        float bq[DHP / 2], bdo[DHP / 2];
        rows_frag<DHP>(base, ld, r0, Tn, dh, lane, bq);
        rows_frag<DHP>(dob, D, r0, Tn, dh, lane, bdo);
        const float dl = row_delta(r0, bdo), L = lrow[min(own, Tn - 1)];
        for (int k0 = wave * 32; k0 < Tk; k0 += AF_NW * 32) {
            float a[DHP / 2], ds[16];
            rows_frag<DHP>(base + D, ld, k0, Tn, dh, lane, a);
            const f32x16_t s = rows_product<DHP>(a, bq);
            rows_frag<DHP>(base + 2 * D, ld, k0, Tn, dh, lane, a);
            const f32x16_t dp = rows_product<DHP>(a, bdo);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int key = k0 + 8 * (v >> 2) + 4 * g + (v & 3);
                ds[v] = key < Tk ? __expf(s[v] * scale - L) * (dp[v] - dl) * scale : 0.f;
            }
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) acc[dt] = cols_product(base + D, ld, k0, Tk, dh, dt, lane, ds, acc[dt]);
        }
    } else {
        float bk[DHP / 2], bv[DHP / 2];
        rows_frag<DHP>(base + D, ld, r0, Tn, dh, lane, bk);
        rows_frag<DHP>(base + 2 * D, ld, r0, Tn, dh, lane, bv);
        for (int t0 = wave * 32; t0 < Tn; t0 += AF_NW * 32) {
            float a[DHP / 2], p[16], ds[16];
            rows_frag<DHP>(dob, D, t0, Tn, dh, lane, a);
            const float dl = row_delta(t0, a);
            const f32x16_t dp = rows_product<DHP>(a, bv);
            rows_frag<DHP>(base, ld, t0, Tn, dh, lane, a);
            const f32x16_t s = rows_product<DHP>(a, bk);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = 8 * (v >> 2) + 4 * g + (v & 3), i = t0 + r;
                p[v] = i < Tn ? __expf(s[v] * scale - lrow[min(i, Tn - 1)]) : 0.f;
                const float d = __shfl(dl, r, 64);
                ds[v] = i < Tn ? p[v] * (dp[v] - d) * scale : 0.f;
            }
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                acc[dt] = cols_product(base, ld, t0, Tn, dh, dt, lane, ds, acc[dt]);
                acc[DT + dt] = cols_product(dob, D, t0, Tn, dh, dt, lane, p, acc[DT + dt]);
            }
        }
    }
    const int nt = pass == 0 ? DT : 2 * DT;
#pragma unroll
    for (int t = 0; t < 2 * DT; ++t)
        if (t < nt) put_tile(tiles + (wave * 2 * DT + t) * AF_SLOT, acc[t], lane);
    __syncthreads();
    if (own >= Tn) return;
    T* row = dqkv + ((int64_t)b * Tn + own) * ld + h * dh;
    const bool masked = pass == 1 && own >= Tk;                    // a masked key: no query looked at it
    for (int t = wave; t < nt; t += AF_NW) {
        f32x16_t s = sum_tiles(tiles + t * AF_SLOT, 2 * DT * AF_SLOT, lane);
        if (masked)
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = 0.f;
        T* dst = pass == 0 ? row : (t < DT ? row + D : row + 2 * D);
        store_tile(dst, t < DT ? t : t - DT, dh, lane, s, 1.f);
    }
}

template <int DHP, typename T>
__global__ __launch_bounds__(AF_NW * 64) void attn_bwd_f32(const T* __restrict__ qkv, const T* __restrict__ o, const T* __restrict__ dout,
                                                           const float* __restrict__ lse, T* __restrict__ dqkv,
                                                           const int* __restrict__ key_len, int Tn, int H, int dh) {
    extern __shared__ __attribute__((aligned(16))) float tiles[];
    bwd_rows_f32<DHP, T>(qkv, o, dout, lse, dqkv, key_len, Tn, H, dh, blockIdx.x * 32, blockIdx.y, blockIdx.z, tiles);
}
// Its two passes and, as blockIdx.z = 2, the forward of the other chain of a small stack (rev_stack.hip).
template <int DHP>
__global__ __launch_bounds__(AF_NW * 64) void attn_pair_f32(const float* __restrict__ qkv, const float* __restrict__ o,
                                                            const float* __restrict__ dout, const float* __restrict__ lse,
                                                            float* __restrict__ dqkv, const int* __restrict__ key_len, int Tn, int H, int dh,
                                                            AttnFwdCall<float> f) {
    extern __shared__ __attribute__((aligned(16))) float tiles[];
    if (blockIdx.z < 2) bwd_rows_f32<DHP, float>(qkv, o, dout, lse, dqkv, key_len, Tn, H, dh, blockIdx.x * 32, blockIdx.y, blockIdx.z, tiles);
    else fwd_rows_f32<DHP>(f.qkv, f.o, f.lse, key_len, Tn, H, dh, blockIdx.x * 32, blockIdx.y, tiles);
}

int attention_forward_f32(hipStream_t s, const float* qkv, float* o, float* lse, int B, int T, int H, int dh, const int* key_len) {
    ProfScope ps(K_ATTN_FWD, s, 4.0 * B * H * (double)T * T * dh);
    const dim3 grid((T + 31) / 32, B * H), block(AF_NW * 64);
    switch ((dh + 31) / 32) {
#define CASE(J) case J: hipLaunchKernelGGL((attn_fwd_f32<32 * J>), grid, block, 0, s, qkv, o, lse, key_len, T, H, dh); break;
        CASE(1) CASE(2) CASE(3) CASE(4)
#undef CASE
        default: set_error("attention: head_dim too large"); return REV_EINVAL;
    }
    REV_HIP(hipGetLastError());
    return REV_OK;
}

template <typename T>
int attention_backward_f32(hipStream_t s, const T* qkv, const T* o, const T* dout, const float* lse, T* dqkv, int B, int Tn, int H,
                           int dh, const int* key_len) {
    ProfScope ps(K_ATTN_BWD, s, 8.0 * B * H * (double)Tn * Tn * dh);
    const dim3 grid((Tn + 31) / 32, B * H, 2), block(AF_NW * 64);
    switch ((dh + 31) / 32) {
#define CASE(J) case J: {                                                                                                   \
        constexpr int bytes = AF_NW * 2 * J * AF_SLOT * 4;                                                                  \
        static LdsLimit lim;                                                                                                \
        if (int rc = lim.ensure(reinterpret_cast<const void*>(attn_bwd_f32<32 * J, T>), bytes)) return rc;                  \
        hipLaunchKernelGGL((attn_bwd_f32<32 * J, T>), grid, block, bytes, s, qkv, o, dout, lse, dqkv, key_len, Tn, H, dh);  \
        break; }
        CASE(1) CASE(2) CASE(3) CASE(4)
#undef CASE
        default: set_error("attention: head_dim too large"); return REV_EINVAL;
    }
    REV_HIP(hipGetLastError());
    return REV_OK;
}
// One launch up to 768 workgroups of each pass.  Beyond, the forward's workgroups, which hold the LDS of the backward's there, have too few
// beside them.  Two launches against one, 220 stacks of four blocks, geometric mean of the pass by workgroups of a pass: 257 to 384 0.96, 513 to
// 768 0.98, 769 to 1024 1.01, 1537 to 2048 1.02, 2049 to 4096 1.03, more 1.04.
constexpr int AF_PAIR_MOST = 768;
int attention_pair_f32(hipStream_t s, const float* qkv, const float* o, const float* dout, const float* lse, float* dqkv, int B, int T, int H,
                       int dh, const int* key_len, const AttnFwdCall<float>& fwd) {
    if ((int64_t)((T + 31) / 32) * B * H > AF_PAIR_MOST) {
        if (int rc = attention_backward_f32<float>(s, qkv, o, dout, lse, dqkv, B, T, H, dh, key_len)) return rc;
        return attention_forward_f32(s, fwd.qkv, fwd.o, fwd.lse, B, T, H, dh, key_len);
    }
    ProfScope ps(K_MIXED, s, 12.0 * B * H * (double)T * T * dh);
    const dim3 grid((T + 31) / 32, B * H, 3), block(AF_NW * 64);
    switch ((dh + 31) / 32) {
#define CASE(J) case J: {                                                                                                   \
        constexpr int bytes = std::max(AF_NW * 2 * J * AF_SLOT * 4, AF_FWD_LDS<32 * J>);                                    \
        static LdsLimit lim;                                                                                                \
        if (int rc = lim.ensure(reinterpret_cast<const void*>(attn_pair_f32<32 * J>), bytes)) return rc;                    \
        hipLaunchKernelGGL((attn_pair_f32<32 * J>), grid, block, bytes, s, qkv, o, dout, lse, dqkv, key_len, T, H, dh, fwd); \
        break; }
        CASE(1) CASE(2) CASE(3) CASE(4)
#undef CASE
        default: set_error("attention: head_dim too large"); return REV_EINVAL;
    }
    REV_HIP(hipGetLastError());
    return REV_OK;
}
template int attention_backward_f32<float>(hipStream_t, const float*, const float*, const float*, const float*, float*, int, int, int, int, const int*);
template int attention_backward_f32<bf16>(hipStream_t, const bf16*, const bf16*, const bf16*, const float*, bf16*, int, int, int, int, const int*);

}  // namespace rev
