// bf16 softmax attention on the matrix cores: forward (flash-style, log-sum-exp
// saved) and backward in two passes, each free of atomics so that every sum has
// a fixed order:
//   pass 1  one wavefront owns 32 query rows, streams key/value tiles:  dQ, delta
//   pass 2  one wavefront owns 32 key rows, streams query/dO tiles:     dK, dV
//
// The score tile is always produced with the OWNED index on the accumulator's
// column (lane) axis: S^T[key, q] in the forward and in pass 1, S[q, key] in
// pass 2.  Row statistics of the owned index are then per-lane scalars, and the
// probability tile, converted to bf16 where it sits, is directly the B operand
// of the next product; the streamed operand of that product is read from its
// row-major LDS tile with the LDS transpose read.  No tile is ever transposed
// through memory or shuffled across lanes.
//
// Heads of 32, 64 and 80 features take the kernels of attention_dma.hip; the kernels here serve the other widths.
#include "attention.h"

namespace rev {

constexpr int AT_ROWS = 64;     // streamed rows per LDS tile

template <int DHP> struct AtCfg {
    static constexpr int KS = DHP / 16;          // contraction steps over the head dim
    static constexpr int DT = DHP / 32;          // 32-wide output tiles over the head dim
    static constexpr int PITCH = DHP + 8;        // LDS row pitch (elements)
    static constexpr int CH = DHP / 8;           // 16-byte chunks per row
};

// B-operand fragments of 32 owned rows straight from global memory:
// lane (r = l%32, g) takes X[row0 + r][16*ks + 8g .. +7]; rows are clamped, columns >= dh read as zero.
template <int DHP>
__device__ __forceinline__ void load_owned(const bf16* __restrict__ base, int64_t ld, int row0, int nrows, int dh,
                                           int lane, bf16x8_t (&frag)[DHP / 16]) {
    const int r = min(row0 + (lane & 31), nrows - 1);
    const bf16* p = base + (int64_t)r * ld + 8 * (lane >> 5);
#pragma unroll
    for (int ks = 0; ks < DHP / 16; ++ks) {
        const int c = 16 * ks + 8 * (lane >> 5);
        u32x4_t v = {0u, 0u, 0u, 0u};
        if (c < dh) v = *reinterpret_cast<const u32x4_t*>(p + 16 * ks);
        union { u32x4_t u; bf16x8_t b; } cv;
        cv.u = v;
        frag[ks] = cv.b;
    }
}

// Cooperative load of `trows` rows [row0, row0+trows) of a [nrows, ld] matrix into an LDS tile;
// rows >= nrows and columns >= dh are zero-filled.
template <int DHP>
__device__ __forceinline__ void load_tile(uint16_t* tile, const bf16* __restrict__ base, int64_t ld, int row0,
                                          int nrows, int dh, int trows) {
    constexpr int CH = AtCfg<DHP>::CH, PITCH = AtCfg<DHP>::PITCH;
    for (int idx = threadIdx.x; idx < trows * CH; idx += blockDim.x) {
        const int row = idx / CH, ch = idx % CH;
        const int gr = row0 + row;
        u32x4_t v = {0u, 0u, 0u, 0u};
        if (gr < nrows && ch * 8 < dh) v = *reinterpret_cast<const u32x4_t*>(base + (int64_t)gr * ld + ch * 8);
        *reinterpret_cast<u32x4_t*>(tile + row * PITCH + ch * 8) = v;
    }
}

// The same load in two halves, for the streamed mode (64-row tiles): the global loads of the NEXT
// tile are issued into registers before the products of the current one and stored to LDS after them,
// so their latency is covered by the matrix-core work instead of being waited for at every tile.
// A thread holds DHP / 32 16-byte pieces of one tile (enough for 64 rows with 4 or more wavefronts);
// the launcher picks the plain-load instantiation for smaller workgroups.
template <int DHP> struct TilePre {
    static constexpr int N = DHP / 32;
    u32x4_t v[N];
};

template <int DHP>
__device__ __forceinline__ void tile_fetch(TilePre<DHP>& t, const bf16* __restrict__ base, int64_t ld, int row0,
                                           int nrows, int dh) {
    constexpr int CH = AtCfg<DHP>::CH;
#pragma unroll
    for (int i = 0; i < TilePre<DHP>::N; ++i) {
        const int idx = threadIdx.x + i * blockDim.x;
        const int row = idx / CH, ch = idx % CH;
        const int gr = row0 + row;
        u32x4_t v = {0u, 0u, 0u, 0u};
        if (idx < AT_ROWS * CH && gr < nrows && ch * 8 < dh) v = *reinterpret_cast<const u32x4_t*>(base + (int64_t)gr * ld + ch * 8);
        t.v[i] = v;
    }
}
template <int DHP>
__device__ __forceinline__ void tile_store(uint16_t* tile, const TilePre<DHP>& t) {
    constexpr int CH = AtCfg<DHP>::CH, PITCH = AtCfg<DHP>::PITCH;
#pragma unroll
    for (int i = 0; i < TilePre<DHP>::N; ++i) {
        const int idx = threadIdx.x + i * blockDim.x;
        const int row = idx / CH, ch = idx % CH;
        if (idx < AT_ROWS * CH) *reinterpret_cast<u32x4_t*>(tile + row * PITCH + ch * 8) = t.v[i];
    }
}

// ----------------------------------------------------------------------------------------
// forward
// ----------------------------------------------------------------------------------------
template <int DHP, bool PIPE>
__global__ __launch_bounds__(512) void attn_fwd_mfma(const bf16* __restrict__ qkv, bf16* __restrict__ o,
                                                     float* __restrict__ lse, const int* __restrict__ key_len,
                                                     int T, int H, int dh, int trows) {
    // trows: streamed rows held in LDS at a time -- 64, or all ceil32(T) rows when they fit (one load, no
    // further barriers)
    using C = AtCfg<DHP>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint16_t* Ks0 = reinterpret_cast<uint16_t*>(smem);
    uint16_t* Vs0 = Ks0 + trows * C::PITCH;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int g = lane >> 5;
    const int bh = blockIdx.y, b = bh / H, h = bh % H;
    const int D = H * dh;
    const int64_t ld = 3 * (int64_t)D;
    const bf16* base = qkv + (int64_t)b * T * ld + h * dh;
    const int q0 = (blockIdx.x * nw + wave) * 32;
    // scores are kept in the base-2 domain (scale * log2 e folded into one multiply, exp2 is one instruction)
    const float c2 = rsqrtf((float)dh) * 1.4426950408889634f;
    // key-padding mask: keys at positions >= Tk take no part in the softmax (Tk = T without a mask).  Their rows are not
    // read: their probability is 0, but 0 times an infinity or a NaN would not be.
    const int Tk = key_len ? min(max(key_len[b], 1), T) : T;

    bf16x8_t bq[C::KS];
    load_owned<DHP>(base, ld, q0, T, dh, lane, bq);

    f32x16_t accO[C::DT];
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) accO[dt][v] = 0.f;
    float m = -INFINITY, l = 0.f;

    // streamed mode (PIPE; trows == 64): the next 64-row tile is prefetched into registers during the products
    constexpr bool pipe = PIPE;
    TilePre<DHP> pk, pv;
    if constexpr (pipe) {
        tile_fetch<DHP>(pk, base + D, ld, 0, Tk, dh);
        tile_fetch<DHP>(pv, base + 2 * D, ld, 0, Tk, dh);
    }
    for (int t0 = 0; t0 < Tk; t0 += trows) {
      __syncthreads();
      if constexpr (pipe) {
          tile_store<DHP>(Ks0, pk);
          tile_store<DHP>(Vs0, pv);
      } else {
          load_tile<DHP>(Ks0, base + D, ld, t0, Tk, dh, trows);
          load_tile<DHP>(Vs0, base + 2 * D, ld, t0, Tk, dh, trows);
      }
      __syncthreads();
      if (pipe) if (t0 + trows < Tk) {
          tile_fetch<DHP>(pk, base + D, ld, t0 + trows, Tk, dh);
          tile_fetch<DHP>(pv, base + 2 * D, ld, t0 + trows, Tk, dh);
      }
      for (int k0 = t0; k0 < min(Tk, t0 + trows); k0 += AT_ROWS) {
        const uint16_t* Ks = Ks0 + (k0 - t0) * C::PITCH;
        const uint16_t* Vs = Vs0 + (k0 - t0) * C::PITCH;
        const int nt = (Tk - k0 > 32) ? 2 : 1;
        float s[2][16];
        float mloc = -INFINITY;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (t < nt) {
                f32x16_t acc;
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[v] = 0.f;
                const uint16_t* kp = Ks + (t * 32 + (lane & 31)) * C::PITCH + 8 * g;
#pragma unroll
                for (int ks = 0; ks < C::KS; ++ks)
                    acc = mfma32(*reinterpret_cast<const bf16x8_t*>(kp + 16 * ks), bq[ks], acc);
                if (k0 + t * 32 + 32 <= Tk) {               // whole tile inside the sequence: no masking
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        s[t][v] = acc[v] * c2;
                        mloc = fmaxf(mloc, s[t][v]);
                    }
                } else {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int key = k0 + t * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
                        s[t][v] = (key < Tk) ? acc[v] * c2 : -INFINITY;
                        mloc = fmaxf(mloc, s[t][v]);
                    }
                }
            }
        }
        mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64));
        const float mn = fmaxf(m, mloc);
        const float corr = __builtin_amdgcn_exp2f(m - mn);
        float lsum = 0.f;
#pragma unroll
        for (int t = 0; t < 2; ++t)
            if (t < nt) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    s[t][v] = __builtin_amdgcn_exp2f(s[t][v] - mn);
                    lsum += s[t][v];
                }
            }
        lsum += __shfl_xor(lsum, 32, 64);
        l = l * corr + lsum;
        m = mn;
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) accO[dt][v] *= corr;
#pragma unroll
        for (int t = 0; t < 2; ++t)
            if (t < nt) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const bf16x8_t pb = pack8(&s[t][8 * c]);
#pragma unroll
                    for (int dt = 0; dt < C::DT; ++dt) {
                        const bf16x8_t a = tr_frag<4, 8>(Vs, C::PITCH, t * 32 + 16 * c, dt * 32, lane);
                        accO[dt] = mfma32(a, pb, accO[dt]);
                    }
                }
            }
      }
    }
    // O^T tile: lane holds query q0 + l%32, features dt*32 + 8*(v/4) + 4g + v%4
    const int q = q0 + (lane & 31);
    if (q < T) {
        const float inv = 1.f / l;
        bf16* orow = o + ((int64_t)b * T + q) * D + h * dh;
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const int d = dt * 32 + 8 * v4 + 4 * g;
                if (d < dh)
                    store4_bf16(orow + d, accO[dt][4 * v4] * inv, accO[dt][4 * v4 + 1] * inv,
                                accO[dt][4 * v4 + 2] * inv, accO[dt][4 * v4 + 3] * inv);
            }
        if (g == 0) lse[(int64_t)bh * T + q] = (m + __log2f(l)) * 0.6931471805599453f;   // back to natural log
    }
}

// ----------------------------------------------------------------------------------------
// backward pass 1: dQ and delta (wavefront owns 32 query rows)
// ----------------------------------------------------------------------------------------
template <int DHP, bool PIPE>
__global__ __launch_bounds__(512) void attn_bwd_dq_mfma(const bf16* __restrict__ qkv, const bf16* __restrict__ o,
                                                        const bf16* __restrict__ dout, const float* __restrict__ lse,
                                                        bf16* __restrict__ dqkv, float* __restrict__ delta,
                                                        const int* __restrict__ key_len, int T, int H, int dh, int trows) {
    using C = AtCfg<DHP>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint16_t* Ks0 = reinterpret_cast<uint16_t*>(smem);
    uint16_t* Vs0 = Ks0 + trows * C::PITCH;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int g = lane >> 5;
    const int bh = blockIdx.y, b = bh / H, h = bh % H;
    const int D = H * dh;
    const int64_t ld = 3 * (int64_t)D;
    const bf16* base = qkv + (int64_t)b * T * ld + h * dh;
    const bf16* dob = dout + (int64_t)b * T * D + h * dh;
    const bf16* ob = o + (int64_t)b * T * D + h * dh;
    const int q0 = (blockIdx.x * nw + wave) * 32;
    const int q = q0 + (lane & 31), qc = min(q, T - 1);
    const float scale = rsqrtf((float)dh);
    const float c2 = scale * 1.4426950408889634f;
    // key-padding mask: keys at positions >= Tk take no part in the softmax (Tk = T without a mask).  Their rows are not
    // read: their probability is 0, but 0 times an infinity or a NaN would not be.
    const int Tk = key_len ? min(max(key_len[b], 1), T) : T;

    bf16x8_t bq[C::KS], bdo[C::KS];
    load_owned<DHP>(base, ld, q0, T, dh, lane, bq);
    load_owned<DHP>(dob, D, q0, T, dh, lane, bdo);
    // delta_q = sum_d dO[q,d] * O[q,d]; the two half-wavefronts hold complementary feature slots
    float dl = 0.f;
    {
        bf16x8_t bo[C::KS];
        load_owned<DHP>(ob, D, q0, T, dh, lane, bo);
#pragma unroll
        for (int ks = 0; ks < C::KS; ++ks)
#pragma unroll
            for (int e = 0; e < 8; ++e) dl += (float)bdo[ks][e] * (float)bo[ks][e];
        dl += __shfl_xor(dl, 32, 64);
    }
    const float L2 = lse[(int64_t)bh * T + qc] * 1.4426950408889634f;
    if (q < T && g == 0) delta[(int64_t)bh * T + q] = dl;

    f32x16_t accQ[C::DT];
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) accQ[dt][v] = 0.f;

    constexpr bool pipe = PIPE;
    TilePre<DHP> pk, pv;
    if constexpr (pipe) {
        tile_fetch<DHP>(pk, base + D, ld, 0, Tk, dh);
        tile_fetch<DHP>(pv, base + 2 * D, ld, 0, Tk, dh);
    }
    for (int t0 = 0; t0 < Tk; t0 += trows) {
      __syncthreads();
      if constexpr (pipe) {
          tile_store<DHP>(Ks0, pk);
          tile_store<DHP>(Vs0, pv);
      } else {
          load_tile<DHP>(Ks0, base + D, ld, t0, Tk, dh, trows);
          load_tile<DHP>(Vs0, base + 2 * D, ld, t0, Tk, dh, trows);
      }
      __syncthreads();
      if (pipe) if (t0 + trows < Tk) {
          tile_fetch<DHP>(pk, base + D, ld, t0 + trows, Tk, dh);
          tile_fetch<DHP>(pv, base + 2 * D, ld, t0 + trows, Tk, dh);
      }
      for (int k0 = t0; k0 < min(Tk, t0 + trows); k0 += AT_ROWS) {
        const uint16_t* Ks = Ks0 + (k0 - t0) * C::PITCH;
        const uint16_t* Vs = Vs0 + (k0 - t0) * C::PITCH;
        const int nt = (Tk - k0 > 32) ? 2 : 1;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (t < nt) {
                f32x16_t aS, aP;
#pragma unroll
                for (int v = 0; v < 16; ++v) { aS[v] = 0.f; aP[v] = 0.f; }
                const uint16_t* kp = Ks + (t * 32 + (lane & 31)) * C::PITCH + 8 * g;
                const uint16_t* vp = Vs + (t * 32 + (lane & 31)) * C::PITCH + 8 * g;
#pragma unroll
                for (int ks = 0; ks < C::KS; ++ks) {
                    aS = mfma32(*reinterpret_cast<const bf16x8_t*>(kp + 16 * ks), bq[ks], aS);
                    aP = mfma32(*reinterpret_cast<const bf16x8_t*>(vp + 16 * ks), bdo[ks], aP);
                }
                // dS without its 1/sqrt(head_dim): that factor is applied once to the finished dQ
                float ds[16];
                if (k0 + t * 32 + 32 <= Tk) {
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        ds[v] = __builtin_amdgcn_exp2f(aS[v] * c2 - L2) * (aP[v] - dl);
                } else {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int key = k0 + t * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
                        ds[v] = (key < Tk) ? __builtin_amdgcn_exp2f(aS[v] * c2 - L2) * (aP[v] - dl) : 0.f;
                    }
                }
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const bf16x8_t dsb = pack8(&ds[8 * c]);
#pragma unroll
                    for (int dt = 0; dt < C::DT; ++dt) {
                        const bf16x8_t a = tr_frag<4, 8>(Ks, C::PITCH, t * 32 + 16 * c, dt * 32, lane);
                        accQ[dt] = mfma32(a, dsb, accQ[dt]);
                    }
                }
            }
        }
      }
    }
    if (q < T) {
        bf16* dq = dqkv + ((int64_t)b * T + q) * ld + h * dh;
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const int d = dt * 32 + 8 * v4 + 4 * g;
                if (d < dh)
                    store4_bf16(dq + d, accQ[dt][4 * v4] * scale, accQ[dt][4 * v4 + 1] * scale,
                                accQ[dt][4 * v4 + 2] * scale, accQ[dt][4 * v4 + 3] * scale);
            }
    }
}

// ----------------------------------------------------------------------------------------
// backward pass 2: dK and dV (wavefront owns 32 key rows)
// ----------------------------------------------------------------------------------------
template <int DHP, bool PIPE>
__global__ __launch_bounds__(512) void attn_bwd_dkv_mfma(const bf16* __restrict__ qkv, const bf16* __restrict__ dout,
                                                         const float* __restrict__ lse, const float* __restrict__ delta,
                                                         bf16* __restrict__ dqkv, const int* __restrict__ key_len,
                                                         int T, int H, int dh, int trows) {
    using C = AtCfg<DHP>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint16_t* Qs0 = reinterpret_cast<uint16_t*>(smem);
    uint16_t* Os0 = Qs0 + trows * C::PITCH;                       // dO tile
    float* lse_s0 = reinterpret_cast<float*>(Os0 + trows * C::PITCH);
    float* del_s0 = lse_s0 + trows;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int g = lane >> 5;
    const int bh = blockIdx.y, b = bh / H, h = bh % H;
    const int D = H * dh;
    const int64_t ld = 3 * (int64_t)D;
    const bf16* base = qkv + (int64_t)b * T * ld + h * dh;
    const bf16* dob = dout + (int64_t)b * T * D + h * dh;
    const int j0 = (blockIdx.x * nw + wave) * 32;
    const float scale = rsqrtf((float)dh);
    const float c2 = scale * 1.4426950408889634f;
    const int Tk = key_len ? min(max(key_len[b], 1), T) : T;      // keys beyond Tk are masked: their dK, dV are zero

    bf16x8_t bk[C::KS], bv[C::KS];
    load_owned<DHP>(base + D, ld, j0, T, dh, lane, bk);
    load_owned<DHP>(base + 2 * D, ld, j0, T, dh, lane, bv);

    f32x16_t accK[C::DT], accV[C::DT];
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) { accK[dt][v] = 0.f; accV[dt][v] = 0.f; }

    constexpr bool pipe = PIPE;
    TilePre<DHP> pq, po;
    float pre_l = 0.f, pre_d = 0.f;                                  // row statistics of the prefetched tile (thread r < 64: row r)
    auto stats_fetch = [&](int row0) {
        const int i = row0 + (int)threadIdx.x;
        if ((int)threadIdx.x < AT_ROWS) {
            pre_l = (i < T) ? lse[(int64_t)bh * T + i] * 1.4426950408889634f : INFINITY;
            pre_d = (i < T) ? delta[(int64_t)bh * T + i] : 0.f;
        }
    };
    if constexpr (pipe) {
        tile_fetch<DHP>(pq, base, ld, 0, T, dh);
        tile_fetch<DHP>(po, dob, D, 0, T, dh);
        stats_fetch(0);
    }
    for (int t0 = 0; t0 < T; t0 += trows) {
      __syncthreads();
      if constexpr (pipe) {
          tile_store<DHP>(Qs0, pq);
          tile_store<DHP>(Os0, po);
          if ((int)threadIdx.x < AT_ROWS) { lse_s0[threadIdx.x] = pre_l; del_s0[threadIdx.x] = pre_d; }
      } else {
          load_tile<DHP>(Qs0, base, ld, t0, T, dh, trows);
          load_tile<DHP>(Os0, dob, D, t0, T, dh, trows);
          for (int r = threadIdx.x; r < trows; r += blockDim.x) {
              const int i = t0 + r;
              // log-sum-exp in the base-2 domain; +inf masks rows beyond the sequence (exp2(. - inf) = 0)
              lse_s0[r] = (i < T) ? lse[(int64_t)bh * T + i] * 1.4426950408889634f : INFINITY;
              del_s0[r] = (i < T) ? delta[(int64_t)bh * T + i] : 0.f;
          }
      }
      __syncthreads();
      if (pipe) if (t0 + trows < T) {
          tile_fetch<DHP>(pq, base, ld, t0 + trows, T, dh);
          tile_fetch<DHP>(po, dob, D, t0 + trows, T, dh);
          stats_fetch(t0 + trows);
      }
      for (int i0 = t0; i0 < min(T, t0 + trows); i0 += AT_ROWS) {
        const uint16_t* Qs = Qs0 + (i0 - t0) * C::PITCH;
        const uint16_t* Os = Os0 + (i0 - t0) * C::PITCH;
        const float* lse_s = lse_s0 + (i0 - t0);
        const float* del_s = del_s0 + (i0 - t0);
        const int nt = (T - i0 > 32) ? 2 : 1;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (t < nt) {
                f32x16_t aS, aP;
#pragma unroll
                for (int v = 0; v < 16; ++v) { aS[v] = 0.f; aP[v] = 0.f; }
                const uint16_t* qp = Qs + (t * 32 + (lane & 31)) * C::PITCH + 8 * g;
                const uint16_t* op = Os + (t * 32 + (lane & 31)) * C::PITCH + 8 * g;
#pragma unroll
                for (int ks = 0; ks < C::KS; ++ks) {
                    aS = mfma32(*reinterpret_cast<const bf16x8_t*>(qp + 16 * ks), bk[ks], aS);
                    aP = mfma32(*reinterpret_cast<const bf16x8_t*>(op + 16 * ks), bv[ks], aP);
                }
                // lane: key j0 + l%32; rows i = i0 + t*32 + 8*(v/4) + 4g + v%4
                float p[16], ds[16];
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) {
                    const int r = t * 32 + 8 * v4 + 4 * g;
                    const float4 Lr = *reinterpret_cast<const float4*>(lse_s + r);
                    const float4 Dr = *reinterpret_cast<const float4*>(del_s + r);
                    const float Lv[4] = {Lr.x, Lr.y, Lr.z, Lr.w};
                    const float Dv[4] = {Dr.x, Dr.y, Dr.z, Dr.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int v = 4 * v4 + e;
                        p[v] = __builtin_amdgcn_exp2f(aS[v] * c2 - Lv[e]);
                        ds[v] = p[v] * (aP[v] - Dv[e]);          // 1/sqrt(head_dim) applied to the finished dK
                    }
                }
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const bf16x8_t pb = pack8(&p[8 * c]);
                    const bf16x8_t dsb = pack8(&ds[8 * c]);
#pragma unroll
                    for (int dt = 0; dt < C::DT; ++dt) {
                        const bf16x8_t ao = tr_frag<4, 8>(Os, C::PITCH, t * 32 + 16 * c, dt * 32, lane);
                        accV[dt] = mfma32(ao, pb, accV[dt]);
                        const bf16x8_t aq = tr_frag<4, 8>(Qs, C::PITCH, t * 32 + 16 * c, dt * 32, lane);
                        accK[dt] = mfma32(aq, dsb, accK[dt]);
                    }
                }
            }
        }
      }
    }
    const int j = j0 + (lane & 31);
    if (j >= Tk) {                       // a masked key: no query looked at it
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) { accK[dt][v] = 0.f; accV[dt][v] = 0.f; }
    }
    if (j < T) {
        bf16* dk = dqkv + ((int64_t)b * T + j) * ld + D + h * dh;
        bf16* dv = dk + D;
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const int d = dt * 32 + 8 * v4 + 4 * g;
                if (d < dh) {
                    store4_bf16(dk + d, accK[dt][4 * v4] * scale, accK[dt][4 * v4 + 1] * scale,
                                accK[dt][4 * v4 + 2] * scale, accK[dt][4 * v4 + 3] * scale);
                    store4_bf16(dv + d, accV[dt][4 * v4], accV[dt][4 * v4 + 1], accV[dt][4 * v4 + 2], accV[dt][4 * v4 + 3]);
                }
            }
    }
}

// ----------------------------------------------------------------------------------------
// launchers
// ----------------------------------------------------------------------------------------
// Wavefronts per workgroup: split the ceil(T/32) row tiles evenly over as few workgroups as
// 8 wavefronts each allow (T=197: 1 x 7, T=257: 2 x 5, T=512: 2 x 8).
#define RC_LDS(expr) do { int _rc = (expr); if (_rc != REV_OK) return _rc; } while (0)

static void row_split(int T, int* nblk, int* nw) {
    const int tiles = (T + 31) / 32;
    *nblk = (tiles + 7) / 8;
    *nw = (tiles + *nblk - 1) / *nblk;
}

// Rows of the streamed operands kept in LDS at a time: every (32-padded) row of the head when two such
// tiles plus the row statistics fit in 128 KB -- then a workgroup loads once and never synchronises
// again (measured faster than streaming even where only one such workgroup fits a CU: 257 tokens at
// head_dim 80) -- otherwise 64-row tiles.
template <int DHP>
static int tile_rows(int T) {
    const int all = (T + 31) / 32 * 32;
    const size_t bytes = (size_t)2 * all * AtCfg<DHP>::PITCH * sizeof(uint16_t) + 2 * all * sizeof(float);
    return bytes <= 128 * 1024 ? all : AT_ROWS;
}

template <typename K>
static int raise_lds(K kern, size_t shmem) {
    if (shmem > 64 * 1024)
        REV_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    return REV_OK;
}

template <int DHP>
static int fwd_launch(hipStream_t s, const bf16* qkv, bf16* o, float* lse, int B, int T, int H, int dh, const int* key_len) {
    int nblk, nw;
    row_split(T, &nblk, &nw);
    const int trows = tile_rows<DHP>(T);
    const size_t shmem = (size_t)2 * trows * AtCfg<DHP>::PITCH * sizeof(uint16_t);
    // (the register prefetch of the streamed mode costs the forward kernel one resident wavefront per
    // SIMD and measured slower there; the backward kernels gain 20 % from it)
    RC_LDS(raise_lds(attn_fwd_mfma<DHP, false>, shmem));
    hipLaunchKernelGGL((attn_fwd_mfma<DHP, false>), dim3(nblk, B * H), dim3(nw * 64), shmem, s, qkv, o, lse, key_len, T, H, dh, trows);
    REV_HIP(hipGetLastError());
    return REV_OK;
}

template <int DHP>
static int bwd_launch(hipStream_t s, const bf16* qkv, const bf16* o, const bf16* dout, const float* lse, bf16* dqkv,
                      float* delta, int B, int T, int H, int dh, const int* key_len, bool solo) {
    int nblk, nw;
    row_split(T, &nblk, &nw);
    // A head's row tiles are split over 4-wavefront workgroups: the backward kernels need 160-210 registers, so only
    // one 5...8-wavefront workgroup fits a CU but three (two) of 4 wavefronts do -- 4 % (197 tokens) to 12 % (257
    // tokens) faster alone.  Next to another stream's kernels the extra resident workgroups cost the neighbour; measured
    // in the parallel schedule: 257 tokens (9 row tiles) +1.9 % with the split, 512 tokens (16 row tiles) -0.7 %, so
    // there it is taken up to 12 row tiles.  A wavefront's work does not depend on the grouping, so the results are
    // bit-identical.
    if ((solo || (T + 31) / 32 <= 12) && nw > 4) {
        nblk = ((T + 31) / 32 + 3) / 4;
        nw = 4;
    }
    // With 4 or more wavefronts the backward kernels always stream 64-row tiles with the next tile
    // prefetched into registers: measured 6-8 % faster than keeping the head resident (197 and 257
    // tokens), with a fifth of the LDS, which also leaves room for a co-running kernel of the other stream.
    const int trows = (nw >= 4) ? AT_ROWS : tile_rows<DHP>(T);
    const size_t shmem = (size_t)2 * trows * AtCfg<DHP>::PITCH * sizeof(uint16_t);
    const size_t shmem2 = shmem + 2 * trows * sizeof(float);
    if (trows == AT_ROWS && nw >= 4) {          // streamed mode with register prefetch of the next tile
        hipLaunchKernelGGL((attn_bwd_dq_mfma<DHP, true>), dim3(nblk, B * H), dim3(nw * 64), shmem, s, qkv, o, dout, lse, dqkv,
                           delta, key_len, T, H, dh, trows);
        hipLaunchKernelGGL((attn_bwd_dkv_mfma<DHP, true>), dim3(nblk, B * H), dim3(nw * 64), shmem2, s, qkv, dout, lse, delta,
                           dqkv, key_len, T, H, dh, trows);
    } else {
        RC_LDS(raise_lds(attn_bwd_dq_mfma<DHP, false>, shmem));
        RC_LDS(raise_lds(attn_bwd_dkv_mfma<DHP, false>, shmem2));
        hipLaunchKernelGGL((attn_bwd_dq_mfma<DHP, false>), dim3(nblk, B * H), dim3(nw * 64), shmem, s, qkv, o, dout, lse, dqkv,
                           delta, key_len, T, H, dh, trows);
        hipLaunchKernelGGL((attn_bwd_dkv_mfma<DHP, false>), dim3(nblk, B * H), dim3(nw * 64), shmem2, s, qkv, dout, lse, delta,
                           dqkv, key_len, T, H, dh, trows);
    }
    REV_HIP(hipGetLastError());
    return REV_OK;
}

static bool mfma_ok(const void* a, const void* b, const void* c, const void* d) {
    return (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c | (uintptr_t)d) & 15) == 0;
}

template <>
int attention_forward<bf16>(hipStream_t s, const bf16* qkv, bf16* o, float* lse, int B, int T, int H, int dh, const int* key_len) {
    if ((dh & 7) || dh > 128 || !mfma_ok(qkv, o, nullptr, nullptr))
        { set_error("attention: head_dim must be a multiple of 8 up to 128 and every buffer 16-byte aligned"); return REV_EINVAL; }
    ProfScope ps(K_ATTN_FWD, s, 4.0 * B * H * (double)T * T * dh);
    if (attention_dma_takes(dh)) return attention_forward_dma(s, qkv, o, lse, B, T, H, dh, key_len);
    if (dh <= 32) return fwd_launch<32>(s, qkv, o, lse, B, T, H, dh, key_len);
    if (dh <= 64) return fwd_launch<64>(s, qkv, o, lse, B, T, H, dh, key_len);
    if (dh <= 96) return fwd_launch<96>(s, qkv, o, lse, B, T, H, dh, key_len);
    return fwd_launch<128>(s, qkv, o, lse, B, T, H, dh, key_len);
}
template <>
int attention_forward<float>(hipStream_t s, const float* qkv, float* o, float* lse, int B, int T, int H, int dh, const int* key_len) {
    return attention_forward_f32(s, qkv, o, lse, B, T, H, dh, key_len);
}

template <>
int attention_backward<bf16>(hipStream_t s, const bf16* qkv, const bf16* o, const bf16* dout, const float* lse,
                             bf16* dqkv, float* delta, int B, int T, int H, int dh, const int* key_len, bool solo) {
    if ((dh & 7) || dh > 128 || !mfma_ok(qkv, o, dout, dqkv)) {
        set_error("attention: head_dim must be a multiple of 8 up to 128 and every buffer 16-byte aligned");
        return REV_EINVAL;
    }
    // Heads wider than 96 take the float32 products: the bf16 dK/dV kernel would need more registers
    // than a wavefront has for a 128-wide head (it spilled).
    if (dh > 96) return attention_backward_f32<bf16>(s, qkv, o, dout, lse, dqkv, B, T, H, dh, key_len);
    ProfScope ps(K_ATTN_BWD, s, 8.0 * B * H * (double)T * T * dh);
    if (attention_dma_takes(dh)) return attention_backward_dma(s, qkv, o, dout, lse, dqkv, delta, B, T, H, dh, key_len);
    if (dh <= 32) return bwd_launch<32>(s, qkv, o, dout, lse, dqkv, delta, B, T, H, dh, key_len, solo);
    if (dh <= 64) return bwd_launch<64>(s, qkv, o, dout, lse, dqkv, delta, B, T, H, dh, key_len, solo);
    return bwd_launch<96>(s, qkv, o, dout, lse, dqkv, delta, B, T, H, dh, key_len, solo);
}
template <>
int attention_backward<float>(hipStream_t s, const float* qkv, const float* o, const float* dout, const float* lse,
                              float* dqkv, float*, int B, int T, int H, int dh, const int* key_len, bool) {
    return attention_backward_f32<float>(s, qkv, o, dout, lse, dqkv, B, T, H, dh, key_len);
}

}  // namespace rev
