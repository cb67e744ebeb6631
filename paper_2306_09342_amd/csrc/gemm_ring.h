// bf16 GEMM for launches too small to fill the chip with the tiles of the two-stage kernel:
//   C[M,N] (+epilogue) = A[M,K] * B[N,K]^T   or, with BKM,   A[M,K] * B[K,N].
//
// A workgroup owns one small output tile and walks the WHOLE contraction, in the order of the two-stage kernel, through a
// deep ring of stages in LDS: all its wavefronts request the stages (direct-to-LDS loads), WM x WN of them multiply, 32*TM x 32*TN
// each.  One barrier per stage says both that a stage has landed and that the stage before it has been read; a
// stage's fragments are read while the products of the stage before run.  Every output element is the sum of the same
// products in the same order as under every other tile, so the choice of the tile never changes a bit of the result.
//
// What bounds it: the rate at which a CU takes in operands, (BM + BN) * K * 2 bytes per workgroup, the LDS reads of a wavefront (38
// cycles each, whoever else reads), and for the smallest tile the chain of its products; all behind about 2.5 us of launch, first
// latency and epilogue.  The requests of a stage and its reads are spread between the products, so that the three run
// side by side; a fragment's registers are refilled as soon as its products are issued, one stage ahead, which leaves room for 96 rows
// of sums and the epilogue's operand per wavefront.  64x128 tiles and larger have eight wavefronts, two per SIMD, and a CU to
// themselves.
// Measured (us, operands from the memory-side cache).  197 rows, N = 768, K = 3072: 8.4 (whole-K 64x128 tiles in two stages: 28; wavefronts that
// split K, whose sums depended on the row count, 7.0); K = 768: 4.8.  One workgroup per CU or less against two-stage tiles, two
// workgroups per CU, K = 3072, N = 768, input gradient: 1576 rows 64x128 16.6 (64x64 with four wavefronts 23.2); 3152 rows 128x128 21.8
// (33.3); 6304 rows 192x128 32.6 (40.3).  Requests at the head of a stage: 128x128 23.9.  Three stages of 192x128 instead of four: 34.8.
// 256x128 with three: as 128x128 tiles in two stages, not kept.
#pragma once
#include "gemm_epilogue.h"
#include <algorithm>
#include <type_traits>

namespace rev {

// SUB: 64-wide chunks of K per stage, NS: stages in the ring
template <int TM, int TN, int WM, int WN, int SUB, int NS> struct RingCfg {
    static constexpr int NW = WM * WN > 4 ? WM * WN : 4;
    static constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN;
    static constexpr int LA = BM / 8, LB = BN / 8, LPC = LA + LB, LPW = SUB * LPC / NW;   // 1 KB loads: per chunk, per wavefront and stage
    static constexpr int A_BYTES = BM * 128, CHUNK = (BM + BN) * 128, STAGE = SUB * CHUNK;
    static constexpr int PITCH = BN + 4;
    static constexpr int OUT_BYTES = BM * PITCH * 4, RING_BYTES = NS * STAGE;
    static constexpr int SHMEM = RING_BYTES > OUT_BYTES ? RING_BYTES : OUT_BYTES;
    static_assert(LA % NW == 0 && LB % NW == 0 && WM * WN <= NW && (NS - 2) * LPW < 64, "RingCfg");
    template <int EPI, bool AKM, bool BKM>                      // gemm_ring_tile
    __device__ __forceinline__ static void tile(const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K, const Epi& epi, int m0, int n0);
};

// The tile at (m0, n0), multiples of its size (the same for all threads).  AKM, BKM: the operand is stored contraction-major, [K, ld].
template <int TM, int TN, int WM, int WN, int SUB, int NS, int EPI, bool AKM, bool BKM>
__device__ __forceinline__ void gemm_ring_tile(const bf16* __restrict__ A, int64_t lda, const bf16* __restrict__ B, int64_t ldb, int M, int N,
                                               int K, const Epi& epi, int m0, int n0) {
    using C = RingCfg<TM, TN, WM, WN, SUB, NS>;
    constexpr int KIND = EPI & ~EPI_ERF;
    constexpr int BM = C::BM, BN = C::BN, NW = C::NW, LPW = C::LPW;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, fr = lane & 31;
    const bool computes = wave < WM * WN;
    const int wm = wave / WN, wn = wave % WN;
    const unsigned lds0 = (unsigned)(uintptr_t)LDS_PTR(unsigned char, smem);

    // ---- this wavefront's loads of a stage: a scalar base per operand, advanced along K, and a 32-bit byte offset per lane.
    // Row-wise tiles: 8 rows of 8 chunks of 16 bytes, chunk c of row r at position c ^ ((r >> 1) & 7).  K-major B: rows of
    // BN columns, as they lie (swizzled for BN >= 64).  Rows / columns beyond the matrix re-read valid ones (never stored);
    // what lies beyond K comes from a block of zeros, for both operands.
    auto swz = [](int cols, int r) { return cols >= 128 ? 4 * (r & 3) : (cols == 64 ? 4 * ((r >> 1) & 1) : 0); };
    unsigned voff[LPW];
    int kidx[LPW];                                              // first k (within a chunk) that the lane fetches
#pragma unroll
    for (int t = 0; t < LPW; ++t) {
        const int i = (wave + NW * t) % C::LPC;
        const bool isA = (NW * t) % C::LPC < C::LA;             // the same for all wavefronts: LA and LPC are multiples of NW
        const int ii = isA ? i : i - C::LA;
        const int64_t ld = isA ? lda : ldb;
        const int left = isA ? M - m0 : N - n0;
        if (!(isA ? AKM : BKM)) {
            const int row = ii * 8 + (lane >> 3), ch = (lane & 7) ^ ((row >> 1) & 7);
            kidx[t] = ch * 8;
            voff[t] = (unsigned)(min(row, left - 1) * ld * 2 + ch * 16);
        } else {
            const int cpr = (isA ? BM : BN) / 8, row = ii * (64 / cpr) + lane / cpr, col = ((lane % cpr) ^ swz(isA ? BM : BN, row)) * 8;
            kidx[t] = row;
            voff[t] = (unsigned)(row * ld * 2 + min(col, left - 8) * 2);
        }
    }
    const char* a_base = reinterpret_cast<const char*>(AKM ? A + m0 : A + (int64_t)m0 * lda);
    const char* b_base = reinterpret_cast<const char*>(BKM ? B + n0 : B + (int64_t)n0 * ldb);
    const char* zero = reinterpret_cast<const char*>(g_zero_chunk);
    const int nst = (K + 64 * SUB - 1) / (64 * SUB);
    const int nfull = K / (64 * SUB);                           // stages that lie within K
    // requests t0 .. t1 - 1 of the wavefront's LPW of a stage
    auto issue = [&](int st, auto full_tag, int t0, int t1) {
        const unsigned sb = lds0 + ((unsigned)st % NS) * C::STAGE;
#pragma unroll
        for (int t = t0; t < t1; ++t) {
            const int sub = (NW * t) / C::LPC, k0 = (st * SUB + sub) * 64;
            const bool isA = (NW * t) % C::LPC < C::LA;
            const char* base = isA ? a_base + (AKM ? (int64_t)k0 * lda * 2 : (int64_t)k0 * 2) : b_base + (BKM ? (int64_t)k0 * ldb * 2 : (int64_t)k0 * 2);
            const unsigned dst = sb + (wave + NW * t) * 1024;
            if (decltype(full_tag)::value) dma16_sbase(base, voff[t], dst);
            else dma16_ptr(k0 + kidx[t] < K ? base + voff[t] : zero, dst);
        }
    };
    auto issue_any = [&](int st) {
        if (st < nfull) issue(st, std::true_type{}, 0, LPW);
        else if (st < nst) issue(st, std::false_type{}, 0, LPW);
    };

    // ---- epilogue geometry; its operands do not depend on the products: requested first, landed long before use ----
    constexpr int QPR = BN / 4, ROWS = NW * 64 / QPR, PASS = BM / ROWS;       // threads per row, rows per pass
    const int c4 = tid % QPR, rr = tid / QPR, n = n0 + 4 * c4;
    constexpr bool AHEAD_OPND = PASS <= 16;
    f32x4_t bv = {0.f, 0.f, 0.f, 0.f}, opnd[PASS];
    if (n < N) {
        if (KIND == EPI_BIAS || KIND == EPI_BIAS_GELU || KIND == EPI_RESIDUAL)
            bv = ld_bf16x4(reinterpret_cast<const bf16*>(epi.bias) + n);
        if (AHEAD_OPND)
#pragma unroll
            for (int p = 0; p < PASS; ++p) opnd[p] = epi_load4<KIND>(epi, min(m0 + rr + p * ROWS, M - 1), n);
    }
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) issue_any(s);

    // ---- fragments ----
    constexpr int KK = 4 * SUB;                                 // product steps per stage
    unsigned a_off[4], b_off[4], at_off[TM], bt_off[TN];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const int koff = ((2 * kk + g) ^ ((fr >> 1) & 7)) << 4;
        a_off[kk] = (wm * TM * 32 + fr) * 128 + koff;
        b_off[kk] = C::A_BYTES + (wn * TN * 32 + fr) * 128 + koff;
    }
    if (AKM || BKM) {
        const int jj = lane & 15, q = lane >> 4;
        const int r = (q >> 1) * 8 + (jj >> 2);                 // rows r and r + 4 are swizzled alike
        auto offset = [&](int cols, int tile) {
            const int c = tile * 32 + (q & 1) * 16 + 4 * (jj & 3);
            return r * (cols * 2) + (((c >> 3) ^ swz(cols, r)) << 4) + (c & 7) * 2;
        };
#pragma unroll
        for (int i = 0; i < TM; ++i) at_off[i] = offset(BM, wm * TM + i);
#pragma unroll
        for (int j = 0; j < TN; ++j) bt_off[j] = C::A_BYTES + offset(BN, wn * TN + j);
    }
    auto tr_read = [&](const unsigned char* q, int cols) {
        union { struct { s16x4_t lo, hi; } s; bf16x8_t v; } u;
        u.s.lo = lds_tr16(reinterpret_cast<const uint16_t*>(q));
        u.s.hi = lds_tr16(reinterpret_cast<const uint16_t*>(q + 4 * (cols * 2)));
        return u.v;
    };
    bf16x8_t fa[KK][TM], fb[KK][TN];
    auto read = [&](int kk, int st) {
        const unsigned char* p = smem + ((unsigned)st % NS) * C::STAGE + (kk >> 2) * C::CHUNK;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if (AKM) fa[kk][i] = tr_read(p + at_off[i] + (kk & 3) * 16 * (BM * 2), BM);
            else fa[kk][i] = *reinterpret_cast<const bf16x8_t*>(p + a_off[kk & 3] + i * 32 * 128);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (BKM) fb[kk][j] = tr_read(p + bt_off[j] + (kk & 3) * 16 * (BN * 2), BN);
            else fb[kk][j] = *reinterpret_cast<const bf16x8_t*>(p + b_off[kk & 3] + j * 32 * 128);
        }
    };
    f32x16_t acc[TN][TM];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.f;
    auto products = [&](int kk) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i) acc[j][i] = mfma32(fb[kk][j], fa[kk][i], acc[j][i]);
    };
    // This wavefront's loads of a stage have landed, with those of the AHEAD stages after it still under way, and its LDS
    // reads have returned; then the same for everybody.
    auto landed = [&](auto ahead_tag) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(decltype(ahead_tag)::value * LPW));
        asm volatile("s_barrier" ::: "memory");
    };
    using Ahead = std::integral_constant<int, NS - 2>;
    // A stage: step by step, the products of the stage before it, then the fragments for the next time in their place, then a
    // share of the requests, which held up the reads behind them where all came first (64x64 tiles, two workgroups per CU: the
    // other way round, 10.7 and 13.3 us at 197 rows, N = 768, K = 3072).
    // A stage whose refill (of the stage read last, before the barrier) lies within K ...
    constexpr bool SPREAD = C::NW > 4;
    auto step = [&](int st) {
        landed(Ahead{});
        if (!SPREAD || !computes) issue(st + NS - 1, std::true_type{}, 0, LPW);
        if (computes) {
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                products(kk);
                __builtin_amdgcn_sched_barrier(0);
                read(kk, st);
                if (SPREAD) issue(st + NS - 1, std::true_type{}, LPW * kk / KK, LPW * (kk + 1) / KK);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // ... and one near the end, or the first
    auto end_step = [&](int st) {
        const int ahead = nst - 1 - st;
        if (ahead >= NS - 2) landed(Ahead{});
        else if (ahead >= (NS - 2) / 2) landed(std::integral_constant<int, (NS - 2) / 2>{});
        else if (ahead >= 1) landed(std::integral_constant<int, 1>{});
        else landed(std::integral_constant<int, 0>{});
        issue_any(st + NS - 1);
        if (computes) {
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                if (st > 0) products(kk);
                read(kk, st);
            }
        }
    };
    end_step(0);
    int st = 1;
    for (; st + NS - 1 < nfull; ++st) step(st);
    for (; st < nst; ++st) end_step(st);
    if (computes) {
        const int last_steps = ((K + 63) / 64 - (nst - 1) * SUB) * 4;          // of the last stage
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
            if (kk < last_steps) products(kk);
    }

    // ---- the tile through LDS, out in full rows ----
    __syncthreads();                                            // the ring has been read
    float* ct = reinterpret_cast<float*>(smem);
    if (computes)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) {
                    const f32x4_t v = {acc[j][i][4 * vq], acc[j][i][4 * vq + 1], acc[j][i][4 * vq + 2], acc[j][i][4 * vq + 3]};
                    *reinterpret_cast<f32x4_t*>(ct + ((wm * TM + i) * 32 + fr) * C::PITCH + (wn * TN + j) * 32 + 8 * vq + 4 * g) = v;
                }
    __syncthreads();
    f32x4_t csum = {0.f, 0.f, 0.f, 0.f};
    if (n < N) {
#pragma unroll
        for (int p = 0; p < PASS; ++p) {
            const int r = rr + p * ROWS, m = m0 + r;
            if (m < M) {
                const f32x4_t v = *reinterpret_cast<const f32x4_t*>(ct + r * C::PITCH + 4 * c4);
                const f32x4_t x = AHEAD_OPND ? opnd[p] : epi_load4<KIND>(epi, m, n);
                const f32x4_t o = epi_store4<EPI>(epi, m, n, v, bv, x);
                if (KIND == EPI_GELU_BWD) csum += o;
            }
        }
    }
    // fused bias gradient: column sums of the tile's rows, one partial row per m-tile
    if (KIND == EPI_GELU_BWD && epi.colsum != nullptr) {
        __syncthreads();
        *reinterpret_cast<f32x4_t*>(ct + (rr * QPR + c4) * 4) = csum;
        __syncthreads();
        if (rr == 0 && n < N) {
            f32x4_t s = csum;
            for (int q = 1; q < ROWS; ++q) s += *reinterpret_cast<const f32x4_t*>(ct + (q * QPR + c4) * 4);
            *reinterpret_cast<f32x4_t*>(epi.colsum + (int64_t)(m0 / BM) * N + n) = s;
        }
    }
}

template <int TM, int TN, int WM, int WN, int SUB, int NS> template <int EPI, bool AKM, bool BKM>
__device__ __forceinline__ void RingCfg<TM, TN, WM, WN, SUB, NS>::tile(const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K,
                                                                       const Epi& epi, int m0, int n0) {
    gemm_ring_tile<TM, TN, WM, WN, SUB, NS, EPI, AKM, BKM>(A, lda, B, ldb, M, N, K, epi, m0, n0);
}

// Which way an XCD's run of tiles goes: the one in which it reads fewer rows of A and B.  (7289 x 384, K = 1536: 19.9 us down
// the columns, 18.8 along the rows.)
inline int ring_n_fast(int M, int N, int bm, int bn) {
    const int tm = (M + bm - 1) / bm, tn = (N + bn - 1) / bn, run = (tm * tn + 7) / 8;
    const int down = std::min(run, tm) * bm + (run + tm - 1) / tm * bn, along = std::min(run, tn) * bn + (run + tn - 1) / tn * bm;
    return along < down;
}
template <typename C>
__device__ __forceinline__ void ring_tile_at(int M, int N, int n_fast, int block, int blocks, int* m0, int* n0) {
    const int tiles_m = (M + C::BM - 1) / C::BM, tiles_n = (N + C::BN - 1) / C::BN, tile = xcd_remap(block, blocks);
    *n0 = __builtin_amdgcn_readfirstlane((n_fast ? tile % tiles_n : tile / tiles_m) * C::BN);
    *m0 = __builtin_amdgcn_readfirstlane((n_fast ? tile / tiles_n : tile % tiles_m) * C::BM);
}
using Ring32 = RingCfg<1, 1, 1, 1, 2, 4>;                      // 64 KB of LDS: two workgroups per CU
using Ring64 = RingCfg<1, 1, 2, 2, 1, 4>;

// One of the products of a launch that holds several.
struct RingPart { const bf16 *A, *B; int64_t lda, ldb; int N, K, n_fast, blocks; Epi epi; };
template <typename C, int EPI, bool BKM> __device__ __forceinline__ void ring_part(const RingPart& p, int M, int block) {
    int m0, n0;
    ring_tile_at<C>(M, p.N, p.n_fast, block, p.blocks, &m0, &n0);
    C::template tile<EPI, false, BKM>(p.A, p.lda, p.B, p.ldb, M, p.N, p.K, p.epi, m0, n0);
}
template <typename C> RingPart ring_part_of(const GemmCall<bf16>& c, int M) {
    return {c.A, c.B, c.lda, c.ldb, c.N, c.K, ring_n_fast(M, c.N, C::BM, C::BN), ((M + C::BM - 1) / C::BM) * ((c.N + C::BN - 1) / C::BN), c.epi};
}

}  // namespace rev
