// bf16 GEMM for launches too small to fill the chip with the tiles of the two-stage kernel:
//   C[M,N] (+epilogue) = A[M,K] * B[N,K]^T   or, with BKM,   A[M,K] * B[K,N].
//
// A workgroup owns one small output tile and walks the WHOLE contraction, in the order of the two-stage kernel, through a
// deep ring of stages in LDS: all its wavefronts request the stages (direct-to-LDS loads), WM x WN of them multiply, 32*TM x 32*TN
// each.  One barrier per stage says both that a stage has landed and that the stage before it has been read; a
// stage's fragments are read while the products of the stage before run.  Every output element is the sum of the same
// products in the same order as under every other tile, so the choice of the tile never changes a bit of the result.
//
// What bounds it: the rate at which a CU takes in operands, (BM + BN) * K * 2 bytes per workgroup at 50 to 80 GB/s, and for the
// smallest tile the chain of its products; both behind about 2.5 us of launch, first latency and epilogue.  The steady
// loop has no branch: with two per load and four per wait a stage took 0.38 us whatever its size, now 0.25.  Measured (197
// rows, operands from the memory-side cache, us): N = 768, K = 768: 4.4; K = 3072: 9.1 (whole-K 64x128 tiles in two stages: 8.3
// and 28; wavefronts that split K, whose sums depended on the row count: 3.6 and 7.0).  Six or eight stages measured the same or
// worse than three or four.
#include "gemm_epilogue.h"
#include <type_traits>

namespace rev {

// SUB: 64-wide chunks of K per stage, NS: stages in the ring
template <int TM, int TN, int WM, int WN, int SUB, int NS> struct RingCfg {
    static constexpr int NW = 4;
    static constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN;
    static constexpr int LA = BM / 8, LB = BN / 8, LPC = LA + LB, LPW = SUB * LPC / NW;   // 1 KB loads: per chunk, per wavefront and stage
    static constexpr int A_BYTES = BM * 128, CHUNK = (BM + BN) * 128, STAGE = SUB * CHUNK;
    static constexpr int PITCH = BN + 4;
    static constexpr int OUT_BYTES = BM * PITCH * 4, RING_BYTES = NS * STAGE;
    static constexpr int SHMEM = RING_BYTES > OUT_BYTES ? RING_BYTES : OUT_BYTES;
    static_assert(LA % NW == 0 && LB % NW == 0 && WM * WN <= NW && (NS - 2) * LPW < 64, "RingCfg");
};

template <int TM, int TN, int WM, int WN, int SUB, int NS, int EPI, bool BKM>
__global__ __launch_bounds__(256) void gemm_ring_kernel(const bf16* __restrict__ A, int64_t lda, const bf16* __restrict__ B, int64_t ldb,
                                                        int M, int N, int K, Epi epi) {
    using C = RingCfg<TM, TN, WM, WN, SUB, NS>;
    constexpr int KIND = EPI & ~EPI_ERF;
    constexpr int BM = C::BM, BN = C::BN, NW = C::NW, LPW = C::LPW;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, fr = lane & 31;
    const bool computes = wave < WM * WN;
    const int wm = wave / WN, wn = wave % WN;
    // m fastest: an XCD's run of tiles then reads each slice of B once and the (small) A from its L2
    const int tiles_m = (M + BM - 1) / BM;
    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    const int n0 = (tile / tiles_m) * BN, m0 = (tile % tiles_m) * BM;
    const unsigned lds0 = (unsigned)(uintptr_t)LDS_PTR(unsigned char, smem);

    // ---- this wavefront's loads of a stage: a scalar base per operand, advanced along K, and a 32-bit byte offset per lane.
    // Row-wise tiles: 8 rows of 8 chunks of 16 bytes, chunk c of row r at position c ^ ((r >> 1) & 7).  K-major B: rows of
    // BN columns, as they lie (swizzled for BN >= 64).  Rows / columns beyond the matrix re-read valid ones (never stored);
    // what lies beyond K comes from a block of zeros, for both operands.
    constexpr int CPR = BN / 8, RPL = 64 / CPR;                 // K-major B: 16-byte pieces per row, rows per load
    auto bswz = [](int r) { return BN == 128 ? 4 * (r & 3) : (BN == 64 ? 4 * ((r >> 1) & 1) : 0); };
    unsigned voff[LPW];
    int kidx[LPW];                                              // first k (within a chunk) that the lane fetches
#pragma unroll
    for (int t = 0; t < LPW; ++t) {
        const int i = (wave + NW * t) % C::LPC;
        const bool isA = (NW * t) % C::LPC < C::LA;             // the same for all wavefronts: LA and LPC are multiples of NW
        const int ii = isA ? i : i - C::LA;
        if (isA || !BKM) {
            const int row = ii * 8 + (lane >> 3), ch = (lane & 7) ^ ((row >> 1) & 7);
            kidx[t] = ch * 8;
            voff[t] = (unsigned)(min(row, (isA ? M - m0 : N - n0) - 1) * (isA ? lda : ldb) * 2 + ch * 16);
        } else {
            const int row = ii * RPL + lane / CPR, col = ((lane % CPR) ^ bswz(row)) * 8;
            kidx[t] = row;
            voff[t] = (unsigned)(row * ldb * 2 + min(col, N - 8 - n0) * 2);
        }
    }
    const char* a_base = reinterpret_cast<const char*>(A + (int64_t)m0 * lda);
    const char* b_base = reinterpret_cast<const char*>(BKM ? B + n0 : B + (int64_t)n0 * ldb);
    const char* zero = reinterpret_cast<const char*>(g_zero_chunk);
    const int nst = (K + 64 * SUB - 1) / (64 * SUB);
    const int nfull = K / (64 * SUB);                           // stages that lie within K
    auto issue = [&](int st, auto full_tag) {
        const unsigned sb = lds0 + ((unsigned)st % NS) * C::STAGE;
#pragma unroll
        for (int t = 0; t < LPW; ++t) {
            const int sub = (NW * t) / C::LPC, k0 = (st * SUB + sub) * 64;
            const bool isA = (NW * t) % C::LPC < C::LA;
            const char* base = isA ? a_base + (int64_t)k0 * 2 : b_base + (BKM ? (int64_t)k0 * ldb * 2 : (int64_t)k0 * 2);
            const unsigned dst = sb + (wave + NW * t) * 1024;
            if (decltype(full_tag)::value) dma16_sbase(base, voff[t], dst);
            else dma16_ptr(k0 + kidx[t] < K ? base + voff[t] : zero, dst);
        }
    };
    auto issue_any = [&](int st) {
        if (st < nfull) issue(st, std::true_type{});
        else if (st < nst) issue(st, std::false_type{});
    };

    // ---- epilogue geometry; its operands do not depend on the products: requested first, landed long before use ----
    constexpr int QPR = BN / 4, ROWS = NW * 64 / QPR, PASS = BM / ROWS;       // threads per row, rows per pass
    const int c4 = tid % QPR, rr = tid / QPR, n = n0 + 4 * c4;
    f32x4_t bv = {0.f, 0.f, 0.f, 0.f}, opnd[PASS];
    if (n < N) {
        if (KIND == EPI_BIAS || KIND == EPI_BIAS_GELU || KIND == EPI_RESIDUAL)
            bv = ld_bf16x4(reinterpret_cast<const bf16*>(epi.bias) + n);
        if (PASS <= 4)
#pragma unroll
            for (int p = 0; p < PASS; ++p) opnd[p] = epi_load4<KIND>(epi, min(m0 + rr + p * ROWS, M - 1), n);
    }
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) issue_any(s);

    // ---- fragments ----
    constexpr int KK = 4 * SUB;                                 // product steps per stage
    unsigned a_off[4], b_off[4], bt_off[TN];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const int koff = ((2 * kk + g) ^ ((fr >> 1) & 7)) << 4;
        a_off[kk] = (wm * TM * 32 + fr) * 128 + koff;
        b_off[kk] = C::A_BYTES + (wn * TN * 32 + fr) * 128 + koff;
    }
    if (BKM) {
        const int jj = lane & 15, q = lane >> 4;
        const int r = (q >> 1) * 8 + (jj >> 2);                 // rows r and r + 4 are swizzled alike
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int c = (wn * TN + j) * 32 + (q & 1) * 16 + 4 * (jj & 3);
            bt_off[j] = C::A_BYTES + r * (BN * 2) + (((c >> 3) ^ bswz(r)) << 4) + (c & 7) * 2;
        }
    }
    struct Frags { bf16x8_t a[KK][TM], b[KK][TN]; };
    auto read = [&](Frags& f, int st) {
        const unsigned char* base = smem + ((unsigned)st % NS) * C::STAGE;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const unsigned char* p = base + (kk >> 2) * C::CHUNK;
#pragma unroll
            for (int i = 0; i < TM; ++i) f.a[kk][i] = *reinterpret_cast<const bf16x8_t*>(p + a_off[kk & 3] + i * 32 * 128);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (BKM) {
                    const unsigned char* q = p + bt_off[j] + (kk & 3) * 16 * (BN * 2);
                    union { struct { s16x4_t lo, hi; } s; bf16x8_t v; } u;
                    u.s.lo = lds_tr16(reinterpret_cast<const uint16_t*>(q));
                    u.s.hi = lds_tr16(reinterpret_cast<const uint16_t*>(q + 4 * (BN * 2)));
                    f.b[kk][j] = u.v;
                } else {
                    f.b[kk][j] = *reinterpret_cast<const bf16x8_t*>(p + b_off[kk & 3] + j * 32 * 128);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    f32x16_t acc[TN][TM];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.f;
    auto products = [&](const Frags& f, int chunks) {           // of the first `chunks` chunks of a stage
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            if (kk % 4 == 0 && kk / 4 >= chunks) break;
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[j][i] = mfma32(f.b[kk][j], f.a[kk][i], acc[j][i]);
        }
    };
    // This wavefront's loads of a stage have landed, with those of the AHEAD stages after it still under way, and its LDS
    // reads have returned; then the same for everybody.
    auto landed = [&](auto ahead_tag) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(decltype(ahead_tag)::value * LPW));
        asm volatile("s_barrier" ::: "memory");
    };
    using Ahead = std::integral_constant<int, NS - 2>;
    // a stage whose refill (of the stage read last, before the barrier) lies within K ...
    auto step = [&](Frags& now, const Frags& before, int st) {
        landed(Ahead{});
        issue(st + NS - 1, std::true_type{});
        if (computes) {
            read(now, st);
            products(before, SUB);
        }
    };
    // ... and one near the end
    const int last_chunks = (K + 63) / 64 - (nst - 1) * SUB;    // of the last stage
    auto end_step = [&](Frags& now, const Frags& before, int st) {
        const int ahead = nst - 1 - st;
        if (ahead >= NS - 2) landed(Ahead{});
        else if (ahead >= (NS - 2) / 2) landed(std::integral_constant<int, (NS - 2) / 2>{});
        else if (ahead >= 1) landed(std::integral_constant<int, 1>{});
        else landed(std::integral_constant<int, 0>{});
        issue_any(st + NS - 1);
        if (computes) {
            read(now, st);
            if (st > 0) products(before, SUB);
        }
    };
    Frags f0, f1;
    end_step(f0, f1, 0);
    int st = 1;
    for (; st + NS < nfull; st += 2) {
        step(f1, f0, st);
        step(f0, f1, st + 1);
    }
    for (; st + 1 < nst; st += 2) {
        end_step(f1, f0, st);
        end_step(f0, f1, st + 1);
    }
    if (st < nst) end_step(f1, f0, st);
    if (computes) {
        if (nst & 1) products(f0, last_chunks);
        else products(f1, last_chunks);
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
                const f32x4_t x = PASS <= 4 ? opnd[p] : epi_load4<KIND>(epi, m, n);
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

template <int TM, int TN, int WM, int WN, int SUB, int NS, int EPI, bool BKM>
static int launch_ring(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K, const Epi& epi) {
    using C = RingCfg<TM, TN, WM, WN, SUB, NS>;
    static LdsLimit lim;
    auto kern = gemm_ring_kernel<TM, TN, WM, WN, SUB, NS, EPI, BKM>;
    if (int rc = lim.ensure(reinterpret_cast<const void*>(kern), C::SHMEM)) return rc;
    const int tiles = ((M + C::BM - 1) / C::BM) * ((N + C::BN - 1) / C::BN);
    hipLaunchKernelGGL(kern, dim3(tiles), dim3(256), C::SHMEM, s, A, lda, B, ldb, M, N, K, epi);
    REV_HIP(hipGetLastError());
    return REV_OK;
}

template <int EPI, bool BKM>
static int dispatch_ring(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K,
                         const Epi& epi, GemmShape shape) {
    switch (shape) {
        case GS_32x32: return launch_ring<1, 1, 1, 1, 2, 4, EPI, BKM>(s, A, lda, B, ldb, M, N, K, epi);     // 64 to 72 KB of LDS:
        case GS_64x64: return launch_ring<1, 1, 2, 2, 1, 4, EPI, BKM>(s, A, lda, B, ldb, M, N, K, epi);     // two workgroups
        case GS_64x128_RING: return launch_ring<1, 2, 2, 2, 1, 3, EPI, BKM>(s, A, lda, B, ldb, M, N, K, epi);   // per CU
        default: set_error("gemm_bf16: no such tile"); return REV_EINVAL;
    }
}

int gemm_bf16_ring(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K,
                   const Epi& epi, bool b_kmajor, GemmShape shape) {
    switch (epi.kind) {
#define CASE(KIND) case KIND: return b_kmajor ? dispatch_ring<KIND, true>(s, A, lda, B, ldb, M, N, K, epi, shape) \
                                              : dispatch_ring<KIND, false>(s, A, lda, B, ldb, M, N, K, epi, shape);
        CASE(EPI_BIAS) CASE(EPI_BIAS_GELU) CASE(EPI_RESIDUAL) CASE(EPI_GELU_BWD) CASE(EPI_PLAIN) CASE(EPI_PLAIN_F32)
        CASE(EPI_BIAS_GELU | EPI_ERF) CASE(EPI_GELU_BWD | EPI_ERF)
#undef CASE
    }
    set_error("gemm_bf16: unknown epilogue");
    return REV_EINVAL;
}

}  // namespace rev
