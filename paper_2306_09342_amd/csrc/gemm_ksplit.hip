// bf16 GEMM for launches too small to fill the chip with whole-K tiles of the pipelined kernel:
//   C[M,N] (+epilogue) = A[M,K] * B[N,K]^T   or, with BKM,   A[M,K] * B[K,N].
//
// A workgroup owns one small output tile (32x32 or 64x64); its wavefronts split the CONTRACTION: wavefront w takes
// the 64-wide chunks w, w + NW, w + 2 NW, ... of K for the whole tile, out of a ring of NS stages in LDS that only it
// uses (direct-to-LDS loads, waited for with its own counter), so the main loop has no barrier.  The NW partial tiles
// are added in wavefront order through LDS and leave through the fused epilogue.
//
// What bounds it: the rate at which a CU can bring operands on chip (about 100 GB/s here), i.e. (BM + BN) * K * 2
// bytes per CU, behind about 2.5 us of launch, first latency and epilogue.  That is why the tile is the smallest one
// whose workgroups still all run at once.  Measured (197 rows, operands from the memory-side cache, us, against 64x128
// tiles over whole K): N = 768, K = 768: 3.4 (9.6); N = 768, K = 3072: 6.5 (27.6); N = 2304, K = 768: 4.6 (9.6);
// N = 3072, K = 768 with 64x64 tiles: 6.7 (12.3).  Eight wavefronts or deeper rings measured the same.
#include "gemm_epilogue.h"

namespace rev {

template <int TM, int TN, int NW, int NS> struct KsCfg {
    static constexpr int BM = 32 * TM, BN = 32 * TN;
    static constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
    static constexpr int PITCH = BN + 4;
    static constexpr int RED_BYTES = NW * BM * PITCH * 4;
    static constexpr int RING_BYTES = NW * NS * STAGE;
    static constexpr int SHMEM = RING_BYTES > RED_BYTES ? RING_BYTES : RED_BYTES;
};

template <int TM, int TN, int NW, int NS, int KIND, bool BKM>
__global__ __launch_bounds__(NW * 64) void gemm_ksplit_kernel(const bf16* __restrict__ A, int64_t lda,
                                                               const bf16* __restrict__ B, int64_t ldb,
                                                               int M, int N, int K, Epi epi) {
    using C = KsCfg<TM, TN, NW, NS>;
    constexpr int BM = C::BM, BN = C::BN;
    constexpr int LA = BM / 8, LB = BN / 8, LPS = LA + LB;      // wavefront-wide loads (1 KB each) per stage
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, fr = lane & 31;
    // m fastest: an XCD's run of tiles then reads each slice of B once and the (small) A from its L2
    const int tiles_m = (M + BM - 1) / BM;
    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    const int n0 = (tile / tiles_m) * BN, m0 = (tile % tiles_m) * BM;

    unsigned char* ring = smem + wave * (NS * C::STAGE);
    const unsigned lds0 = (unsigned)(uintptr_t)LDS_PTR(unsigned char, ring);

    // per-lane source of each load of a stage, advanced by the chunk's k; chunk position c of row r holds the global
    // 16-byte chunk c ^ swz(r)
    const char* src[LPS];
    int kcol[LA];                                               // first k (within a stage) this lane fetches of A
#pragma unroll
    for (int t = 0; t < LA; ++t) {
        const int row = t * 8 + (lane >> 3), ch = (lane & 7) ^ ((row >> 1) & 7);
        kcol[t] = ch * 8;
        src[t] = reinterpret_cast<const char*>(A + (int64_t)min(m0 + row, M - 1) * lda + ch * 8);
    }
    int krow[LB];
#pragma unroll
    for (int t = 0; t < LB; ++t) {
        if (!BKM) {
            const int row = t * 8 + (lane >> 3), ch = (lane & 7) ^ ((row >> 1) & 7);
            krow[t] = ch * 8;
            src[LA + t] = reinterpret_cast<const char*>(B + (int64_t)min(n0 + row, N - 1) * ldb + ch * 8);
        } else {
            // rows of BN columns: 8 (BN = 64) or 16 (BN = 32) rows per load
            constexpr int CPR = BN / 8, RPL = 64 / CPR;
            const int row = t * RPL + lane / CPR;
            const int ch = (lane % CPR) ^ (BN == 64 ? 4 * ((row >> 1) & 1) : 0);
            krow[t] = row;
            src[LA + t] = reinterpret_cast<const char*>(B + min(n0 + ch * 8, N - 8));
        }
    }
    const char* zero = reinterpret_cast<const char*>(g_zero_chunk);
    const int nch = (K + 63) >> 6;
    auto issue = [&](int c, int stage) {
        const int k0 = c * 64;
        const unsigned sb = lds0 + stage * C::STAGE;
#pragma unroll
        for (int t = 0; t < LA; ++t)                            // columns at and beyond K come as zeros
            dma16_ptr(k0 + kcol[t] < K ? src[t] + (int64_t)k0 * 2 : zero, sb + t * 1024);
#pragma unroll
        for (int t = 0; t < LB; ++t) {
            // B beyond K only has to be finite: it meets zeros of A
            const char* p = BKM ? src[LA + t] + (int64_t)min(k0 + krow[t], K - 1) * ldb * 2
                                : (k0 + krow[t] < K ? src[LA + t] + (int64_t)k0 * 2 : zero);
            dma16_ptr(p, sb + C::A_BYTES + t * 1024);
        }
    };

    f32x16_t acc[TN][TM];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.f;

    int mine = 0;                                               // chunks of this wavefront
    if (wave < nch) mine = (nch - wave + NW - 1) / NW;
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (s < mine) issue(wave + s * NW, s);
    int koff[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) koff[kk] = ((2 * kk + g) ^ ((fr >> 1) & 7)) << 4;
    int btoff[TN];
    if (BKM) {
        const int jj = lane & 15, q = lane >> 4;
        const int r = (q >> 1) * 8 + (jj >> 2);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int c = j * 32 + (q & 1) * 16 + 4 * (jj & 3);
            const int sw = BN == 64 ? 4 * ((r >> 1) & 1) : 0;
            btoff[j] = r * (BN * 2) + (((c >> 3) ^ sw) << 4) + (c & 7) * 2;
        }
    }
    int stage = 0;
    for (int i = 0; i < mine; ++i) {
        // the stage's loads are older than those of the up to NS-1 stages requested after it
        if (i + NS <= mine) wait_vm<(NS - 1) * LPS>();
        else wait_vm<0>();
        const unsigned char* st = ring + stage * C::STAGE;
        bf16x8_t a[4][TM], b[4][TN];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
            for (int t = 0; t < TM; ++t)
                a[kk][t] = *reinterpret_cast<const bf16x8_t*>(st + (t * 32 + fr) * 128 + koff[kk]);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (BKM) {
                    const unsigned char* p = st + C::A_BYTES + kk * 16 * (BN * 2) + btoff[j];
                    union { struct { s16x4_t lo, hi; } s; bf16x8_t v; } u;
                    u.s.lo = lds_tr16(reinterpret_cast<const uint16_t*>(p));
                    // rows +4: (r >> 1) & 1 is the same
                    u.s.hi = lds_tr16(reinterpret_cast<const uint16_t*>(p + 4 * (BN * 2)));
                    b[kk][j] = u.v;
                } else {
                    b[kk][j] = *reinterpret_cast<const bf16x8_t*>(st + C::A_BYTES + (j * 32 + fr) * 128 + koff[kk]);
                }
            }
        }
        wait_lds();                                             // the stage is in registers: it may be refilled
        if (i + NS < mine) issue(wave + (i + NS) * NW, stage);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int t = 0; t < TM; ++t) acc[j][t] = mfma32(b[kk][j], a[kk][t], acc[j][t]);
        stage = stage + 1 == NS ? 0 : stage + 1;
    }

    // ---- partial tiles to LDS, summed in wavefront order, epilogue ----
    __syncthreads();
    float* red = reinterpret_cast<float*>(smem);
    {
        float* mine_t = red + wave * (BM * C::PITCH);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) {
                    const f32x4_t v = {acc[j][i][4 * vq], acc[j][i][4 * vq + 1], acc[j][i][4 * vq + 2], acc[j][i][4 * vq + 3]};
                    *reinterpret_cast<f32x4_t*>(mine_t + (i * 32 + fr) * C::PITCH + j * 32 + 8 * vq + 4 * g) = v;
                }
    }
    __syncthreads();
    constexpr int QPR = BN / 4, ROWS = NW * 64 / QPR, PASS = (BM + ROWS - 1) / ROWS;   // ROWS rows per pass
    const int c4 = tid % QPR, rr = tid / QPR;
    const int n = n0 + 4 * c4;
    f32x4_t csum = {0.f, 0.f, 0.f, 0.f};
    if (n < N) {
        f32x4_t bv = {0.f, 0.f, 0.f, 0.f};
        if (KIND == EPI_BIAS || KIND == EPI_BIAS_GELU || KIND == EPI_RESIDUAL)
            bv = ld_bf16x4(reinterpret_cast<const bf16*>(epi.bias) + n);
#pragma unroll
        for (int p = 0; p < PASS; ++p) {
            const int r = rr + p * ROWS, m = m0 + r;
            if (r < BM && m < M) {
                const f32x4_t opnd = epi_load4<KIND>(epi, m, n);
                f32x4_t v = *reinterpret_cast<const f32x4_t*>(red + r * C::PITCH + 4 * c4);
#pragma unroll
                for (int w = 1; w < NW; ++w) v += *reinterpret_cast<const f32x4_t*>(red + (w * BM + r) * C::PITCH + 4 * c4);
                const f32x4_t o = epi_store4<KIND>(epi, m, n, v, bv, opnd);
                if (KIND == EPI_GELU_BWD) csum += o;
            }
        }
    }
    // fused bias gradient: column sums of the tile's rows, one partial row per m-tile
    if (KIND == EPI_GELU_BWD && epi.colsum != nullptr) {
        __syncthreads();
        *reinterpret_cast<f32x4_t*>(red + (rr * QPR + c4) * 4) = csum;
        __syncthreads();
        if (rr == 0 && n < N) {
            f32x4_t s = csum;
            for (int q = 1; q < ROWS; ++q) s += *reinterpret_cast<const f32x4_t*>(red + (q * QPR + c4) * 4);
            *reinterpret_cast<f32x4_t*>(epi.colsum + (int64_t)(m0 / BM) * N + n) = s;
        }
    }
}

template <int TM, int TN, int NW, int NS, int KIND, bool BKM>
static int launch_ks(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K, const Epi& epi) {
    using C = KsCfg<TM, TN, NW, NS>;
    static LdsLimit lim;
    auto kern = gemm_ksplit_kernel<TM, TN, NW, NS, KIND, BKM>;
    if (int rc = lim.ensure(reinterpret_cast<const void*>(kern), C::SHMEM)) return rc;
    const int tiles = ((M + C::BM - 1) / C::BM) * ((N + C::BN - 1) / C::BN);
    hipLaunchKernelGGL(kern, dim3(tiles), dim3(NW * 64), C::SHMEM, s, A, lda, B, ldb, M, N, K, epi);
    REV_HIP(hipGetLastError());
    return REV_OK;
}

template <int KIND, bool BKM>
static int dispatch_ks(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K,
                       const Epi& epi, int tile) {
    if (tile == 32) return launch_ks<1, 1, 4, 2, KIND, BKM>(s, A, lda, B, ldb, M, N, K, epi);     // two workgroups per CU
    return launch_ks<2, 2, 4, 2, KIND, BKM>(s, A, lda, B, ldb, M, N, K, epi);
}

// tile: 32 or 64 (square output tiles)
int gemm_bf16_ksplit(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K,
                     const Epi& epi, bool b_kmajor, int tile) {
    switch (epi.kind) {
#define CASE(KIND) case KIND: return b_kmajor ? dispatch_ks<KIND, true>(s, A, lda, B, ldb, M, N, K, epi, tile) \
                                              : dispatch_ks<KIND, false>(s, A, lda, B, ldb, M, N, K, epi, tile);
        CASE(EPI_BIAS) CASE(EPI_BIAS_GELU) CASE(EPI_RESIDUAL) CASE(EPI_GELU_BWD) CASE(EPI_PLAIN) CASE(EPI_PLAIN_F32)
#undef CASE
    }
    set_error("gemm_bf16: unknown epilogue");
    return REV_EINVAL;
}

}  // namespace rev
