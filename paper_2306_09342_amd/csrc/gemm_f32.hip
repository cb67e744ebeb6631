// float32 GEMMs on the float32 matrix cores (v_mfma_f32_32x32x2_f32: float32 products and sums), three operand forms:
//   gemm_nt_f32            C = A[M,K] * B[N,K]^T      (activation x weight)
//   gemm_nn_f32            C = A[M,K] * B[K,N]        (input gradients, the weight as stored)
//   gemm_wgrad_f32_group   dW[N,K] = G[M,N]^T * A[M,K] (weight gradients, several per launch)
//
// A workgroup owns one output tile of 32x32 or 64x64; its four wavefronts split the contraction: wavefront w takes the
// 32-wide chunks w, w + 4, ... for the whole tile, out of a two-stage ring in LDS that only it uses (direct-to-LDS
// loads, waited for with its own counter), so the main loop has no barrier.  The four partial tiles are added in
// wavefront order through LDS and leave through the fused epilogue.  A chunk costs 1024 matrix-core cycles per 32x32
// and 8 KB (32x32) or 16 KB (64x64, a quarter of the bytes per product) of operands.
//
// An operand whose rows run along the contraction is read 4 floats per lane (lane group g = lane / 32 of product step
// s takes k = 8q + 4g + s); one that is stored contraction-major is read a float per lane from two of its rows, with
// the same assignment of k to steps.
//
// 32x32 tiles unless there are 512 of 64x64: below that the chip is not full and the shorter chain wins.  Both sum the
// same products in the same order.  591 rows, 384 x 1536 (0.7 GFLOP): 8-9 us; 64x64 tiles on the vector units took 150-174.
#include "gemm_epilogue.h"
#include "sums.h"

namespace rev {

template <int KIND>
__device__ __forceinline__ f32x4_t epi_store4_f32(const Epi& e, int m, int n, f32x4_t acc, f32x4_t bv) {
    const int64_t idx = (int64_t)m * e.ldo + n;
    if (KIND == EPI_BIAS || KIND == EPI_BIAS_GELU || KIND == EPI_RESIDUAL) acc += bv;
    if (KIND == EPI_BIAS_GELU) {
        if (e.out != nullptr) *reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(e.out) + idx) = acc;
        f32x4_t a;
#pragma unroll
        for (int k = 0; k < 4; ++k) a[k] = gelu_f(acc[k]);
        *reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(e.out2) + idx) = a;
    } else if (KIND == EPI_RESIDUAL) {
        *reinterpret_cast<f32x4_t*>(e.outf + idx) = *reinterpret_cast<const f32x4_t*>(e.res + idx) + e.sign * acc;
    } else if (KIND == EPI_GELU_BWD) {
        const f32x4_t h = *reinterpret_cast<const f32x4_t*>(reinterpret_cast<const float*>(e.aux) + idx);
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] = acc[k] * gelu_grad_f(h[k]);
        *reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(e.out) + idx) = acc;
    } else if (KIND == EPI_PLAIN_F32) {
        *reinterpret_cast<f32x4_t*>(e.outf + idx) = acc;
    } else {
        *reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(e.out) + idx) = acc;
    }
    return acc;
}

constexpr int F_NW = 4, F_NS = 2, F_KC = 32;           // wavefronts, stages per wavefront, chunk depth
template <int TM, int TN> struct FCfg {
    static constexpr int BM = 32 * TM, BN = 32 * TN;
    static constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
    static constexpr int PITCH = BN + 4;
    static constexpr int RED_BYTES = F_NW * BM * PITCH * 4;
    static constexpr int RING_BYTES = F_NW * F_NS * STAGE;
    static constexpr int SHMEM = RING_BYTES > RED_BYTES ? RING_BYTES : RED_BYTES;
};

// One output tile (m0, n0).  AKM / BKM: the operand is stored contraction-major ([K, ld]).
template <int TM, int TN, int KIND, bool AKM, bool BKM>
__device__ __forceinline__ void gemm_f32_tile(const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb,
                                              int M, int N, int K, const Epi& epi, int m0, int n0) {
    using C = FCfg<TM, TN>;
    constexpr int BM = C::BM, BN = C::BN, LA = BM / 8, LB = BN / 8, LPS = LA + LB;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, fr = lane & 31;
    unsigned char* ring = smem + wave * (F_NS * C::STAGE);
    const unsigned lds0 = (unsigned)(uintptr_t)LDS_PTR(unsigned char, ring);
    const char* zero = reinterpret_cast<const char*>(g_zero_chunk);

    // per-lane source and contraction index (within a chunk) of each wavefront-wide load of 1 KB.  Row-wise operands:
    // 8 rows of 8 chunks, chunk c of row r at position c ^ ((r >> 1) & 7); contraction-major ones: 8 or 4 rows of 32 or 64
    // columns as they lie.  Rows / columns beyond the matrix re-read valid ones (never stored).
    const char* src[LPS];
    int ks[LPS];
    auto setup = [&](int t, const float* X, int64_t ld, int r0, int rows, bool km, int cols_tile, int idx) {
        if (!km) {
            const int row = t * 8 + (lane >> 3), ch = (lane & 7) ^ ((row >> 1) & 7);
            ks[idx] = ch * 4;
            src[idx] = reinterpret_cast<const char*>(X + (int64_t)min(r0 + row, rows - 1) * ld + ch * 4);
        } else {
            const int cpr = cols_tile / 4, row = t * (64 / cpr) + lane / cpr;
            ks[idx] = row;
            src[idx] = reinterpret_cast<const char*>(X + min(r0 + (lane % cpr) * 4, rows - 4));
        }
    };
#pragma unroll
    for (int t = 0; t < LA; ++t) setup(t, A, lda, m0, M, AKM, BM, t);
#pragma unroll
    for (int t = 0; t < LB; ++t) setup(t, B, ldb, n0, N, BKM, BN, LA + t);
    auto issue = [&](int c, int stage) {
        const int k0 = c * F_KC;
        const unsigned sb = lds0 + stage * C::STAGE;
#pragma unroll
        for (int t = 0; t < LPS; ++t) {
            const bool isA = t < LA, km = isA ? AKM : BKM;
            const int k = k0 + ks[t];
            const char* p = km ? src[t] + (int64_t)k * (isA ? lda : ldb) * 4 : src[t] + (int64_t)k0 * 4;
            dma16_ptr(k < K ? p : zero, sb + t * 1024);
        }
    };

    f32x16_t acc[TN][TM];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.f;

    const int nch = (K + F_KC - 1) / F_KC;
    const int mine = wave < nch ? (nch - wave + F_NW - 1) / F_NW : 0;
#pragma unroll
    for (int s = 0; s < F_NS; ++s)
        if (s < mine) issue(wave + s * F_NW, s);
    // fragment of product group q (8 contraction indices, 4 product steps)
    auto frag = [&](const unsigned char* tile, bool km, int cols, int t, int q, float (&f)[4]) {
        if (!km) {
            const f32x4_t v = *reinterpret_cast<const f32x4_t*>(tile + (t * 32 + fr) * 128 + (((2 * q + g) ^ ((fr >> 1) & 7)) << 4));
#pragma unroll
            for (int s = 0; s < 4; ++s) f[s] = v[s];
        } else {
#pragma unroll
            for (int s = 0; s < 4; ++s)
                f[s] = *reinterpret_cast<const float*>(tile + ((8 * q + 4 * g + s) * cols + t * 32 + fr) * 4);
        }
    };
    for (int i = 0; i < mine; ++i) {
        // the stage's loads are older than those of the stage requested after it
        if (i + F_NS <= mine) wait_vm<(F_NS - 1) * LPS>();
        else wait_vm<0>();
        const unsigned char* st = ring + (i % F_NS) * C::STAGE;
#pragma unroll
        for (int q = 0; q < F_KC / 8; ++q) {
            float a[TM][4], b[TN][4];
#pragma unroll
            for (int t = 0; t < TM; ++t) frag(st, AKM, BM, t, q, a[t]);
#pragma unroll
            for (int t = 0; t < TN; ++t) frag(st + C::A_BYTES, BKM, BN, t, q, b[t]);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int t = 0; t < TM; ++t) acc[j][t] = mfma_f32(b[j][s], a[t][s], acc[j][t]);
        }
        wait_lds();                                             // the stage has been read: it may be refilled
        if (i + F_NS < mine) issue(wave + (i + F_NS) * F_NW, i % F_NS);
    }

    // ---- partial tiles to LDS, summed in wavefront order, epilogue ----
    __syncthreads();
    float* red = reinterpret_cast<float*>(smem);
    {
        float* part = red + wave * (BM * C::PITCH);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) {
                    const f32x4_t v = {acc[j][i][4 * vq], acc[j][i][4 * vq + 1], acc[j][i][4 * vq + 2], acc[j][i][4 * vq + 3]};
                    *reinterpret_cast<f32x4_t*>(part + (i * 32 + fr) * C::PITCH + j * 32 + 8 * vq + 4 * g) = v;
                }
    }
    __syncthreads();
    constexpr int QPR = BN / 4, ROWS = F_NW * 64 / QPR, PASS = BM / ROWS;
    const int c4 = tid % QPR, rr = tid / QPR;
    const int n = n0 + 4 * c4;
    f32x4_t csum = {0.f, 0.f, 0.f, 0.f};
    if (n < N) {
        f32x4_t bv = {0.f, 0.f, 0.f, 0.f};
        if (KIND == EPI_BIAS || KIND == EPI_BIAS_GELU || KIND == EPI_RESIDUAL)
            bv = *reinterpret_cast<const f32x4_t*>(reinterpret_cast<const float*>(epi.bias) + n);
#pragma unroll
        for (int p = 0; p < PASS; ++p) {
            const int r = rr + p * ROWS, m = m0 + r;
            if (m < M) {
                f32x4_t v = *reinterpret_cast<const f32x4_t*>(red + r * C::PITCH + 4 * c4);
#pragma unroll
                for (int w = 1; w < F_NW; ++w) v += *reinterpret_cast<const f32x4_t*>(red + (w * BM + r) * C::PITCH + 4 * c4);
                const f32x4_t o = epi_store4_f32<KIND>(epi, m, n, v, bv);
                if (KIND == EPI_GELU_BWD) csum += o;
            }
        }
    }
    if (KIND == EPI_GELU_BWD && epi.colsum != nullptr) {       // one partial row of column sums per m-tile
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

template <int TM, int TN, int KIND, bool BKM>
__global__ __launch_bounds__(F_NW * 64) void gemm_f32_kernel(const float* __restrict__ A, int64_t lda, const float* __restrict__ B,
                                                             int64_t ldb, int M, int N, int K, Epi epi) {
    const int tiles_m = (M + 32 * TM - 1) / (32 * TM);
    const int tile = xcd_remap(blockIdx.x, gridDim.x);         // m fastest: a run of tiles shares a slice of B
    gemm_f32_tile<TM, TN, KIND, false, BKM>(A, lda, B, ldb, M, N, K, epi, (tile % tiles_m) * 32 * TM, (tile / tiles_m) * 32 * TN);
}

// One of the products of a launch that holds several, in 32x32 tiles
struct F32Part { const float *A, *B; int64_t lda, ldb; int N, K, blocks; Epi epi; };
template <int KIND, bool BKM>
__device__ __forceinline__ void f32_part(const F32Part& p, int M, int block) {
    const int tiles_m = (M + 31) / 32, tile = xcd_remap(block, p.blocks);
    gemm_f32_tile<1, 1, KIND, false, BKM>(p.A, p.lda, p.B, p.ldb, M, p.N, p.K, p.epi, (tile % tiles_m) * 32, (tile / tiles_m) * 32);
}
// An input gradient and, behind its tiles, a map of the other chain of a small stack (rev_stack.hip): two products that do not
// depend on each other, neither of which fills the chip.
template <int KIND_NN, int KIND_NT>
__global__ __launch_bounds__(F_NW * 64) void gemm_pair_f32_kernel(F32Part nn, F32Part nt, int M) {
    if ((int)blockIdx.x < nn.blocks) f32_part<KIND_NN, true>(nn, M, blockIdx.x);
    else f32_part<KIND_NT, false>(nt, M, blockIdx.x - nn.blocks);
}

struct WgradF32Problem { const float* G; const float* A; float* out; int64_t ldg, lda; int N, K, tile0; };
struct WgradF32Group { WgradF32Problem p[WGRAD_GROUP_MAX]; int count; };

// The column sums of a cotangent ride in the last workgroups (sum_blocks of them).
struct WgradF32Sums { const float* in; float* out; int64_t ld; int n, blocks; };

template <int TM, int TN>
__device__ __forceinline__ void wgrad_f32_block(const WgradF32Group& grp, int M, int lin) {
    int pi = 0;
#pragma unroll
    for (int k = 1; k < WGRAD_GROUP_MAX; ++k)
        if (k < grp.count && lin >= grp.p[k].tile0) pi = k;
    const WgradF32Problem& q = grp.p[pi];
    const int t = lin - q.tile0, tiles_n = (q.N + 32 * TM - 1) / (32 * TM);
    Epi e = {};
    e.outf = q.out; e.ldo = q.K;
    gemm_f32_tile<TM, TN, EPI_PLAIN_F32, true, true>(q.G, q.ldg, q.A, q.lda, q.N, q.K, M, e, (t % tiles_n) * 32 * TM, (t / tiles_n) * 32 * TN);
}
template <int TM, int TN>
__global__ __launch_bounds__(F_NW * 64) void wgrad_f32_kernel(WgradF32Group grp, int M, WgradF32Sums sums) {
    const int tiles = gridDim.x - sums.blocks;
    if ((int)blockIdx.x >= tiles) {
        extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
        colsum_block<float>(sums.in, sums.ld, M, sums.n, sums.out, blockIdx.x - tiles, reinterpret_cast<float*>(smem));
        return;
    }
    wgrad_f32_block<TM, TN>(grp, M, xcd_remap(blockIdx.x, tiles));
}
// C[M,N] = A[M,K] * B[K,N] and, in the workgroups behind its `gemm_blocks` tiles, weight gradients over the same M rows, the column
// sums and second stages of sums: everything that a block's backward still has to do with the rows of A, and with partial sums
// that earlier launches left.  For blocks whose launches do not fill the chip: each of the four costs 3 to 5 us by itself there,
// whatever it does.  Four blocks of 32 rows, D = 64: 302 -> 264 us; three of 591 rows, D = 384: 503 -> 478.
// A residual map of the other chain comes between the input gradient's tiles and the weight gradients; without one it has no workgroups.
struct WgradF32Beside { WgradF32Group grp; WgradF32Sums sums; RedArgs red; F32Part nn, nt; int tile_blocks, M; };
__global__ __launch_bounds__(F_NW * 64) void gemm_wgrad_f32_kernel(WgradF32Beside w) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    int b = blockIdx.x;
    if (b < w.nn.blocks) {
        f32_part<EPI_PLAIN, true>(w.nn, w.M, b);
    } else if ((b -= w.nn.blocks) < w.nt.blocks) {
        f32_part<EPI_RESIDUAL, false>(w.nt, w.M, b);
    } else if ((b -= w.nt.blocks) < w.tile_blocks) {
        wgrad_f32_block<1, 1>(w.grp, w.M, xcd_remap(b, w.tile_blocks));
    } else if ((b -= w.tile_blocks) < w.sums.blocks) {
        colsum_block<float>(w.sums.in, w.sums.ld, w.M, w.sums.n, w.sums.out, b, reinterpret_cast<float*>(smem));
    } else {
        reduce_block(w.red, b - w.sums.blocks, reinterpret_cast<float4*>(smem));
    }
}

static inline int64_t f32_tiles(int M, int N, int b) { return (int64_t)((M + b - 1) / b) * ((N + b - 1) / b); }
static bool f32_wide(int M, int N) { return f32_tiles(M, N, 64) >= 512; }

int gemm_f32_colsum_strips(int M, int N) { return f32_wide(M, N) ? (M + 63) / 64 : (M + 31) / 32; }

template <int TM, int KIND, bool BKM>
static int launch_f32(hipStream_t s, const float* A, int64_t lda, const float* B, int64_t ldb, int M, int N, int K, const Epi& epi) {
    using C = FCfg<TM, TM>;
    static LdsLimit lim;
    auto kern = gemm_f32_kernel<TM, TM, KIND, BKM>;
    if (int rc = lim.ensure(reinterpret_cast<const void*>(kern), C::SHMEM)) return rc;
    hipLaunchKernelGGL(kern, dim3((unsigned)f32_tiles(M, N, C::BM)), dim3(F_NW * 64), C::SHMEM, s, A, lda, B, ldb, M, N, K, epi);
    REV_HIP(hipGetLastError());
    return REV_OK;
}

static int check_gemm_f32(const float* A, int64_t lda, const float* B, int64_t ldb, int N, int K, const Epi& epi) {
    const uintptr_t ptrs = (uintptr_t)A | (uintptr_t)B | (uintptr_t)epi.out | (uintptr_t)epi.out2 | (uintptr_t)epi.outf |
                           (uintptr_t)epi.bias | (uintptr_t)epi.res | (uintptr_t)epi.aux | (uintptr_t)epi.colsum;
    if (K % 4 || N % 4 || (lda & 3) || (ldb & 3) || epi.ldo % 4 || (ptrs & 15)) {
        set_error("gemm_f32: sizes must be multiples of 4 and every buffer 16-byte aligned");
        return REV_EINVAL;
    }
    return REV_OK;
}

template <bool BKM>
static int gemm_f32(hipStream_t s, const float* A, int64_t lda, const float* B, int64_t ldb, int M, int N, int K, const Epi& epi) {
    if (int rc = check_gemm_f32(A, lda, B, ldb, N, K, epi)) return rc;
    ProfScope ps(K_GEMM_NT, s, 2.0 * M * N * K);
    const bool wide = f32_wide(M, N);
    switch (epi.kind) {
#define CASE(KIND) case KIND: return wide ? launch_f32<2, KIND, BKM>(s, A, lda, B, ldb, M, N, K, epi) \
                                          : launch_f32<1, KIND, BKM>(s, A, lda, B, ldb, M, N, K, epi);
        CASE(EPI_BIAS) CASE(EPI_BIAS_GELU) CASE(EPI_RESIDUAL) CASE(EPI_GELU_BWD) CASE(EPI_PLAIN) CASE(EPI_PLAIN_F32)
#undef CASE
    }
    set_error("gemm_f32: unknown epilogue");
    return REV_EINVAL;
}
int gemm_nt_f32(hipStream_t s, const float* A, int64_t lda, const float* B, int64_t ldb, int M, int N, int K, const Epi& epi) {
    return gemm_f32<false>(s, A, lda, B, ldb, M, N, K, epi);
}
int gemm_nn_f32(hipStream_t s, const float* A, int64_t lda, const float* B, int64_t ldb, int M, int N, int K, const Epi& epi) {
    return gemm_f32<true>(s, A, lda, B, ldb, M, N, K, epi);
}

static F32Part f32_part_of(const GemmCall<float>& c, int M) {
    return {c.A, c.B, c.lda, c.ldb, c.N, c.K, (int)f32_tiles(M, c.N, 32), c.epi};
}
// One launch where both take 32x32 tiles by themselves.
int gemm_pair(hipStream_t s, const GemmCall<float>& nn, const GemmCall<float>& nt, int M) {
    if (f32_wide(M, nn.N) || f32_wide(M, nt.N)) {
        if (int rc = gemm_nn_f32(s, nn.A, nn.lda, nn.B, nn.ldb, M, nn.N, nn.K, nn.epi)) return rc;
        return gemm_nt_f32(s, nt.A, nt.lda, nt.B, nt.ldb, M, nt.N, nt.K, nt.epi);
    }
    if (int rc = check_gemm_f32(nn.A, nn.lda, nn.B, nn.ldb, nn.N, nn.K, nn.epi)) return rc;
    if (int rc = check_gemm_f32(nt.A, nt.lda, nt.B, nt.ldb, nt.N, nt.K, nt.epi)) return rc;
    ProfScope ps(K_GEMM_NT, s, 2.0 * M * ((double)nn.N * nn.K + (double)nt.N * nt.K));
    const F32Part a = f32_part_of(nn, M), b = f32_part_of(nt, M);
    constexpr int lds = FCfg<1, 1>::SHMEM;
    const dim3 grid((unsigned)(a.blocks + b.blocks)), block(F_NW * 64);
#define PAIR(X, Y) if (nn.epi.kind == X && nt.epi.kind == Y) {                                                             \
        static LdsLimit lim;                                                                                               \
        if (int rc = lim.ensure(reinterpret_cast<const void*>(gemm_pair_f32_kernel<X, Y>), lds)) return rc;                \
        hipLaunchKernelGGL((gemm_pair_f32_kernel<X, Y>), grid, block, lds, s, a, b, M);                                    \
        REV_HIP(hipGetLastError());                                                                                        \
        return REV_OK;                                                                                                     \
    }
    PAIR(EPI_GELU_BWD, EPI_BIAS_GELU) PAIR(EPI_PLAIN, EPI_RESIDUAL) PAIR(EPI_PLAIN, EPI_BIAS)
#undef PAIR
    set_error("gemm_pair: no such pair of epilogues");
    return REV_EINVAL;
}

static int wgrad_f32_args(const WgradF32Item* items, int count, int M, WgradF32Group* grp, WgradF32Sums* sums, bool* wide, int* tiles, double* flops) {
    int64_t t64 = 0, t32 = 0;
    grp->count = count;
    for (int k = 0; k < count; ++k) {
        const WgradF32Item& it = items[k];
        if (it.N % 4 || it.K % 4 || (it.ldg & 3) || (it.lda & 3) ||
            (((uintptr_t)it.G | (uintptr_t)it.A | (uintptr_t)it.dW | (uintptr_t)it.colsum) & 15)) {
            set_error("gemm_wgrad_f32: sizes must be multiples of 4 and every buffer 16-byte aligned");
            return REV_EINVAL;
        }
        t64 += f32_tiles(it.N, it.K, 64);
        *flops += 2.0 * M * it.N * it.K;
        if (it.colsum) {
            if (sums->blocks) { set_error("gemm_wgrad_f32: column sums of one cotangent per launch"); return REV_EINVAL; }
            *sums = {it.G, it.colsum, it.ldg, it.N, colsum_blocks(it.N)};
        }
    }
    *wide = t64 >= 512;
    for (int k = 0; k < count; ++k) {
        const WgradF32Item& it = items[k];
        grp->p[k] = {it.G, it.A, it.dW, it.ldg, it.lda, it.N, it.K, (int)t32};
        t32 += f32_tiles(it.N, it.K, *wide ? 64 : 32);
    }
    *tiles = (int)t32;
    return REV_OK;
}

int gemm_wgrad_f32_group(hipStream_t s, const WgradF32Item* items, int count, int M) {
    WgradF32Group grp = {};
    WgradF32Sums sums = {};
    bool wide;
    int tiles;
    double flops = 0;
    if (int rc = wgrad_f32_args(items, count, M, &grp, &sums, &wide, &tiles, &flops)) return rc;
    ProfScope ps(K_GEMM_WGRAD, s, flops);
    static LdsLimit lim1, lim2;
    const dim3 grid((unsigned)(tiles + sums.blocks)), block(F_NW * 64);
    if (wide) {
        if (int rc = lim2.ensure(reinterpret_cast<const void*>(wgrad_f32_kernel<2, 2>), FCfg<2, 2>::SHMEM)) return rc;
        hipLaunchKernelGGL((wgrad_f32_kernel<2, 2>), grid, block, (FCfg<2, 2>::SHMEM), s, grp, M, sums);
    } else {
        if (int rc = lim1.ensure(reinterpret_cast<const void*>(wgrad_f32_kernel<1, 1>), FCfg<1, 1>::SHMEM)) return rc;
        hipLaunchKernelGGL((wgrad_f32_kernel<1, 1>), grid, block, (FCfg<1, 1>::SHMEM), s, grp, M, sums);
    }
    REV_HIP(hipGetLastError());
    return REV_OK;
}

// One launch for all of it as long as 32x32 tiles are what each of the two would take by itself, and the column sums come in one piece.
bool gemm_wgrad_f32_together(int M, int N, const int* wn, const int* wk, int count) {
    int64_t t64 = 0;
    for (int k = 0; k < count; ++k) t64 += f32_tiles(wn[k], wk[k], 64);
    return M <= COLSUM_ROWS && t64 < 512 && !f32_wide(M, N);
}
int gemm_nn_wgrad_f32(hipStream_t s, const GemmCall<float>& nn, int M, const WgradF32Item* items, int count, const RedSeg* segs, int nseg,
                      const GemmCall<float>* beside) {
    if (int rc = check_gemm_f32(nn.A, nn.lda, nn.B, nn.ldb, nn.N, nn.K, nn.epi)) return rc;
    if (beside) {
        if (int rc = check_gemm_f32(beside->A, beside->lda, beside->B, beside->ldb, beside->N, beside->K, beside->epi)) return rc;
        if (f32_wide(M, beside->N)) {                          // a launch of its own
            if (int rc = gemm_nt_f32(s, beside->A, beside->lda, beside->B, beside->ldb, M, beside->N, beside->K, beside->epi)) return rc;
            beside = nullptr;
        }
    }
    WgradF32Beside w = {};
    bool wide;
    double flops = 2.0 * M * nn.N * nn.K;
    if (int rc = wgrad_f32_args(items, count, M, &w.grp, &w.sums, &wide, &w.tile_blocks, &flops)) return rc;
    const int red_blocks = reduce_args(segs, nseg, &w.red, nullptr);
    if (red_blocks < 0) return red_blocks;
    w.M = M;
    w.nn = f32_part_of(nn, M);
    if (beside) {
        w.nt = f32_part_of(*beside, M);
        flops += 2.0 * M * beside->N * beside->K;
    }
    ProfScope ps(K_MIXED, s, flops);
    static LdsLimit lim;
    if (int rc = lim.ensure(reinterpret_cast<const void*>(gemm_wgrad_f32_kernel), FCfg<1, 1>::SHMEM)) return rc;
    hipLaunchKernelGGL(gemm_wgrad_f32_kernel, dim3((unsigned)(w.nn.blocks + w.nt.blocks + w.tile_blocks + w.sums.blocks + red_blocks)),
                       dim3(F_NW * 64), (FCfg<1, 1>::SHMEM), s, w);
    REV_HIP(hipGetLastError());
    return REV_OK;
}

}  // namespace rev
