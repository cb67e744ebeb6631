// bf16 GEMMs in the deep ring (gemm_ring.h): the kernels and their tiles.
#include "gemm_ring.h"

namespace rev {

template <int TM, int TN, int WM, int WN, int SUB, int NS, int EPI, bool BKM>
__global__ __launch_bounds__((RingCfg<TM, TN, WM, WN, SUB, NS>::NW * 64)) void gemm_ring_kernel(
    const bf16* __restrict__ A, int64_t lda, const bf16* __restrict__ B, int64_t ldb, int M, int N, int K, Epi epi, int n_fast) {
    int m0, n0;
    ring_tile_at<RingCfg<TM, TN, WM, WN, SUB, NS>>(M, N, n_fast, blockIdx.x, gridDim.x, &m0, &n0);
    gemm_ring_tile<TM, TN, WM, WN, SUB, NS, EPI, false, BKM>(A, lda, B, ldb, M, N, K, epi, m0, n0);
}

template <int TM, int TN, int WM, int WN, int SUB, int NS, int EPI, bool BKM>
static int launch_ring(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K, const Epi& epi) {
    using C = RingCfg<TM, TN, WM, WN, SUB, NS>;
    static LdsLimit lim;
    auto kern = gemm_ring_kernel<TM, TN, WM, WN, SUB, NS, EPI, BKM>;
    if (int rc = lim.ensure(reinterpret_cast<const void*>(kern), C::SHMEM)) return rc;
    const int tiles = ((M + C::BM - 1) / C::BM) * ((N + C::BN - 1) / C::BN);
    hipLaunchKernelGGL(kern, dim3(tiles), dim3(C::NW * 64), C::SHMEM, s, A, lda, B, ldb, M, N, K, epi, ring_n_fast(M, N, C::BM, C::BN));
    REV_HIP(hipGetLastError());
    return REV_OK;
}

template <int EPI, bool BKM>
static int dispatch_ring(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K,
                         const Epi& epi, GemmShape shape) {
    switch (shape) {
        case GS_32x32: return launch_ring<1, 1, 1, 1, 2, 4, EPI, BKM>(s, A, lda, B, ldb, M, N, K, epi);     // 64 KB of LDS: two
        case GS_64x64: return launch_ring<1, 1, 2, 2, 1, 4, EPI, BKM>(s, A, lda, B, ldb, M, N, K, epi);     // workgroups per CU
        case GS_64x128_RING: return launch_ring<1, 1, 2, 4, 1, 4, EPI, BKM>(s, A, lda, B, ldb, M, N, K, epi);   // 96, 128 and 160 KB: one
        case GS_128x128_RING: return launch_ring<2, 1, 2, 4, 1, 4, EPI, BKM>(s, A, lda, B, ldb, M, N, K, epi);
        case GS_192x128_RING: return launch_ring<3, 1, 2, 4, 1, 4, EPI, BKM>(s, A, lda, B, ldb, M, N, K, epi);
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

// Two products that do not depend on each other, one tile per workgroup: an input gradient, and behind its tiles a map of the other
// chain of a small stack (rev_stack.hip), in tiles of one shape: neither fills the chip, and both are latency for most of their time.
// us in the pass, 197 rows, D = 768, Dm = 3072: GELU' and GELU 7.6 + 8.9 by themselves, 10.2 together.  The gradients of fc1 and the projection
// 14.8 (two launches), fc2 and the projection 16.0, QKV 8.0; in pairs 16.0 (over K = 3072) and 7.2, and the projection beside the weight
// gradients, whose launch takes 11.8 instead of 10.7.
template <typename C, int EPI_NN, int EPI_NT>
__global__ __launch_bounds__((C::NW * 64)) void gemm_pair_kernel(RingPart nn, RingPart nt, int M) {
    if ((int)blockIdx.x < nn.blocks) ring_part<C, EPI_NN, true>(nn, M, blockIdx.x);
    else ring_part<C, EPI_NT, false>(nt, M, blockIdx.x - nn.blocks);
}
template <typename C>
static int dispatch_pair(hipStream_t s, const GemmCall<bf16>& nn, const GemmCall<bf16>& nt, int M) {
    const RingPart a = ring_part_of<C>(nn, M), b = ring_part_of<C>(nt, M);
#define PAIR(X, Y) if (nn.epi.kind == (X) && nt.epi.kind == (Y)) {                                                      \
        static LdsLimit lim;                                                                                            \
        if (int rc = lim.ensure(reinterpret_cast<const void*>(gemm_pair_kernel<C, X, Y>), C::SHMEM)) return rc;         \
        hipLaunchKernelGGL((gemm_pair_kernel<C, X, Y>), dim3(a.blocks + b.blocks), dim3(C::NW * 64), C::SHMEM, s, a, b, M); \
        REV_HIP(hipGetLastError());                                                                                     \
        return REV_OK;                                                                                                  \
    }
    PAIR(EPI_GELU_BWD, EPI_BIAS_GELU) PAIR((EPI_GELU_BWD | EPI_ERF), (EPI_BIAS_GELU | EPI_ERF))
    PAIR(EPI_PLAIN, EPI_RESIDUAL) PAIR(EPI_PLAIN, EPI_BIAS)
#undef PAIR
    set_error("gemm_pair: no such pair of epilogues");
    return REV_EINVAL;
}
int gemm_bf16_ring_pair(hipStream_t s, const GemmCall<bf16>& nn, const GemmCall<bf16>& nt, int M, GemmShape shape) {
    switch (shape) {
        case GS_32x32: return dispatch_pair<Ring32>(s, nn, nt, M);
        case GS_64x64: return dispatch_pair<Ring64>(s, nn, nt, M);
        case GS_64x128_RING: return dispatch_pair<RingCfg<1, 1, 2, 4, 1, 4>>(s, nn, nt, M);
        case GS_128x128_RING: return dispatch_pair<RingCfg<2, 1, 2, 4, 1, 4>>(s, nn, nt, M);
        case GS_192x128_RING: return dispatch_pair<RingCfg<3, 1, 2, 4, 1, 4>>(s, nn, nt, M);
        default: set_error("gemm_bf16: no such tile"); return REV_EINVAL;
    }
}

}  // namespace rev
