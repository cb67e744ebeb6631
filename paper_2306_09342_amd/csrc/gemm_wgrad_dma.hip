// Weight gradients: launches of their own, and the one that ends a small block.  The 128x128 tiles of gemm_wgrad_dma.h read their
// fragments by hand (lds_read_tr16_b64(), waited for later), so the assembly of this file is checked for it (asm_check.py).
#include "gemm_ring.h"
#include "gemm_wgrad_dma.h"

namespace rev {

__global__ __launch_bounds__(256) void wgrad_dma_group_kernel(WgradGroup grp, int M, int steps_per_split) {
    if ((int)blockIdx.x >= grp.tile_blocks) wgrad_dma_sums(grp, M, blockIdx.x - grp.tile_blocks);
    else wgrad_small_block(grp, M, steps_per_split, blockIdx.x);
}
// 256x128 tiles, one workgroup of eight wavefronts per CU (the last of them sum columns in chunks of rows)
using WgradMid = RingCfg<2, 2, 4, 2, 1, 3>;
__global__ __launch_bounds__(512) void wgrad_mid_group_kernel(WgradGroup grp, int M, int steps_per_split) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    if ((int)blockIdx.x >= grp.tile_blocks) wgrad_tail_sums<8>(grp.sums, M, blockIdx.x - grp.tile_blocks, reinterpret_cast<float*>(smem));
    else wgrad_ring_block<2, 2, 4, 2, 1, 3>(grp, M, steps_per_split, blockIdx.x);
}

int launch_wgrad_dma_group(hipStream_t s, const WgradGroup& grp, int M, int sps) {
    static LdsLimit lim, lim_mid;
    if (grp.tile == 256) {
        if (int rc = lim_mid.ensure(reinterpret_cast<const void*>(wgrad_mid_group_kernel), WgradMid::SHMEM)) return rc;
        hipLaunchKernelGGL(wgrad_mid_group_kernel, dim3(grp.tile_blocks + grp.sum_blocks), dim3(512), WgradMid::SHMEM, s, grp, M, sps);
    } else {
        if (int rc = lim.ensure(reinterpret_cast<const void*>(wgrad_dma_group_kernel), 2 * WD_STAGE)) return rc;
        hipLaunchKernelGGL(wgrad_dma_group_kernel, dim3(grp.tile_blocks + grp.sum_blocks), dim3(256), 2 * WD_STAGE, s, grp, M, sps);
    }
    REV_HIP(hipGetLastError());
    return REV_OK;
}

// C[M,N] = A[M,K] * B[K,N] in tiles of the ring and, in the workgroups behind them, weight gradients over the same M rows, column sums
// and second stages of sums: everything that a block's backward still has to do with the rows of A, and with partial
// sums that earlier launches left.  For launches that do not fill the chip, and are mostly latency.  One sample of 197 rows, D = 768, with
// the other weight gradients beside the attention backward (attention_dma.hip): 7.1 (input gradient) + 11.0 (weight gradients) + 3.3 us (sums) -> 11.0,
// and 4.0 more for the attention backward; a pass of 12 blocks 1363 -> 1282.
struct WgradBeside { WgradTail t; RedArgs red; int gemm_blocks, n_fast; };
template <int TM, int TN, int WM, int WN, int SUB, int NS>
__global__ __launch_bounds__(256) void gemm_wgrad_kernel(const bf16* __restrict__ A, int64_t lda, const bf16* __restrict__ B, int64_t ldb,
                                                         int N, int K, Epi epi, WgradBeside w) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    int b = blockIdx.x;
    if (b < w.gemm_blocks) {
        int m0, n0;
        ring_tile_at<RingCfg<TM, TN, WM, WN, SUB, NS>>(w.t.M, N, w.n_fast, b, w.gemm_blocks, &m0, &n0);
        gemm_ring_tile<TM, TN, WM, WN, SUB, NS, EPI_PLAIN, false, true>(A, lda, B, ldb, w.t.M, N, K, epi, m0, n0);
    } else if ((b -= w.gemm_blocks) < w.t.grp.tile_blocks) wgrad_small_block(w.t.grp, w.t.M, w.t.steps, b);
    else if ((b -= w.t.grp.tile_blocks) < w.t.grp.sum_blocks) wgrad_dma_sums(w.t.grp, w.t.M, b);
    else reduce_block(w.red, b - w.t.grp.sum_blocks, reinterpret_cast<float4*>(smem));
}

int launch_gemm_wgrad(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K, const Epi& epi,
                      const WgradTail& tail, const RedSeg* segs, int nseg, GemmShape shape) {
    WgradBeside w = {};
    double bytes = 0;
    const int red_blocks = reduce_args(segs, nseg, &w.red, &bytes);
    if (red_blocks < 0) return red_blocks;
    w.t = tail;
    auto go = [&](auto kern, int bm, int bn, int ring_lds, LdsLimit& lim) -> int {
        const int lds = std::max(ring_lds, 2 * WD_STAGE);
        if (int rc = lim.ensure(reinterpret_cast<const void*>(kern), lds)) return rc;
        w.gemm_blocks = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
        w.n_fast = ring_n_fast(M, N, bm, bn);
        hipLaunchKernelGGL(kern, dim3(w.gemm_blocks + tail.grp.tile_blocks + tail.grp.sum_blocks + red_blocks), dim3(256), lds, s, A, lda, B, ldb, N, K, epi, w);
        REV_HIP(hipGetLastError());
        return REV_OK;
    };
    static LdsLimit lim32, lim64;
    if (shape == GS_32x32) return go(gemm_wgrad_kernel<1, 1, 1, 1, 2, 4>, Ring32::BM, Ring32::BN, Ring32::SHMEM, lim32);
    return go(gemm_wgrad_kernel<1, 1, 2, 2, 1, 4>, Ring64::BM, Ring64::BN, Ring64::SHMEM, lim64);
}

}  // namespace rev
