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
// A residual map of the other chain (rev_stack.hip) comes between the input gradient's tiles and the weight gradients; without one
// it has no workgroups.
struct WgradBeside { WgradTail t; RedArgs red; RingPart nn, nt; };
template <typename C>
__global__ __launch_bounds__(256) void gemm_wgrad_kernel(WgradBeside w) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    int b = blockIdx.x;
    if (b < w.nn.blocks) ring_part<C, EPI_PLAIN, true>(w.nn, w.t.M, b);
    else if ((b -= w.nn.blocks) < w.nt.blocks) ring_part<C, EPI_RESIDUAL, false>(w.nt, w.t.M, b);
    else if ((b -= w.nt.blocks) < w.t.grp.tile_blocks) wgrad_small_block(w.t.grp, w.t.M, w.t.steps, b);
    else if ((b -= w.t.grp.tile_blocks) < w.t.grp.sum_blocks) wgrad_dma_sums(w.t.grp, w.t.M, b);
    else reduce_block(w.red, b - w.t.grp.sum_blocks, reinterpret_cast<float4*>(smem));
}

template <typename C>
static int gemm_wgrad(hipStream_t s, const GemmCall<bf16>& nn, int M, const WgradTail& tail, const RedSeg* segs, int nseg, const GemmCall<bf16>* nt) {
    WgradBeside w = {};
    const int red_blocks = reduce_args(segs, nseg, &w.red, nullptr);
    if (red_blocks < 0) return red_blocks;
    w.t = tail;
    w.nn = ring_part_of<C>(nn, M);
    if (nt) w.nt = ring_part_of<C>(*nt, M);
    constexpr int lds = std::max(C::SHMEM, 2 * WD_STAGE);
    static LdsLimit lim;
    if (int rc = lim.ensure(reinterpret_cast<const void*>(gemm_wgrad_kernel<C>), lds)) return rc;
    hipLaunchKernelGGL(gemm_wgrad_kernel<C>, dim3(w.nn.blocks + w.nt.blocks + tail.grp.tile_blocks + tail.grp.sum_blocks + red_blocks), dim3(256), lds, s, w);
    REV_HIP(hipGetLastError());
    return REV_OK;
}
// nt: nullable
int launch_gemm_wgrad(hipStream_t s, const GemmCall<bf16>& nn, int M, const WgradTail& tail, const RedSeg* segs, int nseg, GemmShape shape,
                      const GemmCall<bf16>* nt) {
    return shape == GS_32x32 ? gemm_wgrad<Ring32>(s, nn, M, tail, segs, nseg, nt) : gemm_wgrad<Ring64>(s, nn, M, tail, segs, nseg, nt);
}

}  // namespace rev
