// bf16 matrix-core GEMM entry points.
//
//  gemm_nt_bf16 / gemm_nn_bf16   C = A * B^T  /  C = A * B  with fused epilogue: picks the tile and, for launches that do
//            not fill the chip, the split of the contraction (gemm_nt_dma.hip, gemm_ksplit.hip).
//  gemm_wgrad_bf16               dW[N,K] = G[M,N]^T * A[M,K]: picks the number of token ranges and
//            launches the kernel of gemm_wgrad_dma.hip; the partial tiles of the ranges are summed
//            afterwards in range order, so results do not depend on scheduling.
#include "mfma.h"

namespace rev {

// ----------------------------------------------------------------------------------------
// which kernel and tile a GEMM launch takes
// ----------------------------------------------------------------------------------------
static inline int tiles_of(int M, int N, int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); }

// Cost of a launch in units of "one tile per workgroup slot": the chip holds 512 workgroups of either
// shape (two per CU); a last round that leaves at most one workgroup per CU was measured at about 0.55
// of a full round, any fuller one costs a whole round.
static double rounds_cost(int tiles) {
    const int full = tiles / 512, rem = tiles % 512;
    return full + (rem == 0 ? 0.0 : (rem <= 256 ? 0.55 : 1.0));
}
// 160x128 tiles do 1.25x the work of 128x128 ones at about 0.9 of their rate.  Only launches with more than
// one full round of 128-row tiles are considered: below that the chip is not full and the cost of a
// partly filled round does not follow the model (measured: the tall tile loses there).
static bool tall_tiles_pay(int M, int N) {
    if (tiles_of(M, N, 128, 128) <= 512) return false;
    const double c128 = rounds_cost(tiles_of(M, N, 128, 128)) * 128.0;
    const double c160 = rounds_cost(tiles_of(M, N, 160, 128)) * 160.0 * 1.10;
    return c160 < 0.97 * c128;
}

// A launch that cannot give every CU a workgroup is bound by the serial chain of one tile (K stages) and by the rate at
// which one CU takes in operands; so the smallest tile is taken whose workgroups all run at once (32x32: two per CU,
// the others one), each splitting K among its wavefronts.  Measured at 49 ... 7289 rows, N and K from 384 to 3072: every
// choice is the best of the seven shapes or within 10 % of it.  From more than 256 tiles of 128x128 on, whole-K tiles fill the chip.
// These lines depend on M and N only, never on what else runs: the split of K fixes the order of the sums.  Training
// batches (more than 3072 rows, where splitting would still gain up to 15 % on narrow outputs) always sum K in one
// order, so that a sample's results do not depend on how many others are in its batch.
constexpr int SPLIT_MAX_ROWS = 3072;
static GemmShape split_shape(int M, int N) {
    if (M > SPLIT_MAX_ROWS) return GS_128x128;
    if (tiles_of(M, N, 32, 32) <= 512) return GS_32x32;
    if (tiles_of(M, N, 64, 64) <= 256) return GS_64x64;
    if (tiles_of(M, N, 64, 128) <= 256) return GS_64x128_K3;
    if (tiles_of(M, N, 128, 128) <= 256) return GS_128x128_K2;
    return GS_128x128;
}
// 160-row tiles (two wavefronts of 160x64) when they turn a short ragged second round of 128-row tiles into a single
// round.  Only for launches that have the device to themselves: next to another stream's kernels that round is filled
// anyway and the larger LDS footprint keeps the neighbour out (measured: sequential schedule faster, parallel schedule
// 5 % slower).  Each output element sums the same products in the same order under both tiles, so the choice does
// not change a bit of the result.  Not with fused column sums (their strips are 64 rows) and not with a short last
// stage (the extra address registers would not fit next to 160 accumulators).
static GemmShape pick_gemm_shape(int M, int N, int K, const Epi& epi) {
    const GemmShape sh = split_shape(M, N);
    if (sh == GS_128x128 && epi.solo && epi.colsum == nullptr && K % 64 == 0 && tall_tiles_pay(M, N)) return GS_160x128;
    return sh;
}

int gemm_colsum_strips(int M, int N) {
    switch (split_shape(M, N)) {
        case GS_32x32: return (M + 31) / 32;
        case GS_64x64: return (M + 63) / 64;
        case GS_64x128_K3: return (M + 63) / 64 * 2;      // 32-row strips
        case GS_128x128_K2: return (M + 127) / 128 * 4;
        default: return (M + 127) / 128 * 2;              // 64-row strips
    }
}

int gemm_bf16_dma(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb,
                  int M, int N, int K, const Epi& epi, bool b_kmajor, GemmShape shape);
int gemm_bf16_ksplit(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K,
                     const Epi& epi, bool b_kmajor, int tile);

static int gemm_bf16(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K,
                     const Epi& epi, bool b_kmajor) {
    const uintptr_t ptrs = (uintptr_t)A | (uintptr_t)B | (uintptr_t)epi.out | (uintptr_t)epi.out2 | (uintptr_t)epi.outf |
                           (uintptr_t)epi.bias | (uintptr_t)epi.res | (uintptr_t)epi.aux | (uintptr_t)epi.colsum;
    if (K % 8 || N % 8 || (lda & 7) || (ldb & 7) || epi.ldo % 8 || (ptrs & 15)) {
        set_error("gemm_bf16: sizes must be multiples of 8 and every buffer 16-byte aligned");
        return REV_EINVAL;
    }
    ProfScope ps(K_GEMM_NT, s, 2.0 * M * N * K);
    const GemmShape shape = pick_gemm_shape(M, N, K, epi);
    if (shape == GS_32x32 || shape == GS_64x64)
        return gemm_bf16_ksplit(s, A, lda, B, ldb, M, N, K, epi, b_kmajor, shape == GS_32x32 ? 32 : 64);
    return gemm_bf16_dma(s, A, lda, B, ldb, M, N, K, epi, b_kmajor, shape);
}

// C[M,N] = A[M,K] * B[K,N]   (B row-major [K, ldb]): the input-gradient form, weights as stored
int gemm_nn_bf16(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb,
                 int M, int N, int K, const Epi& epi) {
    return gemm_bf16(s, A, lda, B, ldb, M, N, K, epi, true);
}
int gemm_nt_bf16(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb,
                 int M, int N, int K, const Epi& epi) {
    return gemm_bf16(s, A, lda, B, ldb, M, N, K, epi, false);
}

// ----------------------------------------------------------------------------------------
// weight gradient: dW[N,K] = sum over tokens m of G[m,n] * A[m,k]
// ----------------------------------------------------------------------------------------
constexpr int WG_BP = 128;            // tile rows (n)
constexpr int WG_BQ = 128;            // tile cols (k)
constexpr int WG_BR = 64;             // tokens per step

// The token reduction is cut into S ranges so that tiles * S fills, but does not exceed, the
// workgroup slots of the chip (256 CUs x 2 resident workgroups): one full round, no ragged second one.
// Narrow layers with very many tokens (window-attention stages: a handful of tiles, thousands of
// steps) get up to 128 ranges; the partial sums stay below 64 MB.
static int wgrad_splits(int M, int N, int K) {
    const int tiles = ((N + WG_BP - 1) / WG_BP) * ((K + WG_BQ - 1) / WG_BQ);
    int S = 512 / tiles;
    const int steps = (M + WG_BR - 1) / WG_BR;
    if (S > steps / 4) S = steps / 4;                          // at least 4 steps per range
    const int64_t cap = ((int64_t)64 << 20) / ((int64_t)N * K * 4);   // at most 64 MB of partial sums
    if (S > cap) S = (int)cap;
    if (S > 128) S = 128;
    if (S < 1) S = 1;
    const int sps = (steps + S - 1) / S;
    return (steps + sps - 1) / sps;                            // no empty ranges
}
int64_t wgrad_partial_elems(int M, int N, int K) {
    const int S = wgrad_splits(M, N, K);
    return S > 1 ? (int64_t)S * N * K : 0;
}

int launch_wgrad_dma(hipStream_t s, const bf16* G, int64_t ldg, const bf16* A, int64_t lda, int M, int N, int K,
                     int S, int sps, float* out);
int launch_wgrad_dma_group(hipStream_t s, WgradGroup grp, int M, int S, int sps);

int gemm_wgrad_bf16(hipStream_t s, const bf16* G, int64_t ldg, const bf16* A, int64_t lda,
                    int M, int N, int K, float* dW, float* partial, int64_t partial_elems, RedSeg* defer) {
    if (defer) defer->P = 0;            // P == 0: nothing left to reduce
    if ((ldg & 7) || (lda & 7) || (N & 7) || (K & 7) || ((uintptr_t)G & 15) || ((uintptr_t)A & 15)) {
        set_error("gemm_wgrad_bf16: sizes must be multiples of 8 and every buffer 16-byte aligned");
        return REV_EINVAL;
    }
    const int S = wgrad_splits(M, N, K);
    if (S > 1 && (partial == nullptr || partial_elems < (int64_t)S * N * K)) {
        set_error("gemm_wgrad_bf16: split scratch too small");
        return REV_EWORKSPACE;
    }
    const int steps = (M + WG_BR - 1) / WG_BR;
    const int sps = (steps + S - 1) / S;
    const int tiles = ((N + WG_BP - 1) / WG_BP) * ((K + WG_BQ - 1) / WG_BQ);
    {
        ProfScope ps(K_GEMM_WGRAD, s, 2.0 * M * N * K);
        int rc = launch_wgrad_dma(s, G, ldg, A, lda, M, N, K, S, sps, S > 1 ? partial : dW);
        if (rc) return rc;
    }
    if (S > 1) {
        const RedSeg g = {partial, dW, nullptr, (int64_t)N * K, (int64_t)N * K, (int64_t)N * K, S};
        if (defer) { *defer = g; return REV_OK; }
        return reduce_multi(s, &g, 1);
    }
    return REV_OK;
}

// Token ranges of a group launch: tiles of all items x S fills, but does not exceed, the 512 workgroup slots; at
// least 4 steps per range; at most 64 MB of pieces per item.
int wgrad_group_ranges(int M, const int* N, const int* K, int count) {
    int tiles_total = 0;
    for (int k = 0; k < count; ++k) tiles_total += ((N[k] + WG_BP - 1) / WG_BP) * ((K[k] + WG_BQ - 1) / WG_BQ);
    const int steps = (M + WG_BR - 1) / WG_BR;
    int S = 512 / (tiles_total > 0 ? tiles_total : 1);
    if (S > steps / 4) S = steps / 4;
    if (S > 128) S = 128;
    for (int k = 0; k < count; ++k) {
        const int64_t cap = ((int64_t)64 << 20) / ((int64_t)N[k] * K[k] * 4);
        if (S > cap) S = (int)cap;
    }
    if (S < 1) S = 1;
    const int sps = (steps + S - 1) / S;
    return (steps + sps - 1) / sps;                            // no empty ranges
}

int gemm_wgrad_bf16_group(hipStream_t s, const WgradItem* items, int count, int M, RedSeg* segs, int max_ranges) {
    bool fast = count >= 1 && count <= WGRAD_GROUP_MAX;
    for (int k = 0; k < count && fast; ++k) {
        const WgradItem& it = items[k];
        if ((it.ldg & 7) || (it.lda & 7) || (it.N & 7) || (it.K & 7) || ((uintptr_t)it.G & 15) || ((uintptr_t)it.A & 15))
            fast = false;
    }
    if (!fast) {                          // one at a time (any shape)
        for (int k = 0; k < count; ++k) {
            const WgradItem& it = items[k];
            int rc = gemm_wgrad_bf16(s, it.G, it.ldg, it.A, it.lda, M, it.N, it.K, it.dW, it.partial, it.partial_elems, &segs[k]);
            if (rc) return rc;
        }
        return REV_OK;
    }
    // token ranges: tiles of all items x S fills, but does not exceed, the 512 workgroup slots; at least 4 steps per
    // range; no more ranges than every item's scratch holds
    WgradGroup grp = {};
    grp.count = count;
    int tiles_total = 0;
    double flops = 0;
    for (int k = 0; k < count; ++k) {
        grp.p[k].tile0 = tiles_total;
        tiles_total += ((items[k].N + WG_BP - 1) / WG_BP) * ((items[k].K + WG_BQ - 1) / WG_BQ);
        flops += 2.0 * M * items[k].N * items[k].K;
    }
    grp.tiles_total = tiles_total;
    const int steps = (M + WG_BR - 1) / WG_BR;
    int Ns[WGRAD_GROUP_MAX], Ks[WGRAD_GROUP_MAX];
    for (int k = 0; k < count; ++k) { Ns[k] = items[k].N; Ks[k] = items[k].K; }
    int S = wgrad_group_ranges(M, Ns, Ks, count);
    if (max_ranges > 0 && S > max_ranges) S = max_ranges;
    for (int k = 0; k < count; ++k) {
        const int64_t cap = items[k].partial ? items[k].partial_elems / ((int64_t)items[k].N * items[k].K) : 0;
        if (S > cap) S = (int)cap;
    }
    if (S < 1) S = 1;
    const int sps = (steps + S - 1) / S;
    S = (steps + sps - 1) / sps;                               // no empty ranges
    for (int k = 0; k < count; ++k) {
        const WgradItem& it = items[k];
        const int64_t nk = (int64_t)it.N * it.K;
        grp.p[k].G = it.G; grp.p[k].A = it.A; grp.p[k].ldg = it.ldg; grp.p[k].lda = it.lda;
        grp.p[k].N = it.N; grp.p[k].K = it.K;
        grp.p[k].out = S > 1 ? it.partial : it.dW;
        grp.p[k].split_stride = nk;
        segs[k] = {it.partial, it.dW, nullptr, nk, nk, nk, S > 1 ? S : 0};
    }
    ProfScope ps(K_GEMM_WGRAD, s, flops);
    return launch_wgrad_dma_group(s, grp, M, S, sps);
}

}  // namespace rev
