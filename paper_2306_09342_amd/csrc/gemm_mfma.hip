// bf16 matrix-core GEMM entry points.
//
//  gemm_nt_bf16 / gemm_nn_bf16   C = A * B^T  /  C = A * B  with fused epilogue: picks the tile (gemm_nt_dma.hip,
//            gemm_ring.hip, gemm_big.hip, gemm_mid.hip).  No choice changes the order of an output's sums.
//  gemm_wgrad_bf16_group         dW[N,K] = G[M,N]^T * A[M,K], up to four in a launch: picks the tile (gemm_wgrad_dma.hip,
//            gemm_wgrad_big.hip) and the number of token ranges; the pieces of the ranges are summed afterwards in
//            range order, so results do not depend on scheduling.
#include "mfma.h"
#include "sums.h"

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
// 160-row tiles (two wavefronts of 160x64) when they turn a short ragged second round of 128-row tiles into a single
// round: they do 1.25x the work of 128x128 ones at about 0.9 of their rate.  Only launches with more than
// one full round of 128-row tiles are considered: below that the chip is not full and the cost of a
// partly filled round does not follow the model (measured: the tall tile loses there).  Only for launches that have the device
// to themselves: next to another stream's kernels that round is filled anyway and the larger LDS footprint keeps the
// neighbour out (measured: sequential schedule faster, parallel schedule 5 % slower).  Not with fused column sums (their
// strips are 64 rows) and not with a short last stage (the extra address registers would not fit next to 160 accumulators):
// pick_gemm_shape.
static bool tall_tiles_pay(int M, int N) {
    if (tiles_of(M, N, 128, 128) <= 512) return false;
    const double c128 = rounds_cost(tiles_of(M, N, 128, 128)) * 128.0;
    const double c160 = rounds_cost(tiles_of(M, N, 160, 128)) * 160.0 * 1.10;
    return c160 < 0.97 * c128;
}

// A launch that cannot give every CU a workgroup is bound by the serial chain of one tile and by the rate at
// which one CU takes in operands; so it takes a tile whose workgroups all run at once, in the deep ring of gemm_ring.hip.  All tiles
// sum the products of an output in the same order, so a sample's results do not depend on how many others are in its batch, and
// the lines below are free to follow the clock.
//
// What a launch in the ring takes, in us: what it spends besides the stages by what the epilogue does, and a stage of 64 of K alone
// and with the chip full of workgroups.  Fitted to 1760 launches of M = 100 ... 16384, D = 128 ... 1280 (the products of a block),
// three times each; met to 6 to 11 %.  The two smallest tiles share a CU, two and two, beyond 256 workgroups.
struct RingCost { GemmShape shape; int bm, bn, least, most; double rest[6], full, stage, stage_full; };
static const RingCost RING[] = {
    //                               bias GELU resid GELU' plain f32   fill   stage
    {GS_32x32, 32, 32, 0, 256,       {4.3, 4.5, 4.0, 4.7, 3.9, 4.0},   0.0, 0.073, 0.025},
    {GS_32x32, 32, 32, 256, 288,     {4.3, 4.5, 4.0, 4.7, 4.0, 4.0},   0.0, 0.071, 0.061},
    {GS_64x64, 64, 64, 0, 256,       {4.2, 4.7, 4.3, 4.9, 3.9, 4.1},   0.0, 0.132, 0.052},
    {GS_64x64, 64, 64, 256, 512,     {4.2, 4.8, 4.8, 5.2, 4.1, 4.4},   0.0, 0.239, 0.076},
    {GS_64x128_RING, 64, 128, 0, 256, {4.1, 4.9, 4.5, 5.4, 3.9, 4.2},  0.5, 0.207, 0.106},
    {GS_128x128_RING, 128, 128, 0, 256, {4.7, 6.3, 5.7, 7.1, 4.4, 5.0}, 1.2, 0.281, 0.223},
    {GS_192x128_RING, 192, 128, 0, 256, {5.1, 7.8, 6.7, 8.7, 4.8, 5.7}, 2.2, 0.389, 0.309}};
// the cheapest of them (tiles of up to 64 rows with small_only), GS_128x128 if none holds the launch
static GemmShape ring_shape(int M, int N, int K, int kind, bool small_only, double* us) {
    GemmShape best = GS_128x128;
    *us = 1e30;
    for (const RingCost& r : RING) {
        const int t = tiles_of(M, N, r.bm, r.bn);
        if (t <= r.least || t > r.most || (small_only && r.bm > 64)) continue;
        const double x = t / 256.0, c = r.rest[kind] + r.full * x + K / 64.0 * (r.stage + r.stage_full * x);
        if (c < *us) { *us = c; best = r.shape; }
    }
    return best;
}
// What a launch takes by itself, in us, by tile: a stage of 64 of K, and what a round spends besides (first loads, epilogue) by
// what the epilogue does.  Fitted to 3235 launches of M = 400 ... 59100, D = 128 ... 2048 (the products of a block and of a
// transition), weighted to tell the tiles apart where they are close; the times themselves are met to 6 to 9 %.  A round is 512
// workgroups, two per CU, of 128x128 or 160x128 tiles, 256 of 256x256 ones.  The workgroups of a launch that does not fill one
// round run faster, for they share less (two to a CU on some of them; the power limit), and so do those of a last, partly
// filled round.
//                                bias  GELU  residual  GELU'  plain  float32
static const double REST_128[] = {4.1,  8.0,  10.0,     9.0,   4.7,   7.1};
static const double REST_160[] = {7.6,  12.8, 15.3,     12.8,  8.4,   9.4};
static const double REST_256[] = {10.5, 18.0, 22.0,     21.0,  10.4,  13.5};
static double cost_128(int tiles, double st, int kind) {
    const int full = tiles / 512;
    const double x = tiles % 512 / 512.0;
    const double last = x == 0 ? 0.0 : full ? 0.40 + 0.70 * x : x <= 0.5 ? 0.54 + 0.36 * x : 0.62 + 0.36 * x;
    return (full + last) * (st * 1.03 + REST_128[kind]);
}
static double cost_160(int tiles, double st, int kind) {
    const int full = tiles / 512;
    const double x = tiles % 512 / 512.0;
    const double last = x == 0 ? 0.0 : full ? 0.66 + 0.49 * x : x <= 0.5 ? 0.65 + 0.30 * x : 0.69 + 0.33 * x;
    return (full + last) * (st * 1.04 + REST_160[kind]);
}
static double cost_256(int tiles, double st, int kind) {
    const int full = tiles / 256;
    const double x = tiles % 256 / 256.0, rest = REST_256[kind];
    return full * (st * 1.25 + rest) + (x == 0 ? 0.0 : st * (0.96 + 0.29 * x) + rest * (0.50 + 0.50 * x));
}
// 256x256 tiles (gemm_big.hip) for a launch by itself, where they save more than the costs above are off by.  Measured,
// 128x128 or 160x128 / 256x256, us: M = 16384, N = 768, K = 3072: 92 / 64 (input gradient), 103 / 78 (residual); M = 8224, N = 1280, K =
// 5120: 125 / 90, 156 / 104; M = 12608, N = K = 1024 (200 tiles), residual: 51 / 44.  Where they leave half of a round empty:
// M = 1568, N = 2560, K = 1280 (70 tiles; 260 of 128x128): 17.8 / 25.0; M = 8192, N = 1024, K = 4096 (128; 512): 66 / 72; or take a
// short second one: M = 4100, N = 4096, K = 1024 (272; 1056), GELU: 53 / 59.  Of the 3235 launches they take 1587, 17 % faster in
// the mean; 45 of these are 3 to 14 % slower, most of them residuals over short contractions from operands that had left the
// caches, where a pass finds them there: D = 256, M = 50176, K = 256 32 / 35 by itself (59100: 34 / 43), but a forward block of it
// 234 / 227 us.
// Next to another stream's kernels a partly filled round costs only the CUs it takes, so there the work per CU decides (a tile's
// time with the chip full of them), unless the launch by itself would take much longer.  Four blocks on two streams, 128x128 /
// 256x256 tiles, us: D = 1024, M = 5122: 2349 / 2232; D = 1536, M = 4096: 3471 / 3178.
// A launch with column sums decides by the work per CU under both schedules, and must not take much longer by itself: their strips
// depend on the tile, so that both add the same ones.  (Rev-ViT-B, two streams, in 128x128 tiles instead: 9.14 ms -> 9.37.)
enum BigRule { BIG_ALONE, BIG_BESIDE, BIG_SUMS };
static bool big_tiles_pay(int M, int N, int K, int kind, BigRule rule, bool tall) {
    if (M < 256 || N < 256 || K % 128 != 0) return false;
    const double st = K / 64;
    const int t128 = tiles_of(M, N, 128, 128), t256 = tiles_of(M, N, 256, 256);
    const double small = cost_128(t128, st, kind), big = cost_256(t256, st, kind);
    if (rule == BIG_ALONE) return big < 0.98 * (tall ? std::fmin(small, cost_160(tiles_of(M, N, 160, 128), st, kind)) : small);
    // the constants of the two rules below are those that were fitted next to another stream's kernels
    static const double small_rest[] = {3.0, 7.0, 8.0, 7.0, 4.4, 8.0}, big_rest[] = {8.0, 15.0, 17.0, 18.0, 8.0, 17.0};
    const int rounds = (t256 + 255) / 256;
    const bool work = t256 * (st * 1.28 + big_rest[kind]) < 0.425 * t128 * (st * 1.12 + small_rest[kind]);
    if (rule == BIG_SUMS) return work && big < 1.05 * small;
    return work && rounds * (st * (0.78 + 0.5 * t256 / (256.0 * rounds)) + big_rest[kind]) < 1.1 * rounds_cost(t128) * (st * 1.12 + small_rest[kind]);
}
// 256x128 tiles (gemm_mid.hip), two workgroups per CU, whose epilogues run beside the other's products.  256x256, 160x128 or
// 128x128 / 256x128, us:
// The GELU epilogues over short contractions, from more than two rounds of 512 on.  GELU' M = 25216, N = 1536, K = 384
// (1188 tiles): 72 / 63; N = 2048, K = 512: 110 / 94; M = 7289, N = 1536, K = 384 (348): 24.7 / 25.0; at K = 768 next to the other
// stream's kernels a pass of Rev-ViT-B (M = 12608) takes 9.16 ms with them and 9.00 without.  GELU
// M = 50000, N = 1024, K = 256: 82 / 71; M = 25216, N = 1536, K = 384: 69 / 67; N = 2048, K = 512: 98 / 99; M = 30000: 106 / 116.
// The QKV maps of the same widths, from one and a half rounds on: K = 384, M = 25216 (891 tiles) 37.9 / 34.1, M = 12608 (450) 19.2 /
// 19.9; K = 512, M = 25216 59.6 / 51.4; K = 192, M = 50176 30.0 / 24.4; K = 128, M = 96000 27.6 / 30.8; K = 768, M = 12608 53.7 / 58.1.
// Below K = 384 only without another stream's kernels: D = 256, M = 50000, three blocks: one stream 2131 / 2118, two 1916 / 1937.
static bool mid_tiles_pay(int M, int N, int K, int kind, bool solo) {
    if (M < 256 || N < 128 || K % 64 != 0) return false;
    const int t = tiles_of(M, N, 256, 128);
    if (kind == EPI_BIAS) return K >= (solo ? 192 : 384) && K <= 512 && t > 768;
    return t > 1024 && ((kind == EPI_GELU_BWD && K <= 512) || (kind == EPI_BIAS_GELU && K <= 384));
}
// The GELU epilogues of somewhat longer contractions, where 256x256 tiles would leave the last round partly empty and no other
// stream's kernel takes those CUs.  256x256 / 256x128, us, three sets of buffers in turn, GELU and GELU' with column sums: M = 12608, N
// = 3072, K = 768 (600 tiles of 256x256) 88 / 82 and 98 / 89; M = 16384 (768, three whole rounds) 95 / 104 and 110 / 112; N = 2560, K =
// 640 (640) 82 / 89 and 95 / 86, together 177 / 175; K = 1280, M = 8224, N = 5120 (660) GELU' 135 / 139.  The column sums of both tiles have the same
// bits, so that both schedules still add the same ones.
static bool mid_fills_better(int M, int N, int K, const Epi& epi) {
    const int t256 = tiles_of(M, N, 256, 256);
    return epi.solo && (epi.kind == EPI_BIAS_GELU || epi.kind == EPI_GELU_BWD) && K <= 768 && t256 > 512 && t256 < 0.85 * 256 * ((t256 + 255) / 256);
}
// The narrow outputs of such models beside another stream's kernels, which take the CUs that a partly filled round leaves: fewer
// operand bytes per product than in 128x128 tiles.  Two-stream backward of six blocks, 128x128 / 256x128, us: D = 384, M = 32000
// 4423 / 4298, M = 25216 3516 / 3485; D = 192, M = 50176 3051 / 2985; D = 256, M = 50000 4270 / 4247; D = 512, M = 25216 4840 / 4845.
static bool mid_shares_better(int M, int N, int K, const Epi& epi) {
    return !epi.solo && (epi.kind == EPI_RESIDUAL || epi.kind == EPI_PLAIN) && M >= 256 && N >= 128 && N <= 384 && K >= 192 && K % 64 == 0 &&
           tiles_of(M, N, 256, 128) > 256;
}
// The tiles of launches that fill the chip, two workgroups per CU or 256x256, and what one takes by itself.
static GemmShape wide_shape(int M, int N, int K, const Epi& epi, double* us) {
    *us = 0.0;                                                // (256x128 tiles: only where nothing else comes near)
    if (mid_tiles_pay(M, N, K, epi.kind, epi.solo)) return GS_256x128;
    const double st = K / 64.0;
    const bool tall = epi.solo && epi.colsum == nullptr && K % 64 == 0 && tall_tiles_pay(M, N);
    if (big_tiles_pay(M, N, K, epi.kind, epi.colsum ? BIG_SUMS : epi.solo ? BIG_ALONE : BIG_BESIDE, tall)) {
        if (mid_fills_better(M, N, K, epi)) return GS_256x128;
        *us = cost_256(tiles_of(M, N, 256, 256), st, epi.kind);
        return GS_256x256;
    }
    if (mid_shares_better(M, N, K, epi)) return GS_256x128;
    *us = tall ? cost_160(tiles_of(M, N, 160, 128), st, epi.kind) : cost_128(tiles_of(M, N, 128, 128), st, epi.kind);
    return tall ? GS_160x128 : GS_128x128;
}
// Short contractions (K < 640), where a launch is mostly first loads and epilogue: tiles of up to 64 rows while 64x64 ones would all
// run at once, 64x128 up to one per CU, and two workgroups per CU from there on.  Longer ones: the cheapest tile of the ring where 64x64 tiles would
// all run at once; beyond, if it undercuts the wide tiles by 3 %, for the fits are off by more than they differ below that.  us, the
// tiles before (64x64 or 64x128 in the ring, 64x128 or 128x128 in two stages, 256x256) and the ring's: 1576 rows, N = 768, K = 3072, input
// gradient: 23.2 / 16.6; 3152: 33.3 / 21.8; 7289: 42.8 / 35.1; 7289, N = 384, K = 1536: 19.6 / 13.7, residual 20.7 / 16.7; 3152, N = 384:
// 15.7 / 11.1.  Of the 1760 launches 427 change tile, to 0.875 of the time in the mean; 11 are 4 to 9 % slower (M = 16384, N = 256, K
// = 768, input gradient, 12.9 -> 14.0).
// Beside another stream's kernels the eight-wavefront tiles of the ring, one per CU on most of them, keep those out for a short
// contraction (and so do launches with column sums, whose tile is the same under both schedules): up to 2048 rows from 161 of them on, where it is
// the wide products (QKV, fc1 and its transpose) that take them.  Two-stream passes of four blocks, these / two-stage tiles, us: D = 1024, 800 rows
// 775 / 758, 1000 rows 870 / 844, 1024 rows 886 / 862; D = 896, 1100 rows 832 / 799; D = 768, 1150 rows 736 / 710; D = 640, 1200 rows 670 /
// 634; one stream, by the launch with column sums alone: D = 1024, 800 rows 903 / 913, 1000 rows 1020 / 1021, D = 768, 1100 rows 626 / 634.  With
// more rows so many tiles are products of D x D, which gain: two streams, D = 768, 4000 rows 1245 / 1269, D = 1024, 2600 rows 1560 / 1597; from 225
// tiles of 128x128 on they do not.  Longer contractions gain all the same: D = 1280, 3152 rows (250, K = 5120) 2196 / 2361.
// So do 64x128 tiles where 64x64 ones would all run at once, two per CU, and the rows are few: passes of two streams, those / 64x64 tiles, us:
// four blocks, D = 1280, 200 rows 588 / 574, D = 1536, 200 rows 751 / 715; 32 blocks, D = 1280, 197 rows 4299 / 4144, and one stream, side by side,
// 3959 / 3854.  More rows gain from them all the same: four blocks, D = 1280, 400 rows 693 / 707, 500 728 / 757; D = 1536, 1000 rows 1322 / 1347.
static GemmShape pick_gemm_shape(int M, int N, int K, const Epi& epi) {
    double ring_us, us;
    const bool brief = K < 640;
    const bool few = tiles_of(M, N, 32, 32) <= 288 || tiles_of(M, N, 64, 64) <= (K < 1536 ? 512 : 384);
    const GemmShape ring = ring_shape(M, N, K, epi.kind, brief, &ring_us);
    if (few && ring == GS_64x128_RING && M <= 320 && (!epi.solo || epi.colsum)) return GS_64x64;
    if (few) return ring;
    if (brief && tiles_of(M, N, 64, 128) <= 256) return GS_64x128_RING;
    const GemmShape wide = wide_shape(M, N, K, epi, &us);
    if (!brief && K <= 1024 && (!epi.solo || epi.colsum)) {
        const int tiles = ring == GS_192x128_RING ? tiles_of(M, N, 192, 128) : tiles_of(M, N, 128, 128);
        if (M <= 2048 ? tiles > 160 : ring == GS_128x128_RING && tiles > 224) return wide;
    }
    return !brief && ring_us < 0.97 * us ? ring : wide;
}

int gemm_colsum_strips(int M, int N, int K) {
    Epi e = {};
    e.kind = EPI_GELU_BWD;
    float sums;
    e.colsum = &sums;                                         // a launch with column sums
    switch (pick_gemm_shape(M, N, K, e)) {
        case GS_256x256: case GS_256x128: return (M + 255) / 256 * 4;
        case GS_32x32: return (M + 31) / 32;
        case GS_64x64: case GS_64x128_RING: return (M + 63) / 64;
        case GS_128x128_RING: return (M + 127) / 128;
        case GS_192x128_RING: return (M + 191) / 192;
        default: return (M + 127) / 128 * 2;              // 64-row strips
    }
}

int gemm_bf16_dma(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb,
                  int M, int N, int K, const Epi& epi, bool b_kmajor, GemmShape shape);
int gemm_bf16_big(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K, const Epi& epi, bool b_kmajor);
int gemm_bf16_mid(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K, const Epi& epi);
int gemm_bf16_ring(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K,
                   const Epi& epi, bool b_kmajor, GemmShape shape);

int gemm_bf16_ring_pair(hipStream_t s, const GemmCall<bf16>& nn, const GemmCall<bf16>& nt, int M, GemmShape shape);

static int check_gemm(const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int N, int K, const Epi& epi) {
    const uintptr_t ptrs = (uintptr_t)A | (uintptr_t)B | (uintptr_t)epi.out | (uintptr_t)epi.out2 | (uintptr_t)epi.outf |
                           (uintptr_t)epi.bias | (uintptr_t)epi.res | (uintptr_t)epi.aux | (uintptr_t)epi.colsum;
    if (K % 8 || N % 8 || (lda & 7) || (ldb & 7) || epi.ldo % 8 || (ptrs & 15)) {
        set_error("gemm_bf16: sizes must be multiples of 8 and every buffer 16-byte aligned");
        return REV_EINVAL;
    }
    return REV_OK;
}
// Widths that are no multiple of 32 take GELU in its erf form.  The polynomial is off by up to 1.3e-4 in the value, more
// than half a bf16 step below -2.1 (six of them at -3), and pays only where the epilogue is a large share of the launch.
static bool takes_erf(int K, int kind) { return K % 32 && (kind == EPI_BIAS_GELU || kind == EPI_GELU_BWD); }

static int gemm_bf16(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K,
                     Epi epi, bool b_kmajor) {
    if (int rc = check_gemm(A, lda, B, ldb, N, K, epi)) return rc;
    ProfScope ps(K_GEMM_NT, s, 2.0 * M * N * K);
    const GemmShape shape = pick_gemm_shape(M, N, K, epi);
    if (takes_erf(K, epi.kind)) epi.kind |= EPI_ERF;
    if (shape <= GS_192x128_RING) return gemm_bf16_ring(s, A, lda, B, ldb, M, N, K, epi, b_kmajor, shape);
    if (shape == GS_256x128 && b_kmajor == (epi.kind == EPI_GELU_BWD || epi.kind == EPI_PLAIN)) return gemm_bf16_mid(s, A, lda, B, ldb, M, N, K, epi);
    if (shape == GS_256x256) return gemm_bf16_big(s, A, lda, B, ldb, M, N, K, epi, b_kmajor);
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
// The tile of two products in one launch: the cheapest of the ring for the workgroups of both together (up to 64 rows with
// small_only), GS_128x128 if none holds them.
static GemmShape pair_shape(const GemmCall<bf16>& nn, const GemmCall<bf16>& nt, int M, bool small_only) {
    GemmShape best = GS_128x128;
    double us = 1e30;
    for (const RingCost& r : RING) {
        const int t = tiles_of(M, nn.N, r.bm, r.bn) + tiles_of(M, nt.N, r.bm, r.bn);
        if (t <= r.least || t > r.most || (small_only && r.bm > 64)) continue;
        const double x = t / 256.0, step = r.stage + r.stage_full * x;
        const double c = r.full * x + std::fmax(r.rest[nn.epi.kind] + nn.K / 64.0 * step, r.rest[nt.epi.kind] + nt.K / 64.0 * step);
        if (c < us) { us = c; best = r.shape; }
    }
    return best;
}
// One launch where a tile of the ring holds both.  An input gradient with column sums keeps the tile that it has by itself, which
// their strips depend on, and takes as many rounds of it as it needs.
int gemm_pair(hipStream_t s, const GemmCall<bf16>& nn, const GemmCall<bf16>& nt, int M) {
    const GemmShape shape = nn.epi.colsum ? pick_gemm_shape(M, nn.N, nn.K, nn.epi) : pair_shape(nn, nt, M, false);
    if (shape > GS_192x128_RING) {
        if (int rc = gemm_nn_bf16(s, nn.A, nn.lda, nn.B, nn.ldb, M, nn.N, nn.K, nn.epi)) return rc;
        return gemm_nt_bf16(s, nt.A, nt.lda, nt.B, nt.ldb, M, nt.N, nt.K, nt.epi);
    }
    if (int rc = check_gemm(nn.A, nn.lda, nn.B, nn.ldb, nn.N, nn.K, nn.epi)) return rc;
    if (int rc = check_gemm(nt.A, nt.lda, nt.B, nt.ldb, nt.N, nt.K, nt.epi)) return rc;
    ProfScope ps(K_GEMM_NT, s, 2.0 * M * ((double)nn.N * nn.K + (double)nt.N * nt.K));
    GemmCall<bf16> p = nn, q = nt;
    if (takes_erf(p.K, p.epi.kind)) p.epi.kind |= EPI_ERF;
    if (takes_erf(q.K, q.epi.kind)) q.epi.kind |= EPI_ERF;
    return gemm_bf16_ring_pair(s, p, q, M, shape);
}

// ----------------------------------------------------------------------------------------
// weight gradient: dW[N,K] = sum over tokens m of G[m,n] * A[m,k]
// ----------------------------------------------------------------------------------------
constexpr int WG_BP = 128;            // tile rows (n)
constexpr int WG_BQ = 128;            // tile cols (k)
constexpr int WG_BR = 64;             // tokens per step

// How a group of weight gradients over the same M tokens is cut.
//
// 128x128 tiles (gemm_wgrad_dma.hip): the token reduction of all of them is cut into S ranges so that tiles * S fills, but
// does not exceed, the 512 workgroup slots of the chip (two per CU); at least 4 steps per range, at most 64 MB of pieces per
// weight.  Narrow layers with very many tokens (window-attention stages: a handful of tiles, thousands of steps) get up to
// 128 ranges.
//
// 64x64 tiles in the ring where they all run at once and the tokens are few (COLSUM_ROWS): over all tokens, so that no second
// stage is left.  us, the 128x128 tiles' ranges / these, the launch that adds the pieces not counted: 197 tokens, D = 128: 7.0 / 4.8; 591,
// 384: 9.6 / 8.6; 1024, 256: 8.7 / 7.1; 1024, 384: 10.6 / 10.6.
//
// 256x128 tiles in the ring in the place of 128x128 ones where they run at once, one per CU, on most of the CUs, with at most a fifth
// more of padding, over ranges of at least 40 steps: 6304 tokens, D = 512: 65 / 53; 768: 115 / 103; 25216, 384: 126 / 123 (of which the
// column sums, which find no idle CU, take 12); below 40 steps the deeper fill costs what the operands save:
// 6304, 384 (25 steps): 32.9 / 33.3;
// 1576, 768 (25): 29.6 / 32.4; and so do CUs that stay idle: 3152, 640 (165 tiles): 44.7 / 46.3.
//
// 256x256 tiles (gemm_wgrad_big.hip): whole rounds of 256 tiles run over all tokens; what is left over (or a group with
// fewer than 256 tiles) is cut into the number of ranges that keeps the CUs busiest, its pieces counted at the time of
// writing and reading them.
//
// The cheaper of the two by measured times (us): a step of 64 tokens takes a round of 512 small tiles 1.0 and a round of 256
// large ones 1.3, a piece costs 0.015 / 0.1 to write and read, a round's fill and last stores 4 / 7, a launch for the
// pieces 4 / 5.  Measured, small and large, whole (the QKV column sums and the launch that adds the pieces included): 12608
// tokens, D = 768: 220 and 174; 8224, 1280: 408 and 273; 16384, 768: 284 and 209; 8192, 1024: 264 and 182.  6000, 512 (57),
// 25216, 384 (134) and 1500, 1280 (84) take small tiles, where the two were within 7 % of each other.
struct WgradPlan {
    bool big;
    int tile, S, sps;                 // 64x64, 128x128, 256x128: token ranges and steps per range
    int tiles, full, splits, stages, stages_per_split;   // 256x256
    int tile_blocks, blocks128;       // workgroups, and those that 128x128 tiles would have over the same ranges
    int64_t piece_elems, elems;       // floats of scratch: the pieces, and with the column sums' chunks
};
// Column sums of n columns behind `blocks` tile workgroups of `steps` stages each: as many workgroups as the last round of
// tiles leaves slots idle, but no more rows for one than it reads (at about 20 GB/s, 40 with 8 wavefronts) in the time of
// a tile; in one chunk where that is short anyway.
static WgradSums sums_plan(int M, int n, int blocks, int steps, bool big, bool one_per_cu) {
    WgradSums p = {};
    if (!one_per_cu && M <= COLSUM_ROWS) {                            // 64 columns a workgroup, no second stage
        p.n = n; p.chunks = 1; p.rows = M;
        return p;
    }
    const int slots = one_per_cu ? 256 : 512, idle = (slots - blocks % slots) % slots, groups = (n + 511) / 512;
    p.n = n;
    const int most_rows = steps * (one_per_cu ? 36 : 13), least = (M + most_rows - 1) / most_rows;
    p.chunks = M <= 256 ? 1 : (idle / groups > least ? idle / groups : least);
    // sums that the idle slots do not hold run after the tiles, with the chip to themselves: then in chunks that fill it (MLP
    // transition, 62720 rows, C = 576: 1672 -> 1629 us; two launches of their own: 1638)
    if (M > 256 && !big && least * groups > idle && p.chunks < slots / (2 * groups)) p.chunks = slots / (2 * groups);
    if (p.chunks > (M + 63) / 64) p.chunks = (M + 63) / 64;
    if (p.chunks < 1) p.chunks = 1;
    p.rows = (M + p.chunks - 1) / p.chunks;
    p.chunks = (M + p.rows - 1) / p.rows;
    return p;
}
// Column sums of n columns under a plan.  Those behind 256x128 tiles take no more chunks than behind 128x128 ones, so that the choice
// between the two never asks for more scratch; that is still enough chunks to end with the tiles, for it is at least the 128x128
// tiles' `least`, which is larger.
static WgradSums sums_of(const WgradPlan& p, int M, int n) {
    if (p.big) return sums_plan(M, n, p.tile_blocks, p.stages_per_split, true, true);
    const WgradSums q = sums_plan(M, n, p.tile_blocks, p.sps, false, p.tile == 256);
    if (p.tile != 256) return q;
    const WgradSums cap = sums_plan(M, n, p.blocks128, p.sps, false, false);
    return q.chunks > cap.chunks ? cap : q;
}
static WgradPlan wgrad_plan(int M, const int* N, const int* K, int count) {
    WgradPlan p = {};
    const int steps = (M + WG_BR - 1) / WG_BR;
    int t128 = 0, t64 = 0, t256x128 = 0;
    int64_t nk = 0;
    for (int k = 0; k < count; ++k) {
        t64 += tiles_of(N[k], K[k], 64, 64);
        t256x128 += tiles_of(N[k], K[k], 256, 128);
        t128 += tiles_of(N[k], K[k], WG_BP, WG_BQ);
        p.tiles += tiles_of(N[k], K[k], 256, 256);
        nk += (int64_t)N[k] * K[k];
    }
    int S = 512 / (t128 > 0 ? t128 : 1);
    if (S > steps / 4) S = steps / 4;
    if (S > 128) S = 128;
    for (int k = 0; k < count; ++k) {
        const int64_t cap = ((int64_t)64 << 20) / ((int64_t)N[k] * K[k] * 4);
        if (S > cap) S = (int)cap;
    }
    const bool few = M <= COLSUM_ROWS && t64 <= 512;
    if (S < 1 || few) S = 1;
    p.sps = (steps + S - 1) / S;
    p.S = (steps + p.sps - 1) / p.sps;                         // no empty ranges
    const double small = 4.0 + (double)((t128 * p.S + 511) / 512) * p.sps + (p.S > 1 ? 4.0 + (double)p.S * nk / 16384 * 0.015 : 0.0);

    p.stages = (M + 127) / 128 * 2;                            // an even number; tokens beyond M count as zeros
    p.full = p.tiles / 256 * 256;
    const int rem = p.tiles - p.full;
    double best = rem > 0 ? 1e30 : 0.0;
    p.splits = 1;
    p.stages_per_split = p.stages;
    for (int q = 1; rem > 0 && q <= 16; ++q) {
        const int sps = ((p.stages + q - 1) / q + 1) / 2 * 2;
        if (q > 1 && (sps < 16 || (p.stages + sps - 1) / sps != q || rem * q > 320)) continue;
        const double c = (double)((rem * q + 255) / 256) * (7.0 + sps * 1.3) + (q > 1 ? 5.0 + rem * q * 0.1 : 0.0);
        if (c < best) { best = c; p.splits = q; p.stages_per_split = sps; }
    }
    const double large = (double)(p.full / 256) * (7.0 + p.stages * 1.3) + best;
    p.tile_blocks = p.full + rem * p.splits;
    p.big = !few && M >= 64 && large < 0.95 * small;
    p.tile = few ? 64 : p.sps >= 40 && t256x128 * p.S <= 256 && t256x128 * p.S >= 180 && t256x128 * 5 <= t128 * 3 ? 256 : 128;
    p.piece_elems = p.big ? (p.splits > 1 ? (int64_t)rem * p.splits * 65536 : 0) : (p.S > 1 ? p.S * nk : 0);
    p.blocks128 = t128 * p.S;
    if (!p.big) p.tile_blocks = (p.tile == 64 ? t64 : p.tile == 256 ? t256x128 : t128) * p.S;
    p.elems = p.piece_elems;
    for (int k = 0; k < count; ++k) p.elems += (int64_t)sums_of(p, M, N[k]).chunks * N[k];
    return p;
}
int64_t wgrad_scratch_elems(int M, const int* N, const int* K, int count) { return wgrad_plan(M, N, K, count).elems; }

int launch_wgrad_dma_group(hipStream_t s, const WgradGroup& grp, int M, int sps);
int launch_wgrad_big(hipStream_t s, const WgradBig& p);
int launch_gemm_wgrad(hipStream_t s, const GemmCall<bf16>& nn, int M, const WgradTail& tail, const RedSeg* segs, int nseg, GemmShape shape,
                      const GemmCall<bf16>* nt);

// One launch for all of it where the column sums come in one piece and 256x256 tiles would not be the better ones for the weight
// gradients.  as_apart: only where a launch of their own would sum them in one piece too, which is what two streams take.
bool gemm_wgrad_bf16_together(int M, const int* wn, const int* wk, int count, bool as_apart) {
    if (M > COLSUM_ROWS) return false;
    const WgradPlan p = wgrad_plan(M, wn, wk, count);
    return !p.big && (!as_apart || p.S == 1);
}

static int check_wgrad_items(const WgradItem* items, int count, int M, int* N, int* K, double* flops) {
    if (count < 1 || count > WGRAD_GROUP_MAX) { set_error("gemm_wgrad_bf16: 1 to 4 weight gradients per launch"); return REV_EINVAL; }
    for (int k = 0; k < count; ++k) {
        const WgradItem& it = items[k];
        if ((it.ldg & 7) || (it.lda & 7) || (it.N & 7) || (it.K & 7) || (((uintptr_t)it.G | (uintptr_t)it.A | (uintptr_t)it.dW) & 15)) {
            set_error("gemm_wgrad_bf16: sizes must be multiples of 8 and every buffer 16-byte aligned");
            return REV_EINVAL;
        }
        N[k] = it.N; K[k] = it.K;
        *flops += 2.0 * M * it.N * it.K;
    }
    return REV_OK;
}

// 64x64 or 128x128 tiles over all of up to COLSUM_ROWS tokens, column sums in one piece: for the last workgroups of another launch
int gemm_wgrad_bf16_beside(const WgradItem* items, int count, int M, WgradTail* out, double* flops) {
    int N[WGRAD_GROUP_MAX], K[WGRAD_GROUP_MAX];
    if (M > COLSUM_ROWS) { set_error("gemm_wgrad_bf16: too many rows to ride in another launch"); return REV_EINVAL; }
    if (int rc = check_wgrad_items(items, count, M, N, K, flops)) return rc;
    *out = {};
    WgradGroup& g = out->grp;
    int nsums = 0, t64 = 0;
    for (int k = 0; k < count; ++k) t64 += tiles_of(N[k], K[k], 64, 64);
    g.count = count;
    g.tile = t64 <= 512 ? 64 : 128;
    for (int k = 0; k < count; ++k) {
        const WgradItem& it = items[k];
        g.p[k] = {it.G, it.A, it.dW, it.ldg, it.lda, 0, it.N, it.K, g.tiles_total};
        g.tiles_total += tiles_of(it.N, it.K, g.tile, g.tile);
        if (!it.colsum) continue;
        if (nsums == WGRAD_SUMS_MAX) { set_error("gemm_wgrad_bf16: too many column sums"); return REV_EINVAL; }
        g.sums[nsums++] = {it.G, it.colsum, it.colsum, it.ldg, it.N, M, 1, g.sum_blocks};
        g.sum_blocks += colsum_blocks(it.N);
    }
    for (int k = nsums; k < WGRAD_SUMS_MAX; ++k) g.sums[k].block0 = g.sum_blocks;
    g.tile_blocks = g.tiles_total;
    out->M = M;
    out->steps = (M + WG_BR - 1) / WG_BR;
    return REV_OK;
}
int gemm_nn_wgrad_bf16(hipStream_t s, const GemmCall<bf16>& nn, int M, const WgradItem* items, int count, const RedSeg* segs, int nseg,
                       const GemmCall<bf16>* beside) {
    if (int rc = check_gemm(nn.A, nn.lda, nn.B, nn.ldb, nn.N, nn.K, nn.epi)) return rc;
    if (beside)
        if (int rc = check_gemm(beside->A, beside->lda, beside->B, beside->ldb, beside->N, beside->K, beside->epi)) return rc;
    WgradTail tail;
    double flops = 2.0 * M * ((double)nn.N * nn.K + (beside ? (double)beside->N * beside->K : 0.0)), us;
    if (int rc = gemm_wgrad_bf16_beside(items, count, M, &tail, &flops)) return rc;
    ProfScope ps(K_MIXED, s, flops);
    // 64x64 tiles where 32x32 ones do not all run at once, or cost more
    const GemmShape shape = beside ? pair_shape(nn, *beside, M, true) : ring_shape(M, nn.N, nn.K, EPI_PLAIN, true, &us);
    return launch_gemm_wgrad(s, nn, M, tail, segs, nseg, shape, beside);
}

int gemm_wgrad_bf16_group(hipStream_t s, const WgradItem* items, int count, int M, float* scratch, int64_t scratch_elems,
                          RedSeg* segs, int* nseg) {
    *nseg = 0;
    int N[WGRAD_GROUP_MAX], K[WGRAD_GROUP_MAX];
    double flops = 0;
    if (int rc = check_wgrad_items(items, count, M, N, K, &flops)) return rc;
    const WgradPlan pl = wgrad_plan(M, N, K, count);
    if (pl.elems > 0 && (scratch == nullptr || scratch_elems < pl.elems)) {
        set_error("gemm_wgrad_bf16: scratch too small");
        return REV_EWORKSPACE;
    }
    WgradSums sums[WGRAD_SUMS_MAX] = {};
    int nsums = 0, sum_blocks = 0;
    float* sums_scratch = scratch + pl.piece_elems;
    for (int k = 0; k < count; ++k)
        if (items[k].colsum) {
            if (nsums == WGRAD_SUMS_MAX) { set_error("gemm_wgrad_bf16: too many column sums"); return REV_EINVAL; }
            WgradSums& q = sums[nsums++];
            q = sums_of(pl, M, N[k]);
            q.g = items[k].G; q.ld = items[k].ldg; q.total = items[k].colsum; q.block0 = sum_blocks;
            q.out = pl.big || q.chunks > 1 ? sums_scratch : q.total;
            sums_scratch += (int64_t)q.chunks * q.n;
            sum_blocks += !pl.big && pl.tile != 256 && q.chunks == 1 ? colsum_blocks(q.n) : q.chunks * ((q.n + 511) / 512);
        }
    for (int k = nsums; k < WGRAD_SUMS_MAX; ++k) sums[k].block0 = sum_blocks;
    ProfScope ps(K_GEMM_WGRAD, s, flops);
    if (pl.big) {
        WgradBig b = {};
        b.count = count; b.M = M; b.tiles = pl.tiles; b.full = pl.full; b.splits = pl.splits;
        b.stages = pl.stages; b.stages_per_split = pl.stages_per_split; b.tile_blocks = pl.tile_blocks;
        b.partial = scratch; b.sum_blocks = sum_blocks;
        for (int k = 0; k < WGRAD_SUMS_MAX; ++k) b.sums[k] = sums[k];
        for (int k = 0, t = 0; k < count; ++k) {
            const WgradItem& it = items[k];
            b.p[k] = {it.G, it.A, it.dW, it.ldg, it.lda, it.N, it.K, t};
            t += tiles_of(it.N, it.K, 256, 256);
        }
        return launch_wgrad_big(s, b);
    }
    WgradGroup grp = {};
    grp.count = count; grp.tile = pl.tile; grp.tile_blocks = pl.tile_blocks; grp.sum_blocks = sum_blocks;
    const int bp = pl.tile, bq = pl.tile == 64 ? 64 : 128;
    for (int k = 0; k < WGRAD_SUMS_MAX; ++k) grp.sums[k] = sums[k];
    float* part = scratch;
    for (int k = 0; k < count; ++k) {
        const WgradItem& it = items[k];
        const int64_t nk = (int64_t)it.N * it.K;
        grp.p[k] = {it.G, it.A, pl.S > 1 ? part : it.dW, it.ldg, it.lda, nk, it.N, it.K, grp.tiles_total};
        grp.tiles_total += tiles_of(it.N, it.K, bp, bq);
        if (pl.S > 1) {
            segs[(*nseg)++] = {part, it.dW, nullptr, nk, nk, nk, pl.S};
            part += pl.S * nk;
        }
    }
    for (int k = 0; k < nsums; ++k)
        if (sums[k].chunks > 1) segs[(*nseg)++] = {sums[k].out, sums[k].total, nullptr, sums[k].n, sums[k].n, sums[k].n, sums[k].chunks};
    return launch_wgrad_dma_group(s, grp, M, pl.sps);
}

}  // namespace rev
