// Internal declarations shared by the translation units of librevstack.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <stdint.h>
#include <string>
#include <cmath>
#include <atomic>

#include "rev_stack.h"

namespace rev {

typedef __hip_bfloat16 bf16;

// ---- error plumbing -------------------------------------------------------
void set_error(const std::string& msg);
int  hip_fail(hipError_t e, const char* what, const char* file, int line);

#define REV_HIP(expr)                                                        \
    do {                                                                     \
        hipError_t _e = (expr);                                              \
        if (_e != hipSuccess) return ::rev::hip_fail(_e, #expr, __FILE__, __LINE__); \
    } while (0)

// Raises a kernel's dynamic-LDS limit once per process.  Callable from several host threads: the runtime call is
// idempotent and the flag is published only after it has succeeded, so whoever finds it set may launch.
struct LdsLimit {
    std::atomic<bool> done{false};
    int ensure(const void* kern, int bytes) {
        if (done.load(std::memory_order_acquire)) return 0;
        hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(MaxDynamicSharedMemorySize)", __FILE__, __LINE__);
        done.store(true, std::memory_order_release);
        return 0;
    }
};

// ---- kernel families for the per-family timing ------------------------------
enum Kind {
    K_GEMM_NT = 0,   // activation x weight^T contractions (forward/recompute and dgrad)
    K_GEMM_WGRAD,    // weight-gradient contractions (long reduction over tokens)
    K_ATTN_FWD,
    K_ATTN_BWD,
    K_LN_FWD,
    K_LN_BWD,
    K_COLSUM,        // bias gradients (column sums), first stage
    K_REDUCE,        // fixed-order second stage of column sums / split reductions
    K_CONVERT,       // dtype conversion
    K_OPTIM,         // optimizer update
    K_MIXED,         // launches of small blocks that hold products of several of the families above
    K_LN_PAIR,       // LayerNorm backward of one block with LayerNorm forward of another
    K_COUNT
};

// Brackets a launch with events when profiling is on; otherwise nothing.
struct ProfScope {
    ProfScope(Kind k, hipStream_t s, double work);
    ~ProfScope();
    Kind kind; hipStream_t stream; void* rec;
};
bool profiling();

// AdamW update of n packed elements (optimizer.hip)
int adamw_step(hipStream_t s, int64_t n, float* master, void* params_bf16, const float* grad, float* m, float* v,
               int step, float lr, float beta1, float beta2, float eps, float weight_decay);
// plain SGD update of n packed elements (optimizer.hip)
int sgd_step(hipStream_t s, int64_t n, float* master, void* params_bf16, const float* grad, float lr);

// ---- small device helpers ------------------------------------------------------
__device__ __forceinline__ float to_f(float v) { return v; }
__device__ __forceinline__ float to_f(bf16 v) { return __bfloat162float(v); }
template <typename T> __device__ __forceinline__ T from_f(float v);
template <> __device__ __forceinline__ float from_f<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16 from_f<bf16>(float v) { return __float2bfloat16(v); }

// Sum over the 64 lanes, result in every lane.  Rotations inside each row of 16 lanes are DPP
// modifiers of the add itself (no LDS round trip); the four row sums are then read out as scalars.
// The order of the additions is fixed.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_mov<0x128>(v);    // row_ror:8
    v += dpp_mov<0x124>(v);    // row_ror:4
    v += dpp_mov<0x122>(v);    // row_ror:2
    v += dpp_mov<0x121>(v);    // row_ror:1
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
    return (r0 + r1) + (r2 + r3);
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// exact GELU and its derivative (erf form)
__device__ __forceinline__ float gelu_f(float x) {
    return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f));
}
__device__ __forceinline__ float gelu_grad_f(float x) {
    float cdf = 0.5f * (1.0f + erff(x * 0.70710678118654752f));
    float pdf = 0.39894228040143268f * __expf(-0.5f * x * x);
    return cdf + x * pdf;
}

// One fixed-order column reduction, described so that several of them can share a launch:
// out[i] = sum over p = 0..P-1 (ascending) of partial[p * stride + i] for i < n; elements [0, split) go to
// `out`, elements [split, n) to `out2` (dropped if out2 is null).
struct RedSeg {
    const float* partial;
    float* out;
    float* out2;
    int64_t stride, n, split;
    int P;
};
constexpr int RED_MAX_SEGS = 12;
// All segments in one launch (every length a multiple of 4, nseg <= RED_MAX_SEGS).
int reduce_multi(hipStream_t s, const RedSeg* segs, int nseg);

// ---- epilogue description shared by the GEMM launchers ----------------------------
enum EpiKind {
    EPI_BIAS = 0,      // out = acc + bias[n]                               (out: act type)
    EPI_BIAS_GELU,     // h = acc + bias[n]; out = h (skipped when out is null); out2 = gelu(h)   (act type)
    EPI_RESIDUAL,      // outf = res[m,n] + sign * (acc + bias[n])          (float32)
    EPI_GELU_BWD,      // out = acc * gelu'(aux[m,n])                       (act type)
    EPI_PLAIN,         // out = acc                                         (act type)
    EPI_PLAIN_F32,     // outf = acc                                        (float32)
    EPI_ERF = 16       // added to a GELU kind by the bf16 dispatch: the normal CDF by erff instead of the polynomial
};

struct Epi {
    int kind;
    void* out;          // act-typed output  [M, ldo]
    void* out2;         // second act-typed output (gelu)
    float* outf;        // float32 output
    const void* bias;   // parameter-typed [N]
    const float* res;   // float32 [M, ldo]
    const void* aux;    // act-typed [M, ldo] (pre-activation for GELU backward)
    float sign;
    int64_t ldo;
    float* colsum;      // EPI_GELU_BWD, matrix-core path: per-row-strip column sums of the output,
                        // [gemm_colsum_strips(M, N, K)][N] float32 (nullable)
    bool solo;          // the launch runs alone on the device (one stream): the tile shape may be chosen
                        // to fill the chip by itself; results do not depend on it
};
// rows of column-sum partials (strips of 32 or 64 token rows) that a bf16 GEMM writes
int gemm_colsum_strips(int M, int N, int K);
// tile of a bf16 GEMM launch: gemm_ring.hip (the first five), gemm_nt_dma.hip, gemm_mid.hip and gemm_big.hip (the last two)
enum GemmShape { GS_32x32, GS_64x64, GS_64x128_RING, GS_128x128_RING, GS_192x128_RING, GS_128x128, GS_160x128, GS_256x128, GS_256x256 };

// C[M,N] (+epilogue) = A[M,K] * B[N,K]^T.  A, B row-major with leading dims lda, ldb.
// fp32 flavour: A, B float.  bf16 flavour: A, B bf16.
int gemm_nt_f32(hipStream_t s, const float* A, int64_t lda, const float* B, int64_t ldb,
                int M, int N, int K, const Epi& epi);
int gemm_nt_bf16(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb,
                 int M, int N, int K, const Epi& epi);
// C[M,N] = A[M,K] * B[K,N]  (B row-major [K, ldb]): the input-gradient form, weights as stored.
int gemm_nn_bf16(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb,
                 int M, int N, int K, const Epi& epi);
int gemm_nn_f32(hipStream_t s, const float* A, int64_t lda, const float* B, int64_t ldb,
                int M, int N, int K, const Epi& epi);
// An input gradient A[M,K] * B[K,N] (GELU' or plain) and a map of the other chain A[M,K] * B[N,K]^T (GELU, residual or bias, in
// this order of the pairs), which do not depend on each other: one launch where neither fills the chip, two otherwise.
template <typename T> struct GemmCall { const T* A; int64_t lda; const T* B; int64_t ldb; int N, K; Epi epi; };
int gemm_pair(hipStream_t s, const GemmCall<bf16>& nn, const GemmCall<bf16>& nt, int M);
int gemm_pair(hipStream_t s, const GemmCall<float>& nn, const GemmCall<float>& nt, int M);
// rows of column-sum partials a float32 GEMM with an [M, N] output writes
int gemm_f32_colsum_strips(int M, int N);
// dW[N,K] (float32, ld = K) = G[M,N]^T * A[M,K], reduction over the M tokens: up to WGRAD_GROUP_MAX of them over the same
// tokens in ONE launch (the four of a transformer block), whose tiles together fill the device, so that the token
// range is cut into fewer pieces than each would need alone.  segs receives the fixed-order reductions of the pieces
// that are left for a reduce_multi (at most one per item and per column sum), their number in *nseg.
constexpr int WGRAD_GROUP_MAX = 4;
struct WgradItem {
    const bf16* G; int64_t ldg;        // cotangent [M, N]
    const bf16* A; int64_t lda;        // activation [M, K]
    int N, K;
    float* dW;                         // [N, K]
    float* colsum;                     // column sums of G [N] (nullable, at most WGRAD_SUMS_MAX of a group): the bias gradient
};
int gemm_wgrad_bf16_group(hipStream_t s, const WgradItem* items, int count, int M, float* scratch, int64_t scratch_elems,
                          RedSeg* segs, int* nseg);
int64_t wgrad_scratch_elems(int M, const int* N, const int* K, int count);   // floats of scratch it needs for these shapes
// Rows up to which the column sums that ride in a launch of weight gradients come in one piece (sums.h): 1024 rows take about 7 us,
// less than the products beside them.
constexpr int COLSUM_ROWS = 1024;
// The float32 flavour: up to WGRAD_GROUP_MAX weight gradients in one launch, no pieces; colsum (nullable, one of a group, up to
// COLSUM_ROWS rows): the column sums of G.
struct WgradF32Item { const float* G; int64_t ldg; const float* A; int64_t lda; int N, K; float* dW; float* colsum; };
int gemm_wgrad_f32_group(hipStream_t s, const WgradF32Item* items, int count, int M);
// C[M,N] = A[M,K] * B[K,N], weight gradients over the same M rows, and second stages of sums in one launch, for small blocks
// (gemm_wgrad_f32_together); beside (nullable): a residual map of the other chain, in the same launch
bool gemm_wgrad_f32_together(int M, int N, const int* wn, const int* wk, int count);
int gemm_nn_wgrad_f32(hipStream_t s, const GemmCall<float>& nn, int M, const WgradF32Item* items, int count, const RedSeg* segs, int nseg,
                      const GemmCall<float>* beside);
// Column sums that ride in a weight-gradient launch: its last workgroups take 512 columns of one of `chunks` runs of `rows`
// tokens each (n = 0: none); the chunks' sums go to out[chunk * n + column].
// At most two cotangents; block0: the first of a cotangent's workgroups, counted from the first behind the tiles.
constexpr int WGRAD_SUMS_MAX = 2;
struct WgradSums { const bf16* g; float* out; float* total; int64_t ld; int n, rows, chunks, block0; };
// device-side description of the launch (gemm_wgrad_dma.hip)
struct WgradProblem { const bf16* G; const bf16* A; float* out; int64_t ldg, lda, split_stride; int N, K, tile0; };
// tile: 64 (64x64), 128 (128x128) or 256 (256x128)
struct WgradGroup { WgradProblem p[WGRAD_GROUP_MAX]; WgradSums sums[WGRAD_SUMS_MAX]; int count, tile, tiles_total, tile_blocks, sum_blocks; };
// Weight gradients that ride in the last workgroups of another launch over the same M rows, where gemm_wgrad_bf16_together says so:
// of the attention backward (attention_backward_wgrad), and, with second stages of sums too, of an input gradient out[M,N] =
// A[M,K] * B[K,N], where a residual map of the other chain may ride too (beside, nullable).
struct WgradTail { WgradGroup grp; int M, steps; };
bool gemm_wgrad_bf16_together(int M, const int* wn, const int* wk, int count, bool as_apart);
int gemm_wgrad_bf16_beside(const WgradItem* items, int count, int M, WgradTail* out, double* flops);
int gemm_nn_wgrad_bf16(hipStream_t s, const GemmCall<bf16>& nn, int M, const WgradItem* items, int count, const RedSeg* segs, int nseg,
                       const GemmCall<bf16>* beside);
// The same in 256x256 tiles (gemm_wgrad_big.hip): `full` tiles run over all tokens, the others over `splits` ranges of them.
struct WgradBigProblem { const bf16* G; const bf16* A; float* dW; int64_t ldg, lda; int N, K, tile0; };
struct WgradBig {
    WgradBigProblem p[WGRAD_GROUP_MAX];
    WgradSums sums[WGRAD_SUMS_MAX];
    float* partial;               // 256x256 blocks [(tile - full) * splits + range]
    int M, count, tiles, full, splits, stages, stages_per_split, tile_blocks, sum_blocks;
};

// attention with float32 products (attention_f32.hip): float32 mode, and the backward of bf16 heads wider than 96
int attention_forward_f32(hipStream_t s, const float* qkv, float* o, float* lse, int B, int T, int H, int dh, const int* key_len);
template <typename T>
int attention_backward_f32(hipStream_t s, const T* qkv, const T* o, const T* dout, const float* lse, T* dqkv, int B, int Tn, int H,
                           int dh, const int* key_len);

// ---- memory-bound kernels ---------------------------------------------------------
// y = LN(x; g, b), stats[2*row] = mean, stats[2*row+1] = rstd
template <typename TA, typename TP>
int ln_forward(hipStream_t s, const float* x, const TP* g, const TP* b, float eps,
               TA* y, float* stats, int M, int D);
// out = r + LNbwd(dn; x, stats, g);  outb (nullable) = act-typed copy of out;
// dgb[0:D] = d gamma, dgb[D:2D] = d beta, dbias[D] (nullable) = column sums of out;
// all three float32, summed in a fixed order via `partial` (>= ln_bwd_partial_elems floats)
template <typename TA, typename TP>
int ln_backward(hipStream_t s, const TA* dn, const float* x, const float* stats, const TP* g,
                const float* r, float* out, TA* outb, float* dgb, float* dbias,
                float* partial, int M, int D, RedSeg* defer = nullptr);
int64_t ln_bwd_partial_elems(int M, int D);
// Two launches that do not depend on each other as one, where neither fills the chip (two otherwise); the arguments of
// ln_backward and ln_forward, with the same results.
template <typename TA, typename TP>
struct LnBwdCall {
    const TA* dn; const float *x, *stats; const TP* g; const float* r; float* out; TA* outb; float *dgb, *dbias, *partial;
};
template <typename TA, typename TP> struct LnFwdCall { const float* x; const TP *g, *b; float eps; TA* y; float* stats; };
template <typename TA, typename TP>
int ln_pair(hipStream_t s, const LnBwdCall<TA, TP>& b, const LnFwdCall<TA, TP>& f, int M, int D, RedSeg* defer);

// out[n] = sum_m in[m, n]   (float32 out, fixed summation order).  With `defer` the second stage is not
// launched: its description is returned for a later reduce_multi.
template <typename T>
int colsum(hipStream_t s, const T* in, int64_t ld, int M, int N, float* out, float* partial, RedSeg* defer = nullptr);
int64_t colsum_partial_elems(int M, int N);

// out = in in bf16 (nullable) and the column sums of in; their second stage is left for a reduce_multi.  partial:
// colsum_partial_elems floats, at most M * N
int convert_colsum(hipStream_t s, const float* in, bf16* out, int M, int N, float* sums, float* partial, RedSeg* defer);

// ---- attention ----------------------------------------------------------------------
// qkv [B*T, 3D] (q|k|v, head-major inside each), o [B*T, D], lse [B, H, T].
// key_len (nullable, device, [B]): key-padding mask -- the keys at positions >= key_len[b] (clamped to
// [1, T]) of sample b are left out of every softmax of that sample; all T query rows are computed.
template <typename TA>
int attention_forward(hipStream_t s, const TA* qkv, TA* o, float* lse, int B, int T, int H, int dh,
                      const int* key_len = nullptr);
template <typename TA>
int attention_backward(hipStream_t s, const TA* qkv, const TA* o, const TA* dout, const float* lse,
                       TA* dqkv, float* delta, int B, int T, int H, int dh, const int* key_len = nullptr,
                       bool solo = false);     // solo: the launch has the device to itself (one stream)

// The attention backward of bf16 heads and weight gradients over the same rows in one launch, where attention_takes_wgrad says so;
// beside (nullable): with the attention forward of the other chain
template <typename T> struct AttnFwdCall { const T* qkv; T* o; float* lse; };
bool attention_takes_wgrad(int B, int T, int H, int dh);
int attention_backward_wgrad(hipStream_t s, const bf16* qkv, const bf16* o, const bf16* dout, const float* lse, bf16* dqkv, int B, int T,
                             int H, int dh, const int* key_len, const WgradItem* items, int count, const AttnFwdCall<bf16>* beside = nullptr);
// float32: the backward and the forward of the other chain, in one launch while both leave the chip idle
int attention_pair_f32(hipStream_t s, const float* qkv, const float* o, const float* dout, const float* lse, float* dqkv, int B, int T, int H,
                       int dh, const int* key_len, const AttnFwdCall<float>& fwd);

}  // namespace rev
