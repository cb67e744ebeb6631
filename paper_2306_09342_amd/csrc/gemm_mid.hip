// bf16 GEMM in 256x128 tiles, two workgroups of four wavefronts per CU, for the wide maps over short contractions:
//   h = A[M,K] * B[N,K]^T + bias, with or without gelu(h)   and, with BKM,   A[M,K] * B[K,N] * gelu'(h);   M >= 256, N >= 128, K
//   a multiple of 64.  Beside another stream's kernels also for narrow outputs, residual and plain.
//
// 128 columns x 64 rows of each half of the tile per wavefront (weights on the A port, so an accumulator quad holds 4
// consecutive columns).  A stage is 64 of K in three PARTS of 16 KB (B, rows 0..127 of A, rows 128..255), which travel in that
// order through a ring of five slots.  A stage is two phases of 16 products; one barrier per phase says both that its parts
// have landed and that those of the phase before have been read, whose slots are then requested again: three to four parts
// are in flight.
//
// What bounds it: operand rate and LDS reads while it multiplies (about 1.2 of the time of the 256x256 tiles of gemm_big.hip
// per product), HBM and vector ALU in the epilogue.  The two workgroups of a CU are not in step, so the epilogue of one runs
// beside the products of the other: over short contractions that outweighs the slower products.  us, 256x256 or 128x128 tiles
// / these: M = 25216, N = 1536, K = 384: 72 / 63; N = 2048, K = 512: 110 / 94; with GELU M = 50000, N = 1024, K = 256: 82 / 71.
// A forward and backward pass of 12 such blocks (width 384, 128 samples of 197): 10.82 -> 10.52 ms.  Without GELU, M = 25216:
// N = 1152, K = 384: 37.9 / 34.1; N = 1536, K = 512: 59.6 / 51.4 (less than two rounds of these, two and three of the others).
//
// The last tile of a row or column of tiles is moved back to end at M or N; what its neighbour also computes is not stored.
#include "gemm_epilogue.h"
#include <type_traits>

namespace rev {

constexpr int GM_PART = 16384, GM_SLOTS = 5, GM_LDS = GM_SLOTS * GM_PART;
template <int V> using gm_int = std::integral_constant<int, V>;

template <int KIND, bool BKM>
__global__ __launch_bounds__(256, 2) void gemm_mid_kernel(const bf16* __restrict__ A, int64_t lda, const bf16* __restrict__ B,
                                                          int64_t ldb, int M, int N, int K, Epi epi, int gn) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int g = lane >> 5, fr = lane & 31;
    const int tiles_n = (N + 127) / 128, tiles_m = (M + 255) / 256;
    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    const int per_group = gn * tiles_m, tg = tile / per_group, in_grp = tile - tg * per_group;
    const int gw = min(gn, tiles_n - tg * gn);
    const int m_first = (in_grp / gw) * 256, n_first = (tg * gn + in_grp % gw) * 128;
    const int m0 = __builtin_amdgcn_readfirstlane(min(m_first, M - 256)), n0 = __builtin_amdgcn_readfirstlane(min(n_first, N - 128));

    // ---- sources: four wavefront-wide loads per part ----
    unsigned va, vb;
    {
        const int row = wave * 8 + (lane >> 3), ch = (lane & 7) ^ ((row >> 1) & 7);
        va = (unsigned)(row * lda * 2 + ch * 16);
        if (BKM) {
            const int krow = wave * 4 + (lane >> 4);
            vb = (unsigned)(krow * ldb * 2 + (((lane & 15) ^ (4 * (krow & 3))) << 4));
        } else {
            vb = (unsigned)(row * ldb * 2 + ch * 16);
        }
    }
    const char* a_base = reinterpret_cast<const char*>(A + (int64_t)m0 * lda);
    const char* b_base = reinterpret_cast<const char*>(BKM ? B + n0 : B + (int64_t)n0 * ldb);
    const unsigned lds0 = (unsigned)(uintptr_t)LDS_PTR(unsigned char, smem);
    // a part goes to slot wslot, 16 KB; parts are requested and used in the order B, A0, A1 of one stage after the other
    int wslot = 0;
    auto next = [](int s) { return s == GM_SLOTS - 1 ? 0 : s + 1; };
    auto request_a = [&](int half, int kt) {
        const unsigned d = lds0 + wslot * GM_PART + wave * 1024;
        const char* src = a_base + half * 256 * lda + (int64_t)kt * 128;
#pragma unroll
        for (int t = 0; t < 4; ++t) dma16_sbase(src + t * 64 * lda, va, d + t * 4096);
        wslot = next(wslot);
    };
    auto request_b = [&](int kt) {
        const unsigned d = lds0 + wslot * GM_PART + wave * 1024;
        const char* src = BKM ? b_base + (int64_t)kt * 128 * ldb : b_base + (int64_t)kt * 128;
#pragma unroll
        for (int t = 0; t < 4; ++t) dma16_sbase(src + t * (BKM ? 32 : 64) * ldb, vb, d + t * 4096);
        wslot = next(wslot);
    };
    const int nk = K >> 6;
    request_b(0); request_a(0, 0); request_a(1, 0);
    if (nk > 1) request_b(1);

    unsigned a_off[4], b_off[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const int koff = ((2 * kk + g) ^ ((fr >> 1) & 7)) << 4;
        a_off[kk] = lds0 + (wn * 64 + fr) * 128 + koff;
        b_off[kk] = lds0 + (wm * 64 + fr) * 128 + koff;
    }
    if (BKM) {
        const int jj = lane & 15, qq = lane >> 4;
        const int r = (qq >> 1) * 8 + (jj >> 2);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int c = wm * 64 + i * 32 + (qq & 1) * 16 + 4 * (jj & 3);
            b_off[i] = lds0 + r * 256 + (((c >> 3) ^ (4 * (r & 3))) << 4) + (c & 7) * 2;
        }
    }
    u32x4_t a[4][2], b[4][2];
    auto read_a = [&](int kk, unsigned at) {
        a[kk][0] = lds_read_b128(a_off[kk] + at, 0);
        a[kk][1] = lds_read_b128(a_off[kk] + at, 4096);
    };
    auto read_b = [&](auto kk_tag, unsigned at) {
        constexpr int kk = decltype(kk_tag)::value;
        if constexpr (BKM) {
#pragma unroll
            for (int i = 0; i < 2; ++i) b[kk][i] = join64(lds_read_tr16_b64(b_off[i] + at, kk * 4096), lds_read_tr16_b64(b_off[i] + at, kk * 4096 + 1024));
        } else {
            b[kk][0] = lds_read_b128(b_off[kk] + at, 0);
            b[kk][1] = lds_read_b128(b_off[kk] + at, 4096);
        }
    };
    f32x16_t acc[2][2][2];                                         // [A half][32 rows of A][32 columns of B]
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[h][j][i][v] = 0.f;
    auto products = [&](f32x16_t (&c)[2][2], int kk) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i) c[j][i] = mfma32(as_bf16x8(b[kk][i]), as_bf16x8(a[kk][j]), c[j][i]);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto landed = [&](auto n_tag) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(decltype(n_tag)::value) : "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    int rslot = 0;
    // kind 0: requests go on; 1: the last stage but one; 2: the last
    auto stage = [&](auto kind_tag, int kt) {
        constexpr int kind = decltype(kind_tag)::value;
        constexpr int RB = BKM ? 6 : 4;                            // LDS reads per step of 16
        landed(gm_int<(kind == 2 ? 4 : 8)>{});
        if (kind != 2) request_a(0, kt + 1);
        const unsigned at_b = rslot * GM_PART;
        rslot = next(rslot);
        const unsigned at_a = rslot * GM_PART;
        rslot = next(rslot);
        read_b(gm_int<0>{}, at_b); read_a(0, at_a);
        read_b(gm_int<1>{}, at_b); read_a(1, at_a);
        __builtin_amdgcn_s_setprio(1);
        lds_wait4<RB>(a[0][0], a[0][1], b[0][0], b[0][1]);
        read_b(gm_int<2>{}, at_b); read_a(2, at_a); products(acc[0], 0);
        lds_wait4<RB>(a[1][0], a[1][1], b[1][0], b[1][1]);
        read_b(gm_int<3>{}, at_b); read_a(3, at_a); products(acc[0], 1);
        lds_wait4<RB>(a[2][0], a[2][1], b[2][0], b[2][1]);
        products(acc[0], 2);
        lds_wait4<0>(a[3][0], a[3][1], b[3][0], b[3][1]);
        products(acc[0], 3);
        __builtin_amdgcn_s_setprio(0);

        landed(gm_int<(kind == 2 ? 0 : 8)>{});
        if (kind != 2) request_a(1, kt + 1);
        if (kind == 0) request_b(kt + 2);
        const unsigned at_c = rslot * GM_PART;
        rslot = next(rslot);
        read_a(0, at_c); read_a(1, at_c); read_a(2, at_c); read_a(3, at_c);
        __builtin_amdgcn_s_setprio(1);
        lds_wait4<6>(a[0][0], a[0][1], b[0][0], b[0][1]);
        products(acc[1], 0);
        lds_wait4<4>(a[1][0], a[1][1], b[1][0], b[1][1]);
        products(acc[1], 1);
        lds_wait4<2>(a[2][0], a[2][1], b[2][0], b[2][1]);
        products(acc[1], 2);
        lds_wait4<0>(a[3][0], a[3][1], b[3][0], b[3][1]);
        products(acc[1], 3);
        __builtin_amdgcn_s_setprio(0);
    };
    int kt = 0;
    for (; kt + 2 < nk; ++kt) stage(gm_int<0>{}, kt);
    if (kt + 1 < nk) stage(gm_int<1>{}, kt++);
    stage(gm_int<2>{}, kt);

    // ---- epilogue: 32 rows x 64 columns at a time through LDS of the wavefront's own, out in rows of 64 columns ----
    __syncthreads();
    constexpr int CP = 68, NP = 8;
    float* ct = reinterpret_cast<float*>(smem) + wave * (32 * CP);
    const int c4 = lane & 15, rr = lane >> 4;
    const int n = n0 + wm * 64 + 4 * c4;
    auto row_of = [&](int q) { return m0 + (q >> 1) * 128 + wn * 64 + (q & 1) * 32 + rr; };
    constexpr bool OPND = KIND == EPI_RESIDUAL || KIND == EPI_GELU_BWD;
    f32x4_t opnd[2][NP];
    auto request = [&](f32x4_t (&o)[NP], int q) {
#pragma unroll
        for (int p = 0; p < NP; ++p) o[p] = epi_load4<KIND>(epi, row_of(q) + 4 * p, n);
    };
    if (OPND) request(opnd[0], 0);
    f32x4_t bv = {0.f, 0.f, 0.f, 0.f}, cs = {0.f, 0.f, 0.f, 0.f}, cs_first = cs;
    if (KIND == EPI_BIAS || KIND == EPI_BIAS_GELU || KIND == EPI_RESIDUAL) bv = ld_bf16x4(reinterpret_cast<const bf16*>(epi.bias) + n);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (OPND && q < 3) request(opnd[(q + 1) & 1], q + 1);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                const f32x16_t& c = acc[q >> 1][q & 1][i];
                *reinterpret_cast<f32x4_t*>(ct + fr * CP + i * 32 + 8 * vq + 4 * g) = f32x4_t{c[4 * vq], c[4 * vq + 1], c[4 * vq + 2], c[4 * vq + 3]};
            }
        f32x4_t v[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) v[p] = *reinterpret_cast<const f32x4_t*>(ct + (p * 4 + rr) * CP + 4 * c4);
        if (n >= n_first) {
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int m = row_of(q) + 4 * p;
                if (m >= m_first) {
                    const f32x4_t o = epi_store4<KIND>(epi, m, n, v[p], bv, opnd[q & 1][p]);
                    if (KIND == EPI_GELU_BWD) cs += o;
                }
            }
        }
        if (KIND == EPI_GELU_BWD && epi.colsum != nullptr) {
            // column sums of the wavefront's 64 rows: a strip, four from the tile's first row, in two halves as the 256x256 tiles add them
#pragma unroll
            for (int off = 16; off < 64; off <<= 1)
#pragma unroll
                for (int k = 0; k < 4; ++k) cs[k] += __shfl_xor(cs[k], off, 64);
            if ((q & 1) == 0) cs_first = cs;
            else if (rr == 0 && n >= n_first) *reinterpret_cast<f32x4_t*>(epi.colsum + (int64_t)((m_first >> 6) + (q & 2) + wn) * N + n) = cs_first + cs;
            cs = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
    }
}

template <int KIND, bool BKM>
static int launch_mid(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K, const Epi& epi) {
    static LdsLimit lim;
    auto kern = gemm_mid_kernel<KIND, BKM>;
    if (int rc = lim.ensure(reinterpret_cast<const void*>(kern), GM_LDS)) return rc;
    const int tiles_n = (N + 127) / 128, tiles = (M + 255) / 256 * tiles_n;
    const int gn = tiles_n <= 12 ? tiles_n : 8;
    hipLaunchKernelGGL(kern, dim3(tiles), dim3(256), GM_LDS, s, A, lda, B, ldb, M, N, K, epi, gn);
    REV_HIP(hipGetLastError());
    return REV_OK;
}

// GELU' and plain: B as stored, [K, N]; bias, GELU and residual: [N, K]
int gemm_bf16_mid(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K, const Epi& epi) {
    switch (epi.kind) {
        case EPI_BIAS: return launch_mid<EPI_BIAS, false>(s, A, lda, B, ldb, M, N, K, epi);
        case EPI_BIAS_GELU: return launch_mid<EPI_BIAS_GELU, false>(s, A, lda, B, ldb, M, N, K, epi);
        case EPI_RESIDUAL: return launch_mid<EPI_RESIDUAL, false>(s, A, lda, B, ldb, M, N, K, epi);
        case EPI_GELU_BWD: return launch_mid<EPI_GELU_BWD, true>(s, A, lda, B, ldb, M, N, K, epi);
        case EPI_PLAIN: return launch_mid<EPI_PLAIN, true>(s, A, lda, B, ldb, M, N, K, epi);
    }
    set_error("gemm_bf16: unknown epilogue");
    return REV_EINVAL;
}

}  // namespace rev
