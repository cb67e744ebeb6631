// bf16 GEMM in 256x256 tiles, for launches whose tiles fill most of the chip (big_tiles_pay, gemm_mfma.hip):
//   C[M,N] (+epilogue) = A[M,K] * B[N,K]^T   or, with BKM,   A[M,K] * B[K,N];   M, N >= 256, K a multiple of 128.
//
// One workgroup of 8 wavefronts per CU, 128 output columns x 64 rows of the tile per wavefront (weights on the A port, so an
// accumulator quad holds 4 consecutive columns).  A stage is 64 of K; it travels as four PARTS of 16 KB (B rows or columns
// 0..127 and 128..255, A the same) through two stages of LDS.  A part is requested again, for the stage after next, as soon as everybody has
// read it, so seven phases of products pass between a request and its use.
//
// A stage is four phases of one quadrant each (B part x A part, 8 products of 32x32x16 per wavefront).  In a phase a wavefront first reads
// the part that the quadrant needs beyond those it holds (A0, A1, B1, next stage's B0), requests one, and then multiplies.  The two
// wavefronts of a SIMD are half a phase apart, so that one multiplies while the other reads; the barrier between the halves
// also orders the reads of a part before its next request.
//
// The last tile of a row or column of tiles is moved back to end at M or N; what its neighbour also computes is not stored.
//
// What bounds it: the matrix cores under this card's power limit while it multiplies (a stage takes 1.28 us with all CUs at
// work, 0.84 with 48 of them), and the epilogue, which nothing overlaps: 8 us a tile for a plain output, 15 for GELU, 18 for
// GELU' (vector ALU).  The 128x128 kernel, two workgroups per CU, hides the epilogue but has one stage in flight per workgroup and twice
// the operand bytes per product: 1.1 us for half the products.  us, 128x128 or 160x128 tiles before and now: M = 8224, N = 1280, K = 5120:
// 125 -> 90 (1.19 PFLOP/s), with the residual 156 -> 104; N = 3840, K = 1280: 86 -> 69; M = 16384, N = 768, K = 3072: 92 -> 65;
// N = 3072, K = 768 with GELU: 114 -> 92.
#include "gemm_epilogue.h"
#include <type_traits>

namespace rev {

constexpr int GB_PART = 16384, GB_LDS = 8 * GB_PART;
template <int V> using gb_int = std::integral_constant<int, V>;

template <int KIND, bool BKM>
__global__ __launch_bounds__(512, 2) void gemm_big_kernel(const bf16* __restrict__ A, int64_t lda, const bf16* __restrict__ B,
                                                          int64_t ldb, int M, int N, int K, Epi epi, int gn) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 2, wm = wave & 1, wn = wave >> 1;      // wavefronts w and w + 4 share a SIMD
    const int g = lane >> 5, fr = lane & 31;
    const int tiles_n = (N + 255) / 256, tiles_m = (M + 255) / 256;
    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    const int per_group = gn * tiles_m, tg = tile / per_group, in_grp = tile - tg * per_group;
    const int gw = min(gn, tiles_n - tg * gn);
    const int m_first = (in_grp / gw) * 256, n_first = (tg * gn + in_grp % gw) * 256;   // the first row and column that are this tile's
    const int m0 = __builtin_amdgcn_readfirstlane(min(m_first, M - 256)), n0 = __builtin_amdgcn_readfirstlane(min(n_first, N - 256));

    // ---- sources: two wavefront-wide loads per part ----
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
    const unsigned lds0 = (unsigned)(uintptr_t)LDS_PTR(unsigned char, smem), lds_w = lds0 + wave * 1024;
    // parts: 0 B0, 1 B1, 2 A0, 3 A1; in LDS B0 B1 of stage 0, B0 B1 of stage 1, then the same of A
    auto issue = [&](auto part_tag, int kt) {
        constexpr int part = decltype(part_tag)::value;
        const unsigned sb = lds_w + (part >> 1) * (4 * GB_PART) + (kt & 1) * (2 * GB_PART) + (part & 1) * GB_PART;
        if constexpr (part >= 2) {
            const char* src = a_base + (part & 1) * 256 * lda + kt * 128;
            dma16_sbase(src, va, sb);
            dma16_sbase(src + 128 * lda, va, sb + 8192);
        } else if constexpr (BKM) {
            const char* src = b_base + (part & 1) * 256 + (int64_t)kt * 128 * ldb;
            dma16_sbase(src, vb, sb);
            dma16_sbase(src + 64 * ldb, vb, sb + 8192);
        } else {
            const char* src = b_base + (part & 1) * 256 * ldb + kt * 128;
            dma16_sbase(src, vb, sb);
            dma16_sbase(src + 128 * ldb, vb, sb + 8192);
        }
    };
    using PB0 = gb_int<0>; using PB1 = gb_int<1>; using PA0 = gb_int<2>; using PA1 = gb_int<3>;
    issue(PB0{}, 0); issue(PA0{}, 0); issue(PA1{}, 0); issue(PB1{}, 0);
    issue(PB0{}, 1); issue(PA0{}, 1); issue(PA1{}, 1); issue(PB1{}, 1);

    unsigned a_addr[4], b_addr[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const int koff = ((2 * kk + g) ^ ((fr >> 1) & 7)) << 4;
        a_addr[kk] = lds0 + 4 * GB_PART + (wn * 32 + fr) * 128 + koff;
        b_addr[kk] = lds0 + (wm * 64 + fr) * 128 + koff;
    }
    if (BKM) {
        const int jj = lane & 15, qq = lane >> 4;
        const int r = (qq >> 1) * 8 + (jj >> 2);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int c = wm * 64 + i * 32 + (qq & 1) * 16 + 4 * (jj & 3);
            b_addr[i] = lds0 + r * 256 + (((c >> 3) ^ (4 * (r & 3))) << 4) + (c & 7) * 2;
        }
    }
    u32x4_t b0[4][2], b1[4][2], a0[4], a1[4];
    auto read_b = [&](u32x4_t (&f)[4][2], auto half_tag, auto par_tag) {
        constexpr int off = decltype(half_tag)::value * GB_PART + decltype(par_tag)::value * (2 * GB_PART);
        if constexpr (BKM) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                f[0][i] = join64(lds_read_tr16_b64(b_addr[i], off), lds_read_tr16_b64(b_addr[i], off + 1024));
                f[1][i] = join64(lds_read_tr16_b64(b_addr[i], off + 4096), lds_read_tr16_b64(b_addr[i], off + 5120));
                f[2][i] = join64(lds_read_tr16_b64(b_addr[i], off + 8192), lds_read_tr16_b64(b_addr[i], off + 9216));
                f[3][i] = join64(lds_read_tr16_b64(b_addr[i], off + 12288), lds_read_tr16_b64(b_addr[i], off + 13312));
            }
        } else {
            f[0][0] = lds_read_b128(b_addr[0], off); f[0][1] = lds_read_b128(b_addr[0], off + 4096);
            f[1][0] = lds_read_b128(b_addr[1], off); f[1][1] = lds_read_b128(b_addr[1], off + 4096);
            f[2][0] = lds_read_b128(b_addr[2], off); f[2][1] = lds_read_b128(b_addr[2], off + 4096);
            f[3][0] = lds_read_b128(b_addr[3], off); f[3][1] = lds_read_b128(b_addr[3], off + 4096);
        }
    };
    auto read_a = [&](u32x4_t (&f)[4], auto half_tag, auto par_tag) {
        constexpr int off = decltype(half_tag)::value * GB_PART + decltype(par_tag)::value * (2 * GB_PART);
        f[0] = lds_read_b128(a_addr[0], off);
        f[1] = lds_read_b128(a_addr[1], off);
        f[2] = lds_read_b128(a_addr[2], off);
        f[3] = lds_read_b128(a_addr[3], off);
    };
    auto pin_b = [&](u32x4_t (&f)[4][2]) {
        asm volatile("" : "+v"(f[0][0]), "+v"(f[0][1]), "+v"(f[1][0]), "+v"(f[1][1]), "+v"(f[2][0]), "+v"(f[2][1]), "+v"(f[3][0]), "+v"(f[3][1]));
    };
    auto pin_a = [&](u32x4_t (&f)[4]) { asm volatile("" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3])); };

    f32x16_t acc[2][2][2];                                         // [B half][A half][32-column tile of B]
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[h][j][i][v] = 0.f;
    auto barrier = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto products = [&](u32x4_t (&fb)[4][2], u32x4_t (&fa)[4], f32x16_t (&c)[2]) {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int i = 0; i < 2; ++i) c[i] = mfma32(as_bf16x8(fb[kk][i]), as_bf16x8(fa[kk]), c[i]);
        __builtin_amdgcn_s_setprio(0);
    };
    // kind 0 requests as it goes; kind 1 is the last stage but one, kind 2 the last
    auto stage = [&](auto par_tag, auto kind_tag, int kt) {
        constexpr int par = decltype(par_tag)::value, kind = decltype(kind_tag)::value;
        using SP = gb_int<par>; using NP = gb_int<1 - par>;
        read_a(a0, gb_int<0>{}, SP{});
        if (kind == 0) issue(PB0{}, kt + 2);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kind == 0 ? 12 : kind == 1 ? 10 : 2) : "memory");
        pin_a(a0);
        barrier();
        products(b0, a0, acc[0][0]);
        barrier();

        read_a(a1, gb_int<1>{}, SP{});
        if (kind == 0) issue(PA0{}, kt + 2);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kind == 0 ? 12 : kind == 1 ? 8 : 0) : "memory");
        pin_a(a1);
        barrier();
        products(b0, a1, acc[0][1]);
        barrier();

        read_b(b1, gb_int<1>{}, SP{});
        if (kind == 0) issue(PA1{}, kt + 2);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kind == 0 ? 12 : kind == 1 ? 6 : 0) : "memory");
        pin_b(b1);
        barrier();
        products(b1, a1, acc[1][1]);
        barrier();

        if (kind != 2) read_b(b0, gb_int<0>{}, NP{});
        if (kind == 0) issue(PB1{}, kt + 2);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kind == 0 ? 12 : kind == 1 ? 4 : 0) : "memory");
        if (kind != 2) pin_b(b0);
        barrier();
        products(b1, a0, acc[1][0]);
        barrier();
    };
    const int nst = K >> 6;
    wait_vm<12>();                                                 // B0 and A0 of stage 0 have landed
    barrier();
    read_b(b0, gb_int<0>{}, gb_int<0>{});
    wait_lds();
    pin_b(b0);
    barrier();
    if (grp) barrier();                                            // half a phase behind
    int kt = 0;
    for (; kt + 3 < nst; kt += 2) {                                // an even number of stages, at least two
        stage(gb_int<0>{}, gb_int<0>{}, kt);
        stage(gb_int<1>{}, gb_int<0>{}, kt + 1);
    }
    stage(gb_int<0>{}, gb_int<1>{}, kt);
    stage(gb_int<1>{}, gb_int<2>{}, kt + 1);
    if (!grp) barrier();

    // ---- epilogue: 32 rows x 64 columns at a time through LDS of the wavefront's own, out in rows of 64 columns ----
    constexpr int CP = 68, NP = 8;
    float* ct = reinterpret_cast<float*>(smem) + wave * (32 * CP);
    const int c4 = lane & 15, rr = lane >> 4;
    auto row_of = [&](int j) { return m0 + j * 128 + wn * 32 + rr; };
    auto col_of = [&](int h) { return n0 + h * 128 + wm * 64 + 4 * c4; };
    constexpr bool OPND = KIND == EPI_RESIDUAL || KIND == EPI_GELU_BWD;
    f32x4_t opnd[2][NP], bv[2], csum[2][2];
    auto request = [&](f32x4_t (&o)[NP], int j, int h) {
#pragma unroll
        for (int p = 0; p < NP; ++p) o[p] = epi_load4<KIND>(epi, row_of(j) + 4 * p, col_of(h));
    };
    if (OPND) request(opnd[0], 0, 0);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        bv[h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (KIND == EPI_BIAS || KIND == EPI_BIAS_GELU || KIND == EPI_RESIDUAL) bv[h] = ld_bf16x4(reinterpret_cast<const bf16*>(epi.bias) + col_of(h));
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int j = q >> 1, h = q & 1;
        if (OPND && q < 3) request(opnd[(q + 1) & 1], (q + 1) >> 1, (q + 1) & 1);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                const f32x16_t& c = acc[h][j][i];
                *reinterpret_cast<f32x4_t*>(ct + fr * CP + i * 32 + 8 * vq + 4 * g) = f32x4_t{c[4 * vq], c[4 * vq + 1], c[4 * vq + 2], c[4 * vq + 3]};
            }
        f32x4_t v[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) v[p] = *reinterpret_cast<const f32x4_t*>(ct + (p * 4 + rr) * CP + 4 * c4);
        f32x4_t cs = {0.f, 0.f, 0.f, 0.f};
        const int n = col_of(h);
        if (n >= n_first) {
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int m = row_of(j) + 4 * p;
                if (m >= m_first) {
                    const f32x4_t o = epi_store4<KIND>(epi, m, n, v[p], bv[h], opnd[q & 1][p]);
                    if (KIND == EPI_GELU_BWD) cs += o;
                }
            }
        }
        csum[j][h] = cs;
    }
    if (KIND == EPI_GELU_BWD && epi.colsum != nullptr) {
        // column sums of strips of 64 rows, counted from m0: lanes of a column folded, then the wavefronts of a strip
        float* cs = reinterpret_cast<float*>(smem) + 8 * 32 * CP;  // [4 wn][2 j][256 columns]
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                f32x4_t s = csum[j][h];
#pragma unroll
                for (int off = 16; off < 64; off <<= 1)
#pragma unroll
                    for (int k = 0; k < 4; ++k) s[k] += __shfl_xor(s[k], off, 64);
                if (rr == 0) *reinterpret_cast<f32x4_t*>(cs + (wn * 2 + j) * 256 + h * 128 + wm * 64 + 4 * c4) = s;
            }
        __syncthreads();
        const int n = tid & 255, j = tid >> 8;
        if (n0 + n >= n_first) {
            const int strip = (m_first >> 6) + 2 * j;              // strips of this tile: four from its first row
#pragma unroll
            for (int s = 0; s < 2; ++s)
                epi.colsum[(int64_t)(strip + s) * N + n0 + n] = cs[(2 * s * 2 + j) * 256 + n] + cs[((2 * s + 1) * 2 + j) * 256 + n];
        }
    }
}

template <int KIND, bool BKM>
static int launch_big(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K, const Epi& epi) {
    static LdsLimit lim;
    auto kern = gemm_big_kernel<KIND, BKM>;
    if (int rc = lim.ensure(reinterpret_cast<const void*>(kern), GB_LDS)) return rc;
    const int tiles_n = (N + 255) / 256, tiles = (M + 255) / 256 * tiles_n;
    const int gn = tiles_n <= 6 ? tiles_n : 4;
    hipLaunchKernelGGL(kern, dim3(tiles), dim3(512), GB_LDS, s, A, lda, B, ldb, M, N, K, epi, gn);
    REV_HIP(hipGetLastError());
    return REV_OK;
}

// Bias, GELU and residual: B is [N, K]; GELU' and plain: B as stored, [K, N]; float32: either.
int gemm_bf16_big(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K, const Epi& epi, bool b_kmajor) {
    switch (epi.kind * 2 + b_kmajor) {
#define CASE(KIND, BKM) case KIND * 2 + BKM: return launch_big<KIND, BKM>(s, A, lda, B, ldb, M, N, K, epi);
        CASE(EPI_BIAS, false) CASE(EPI_BIAS_GELU, false) CASE(EPI_RESIDUAL, false) CASE(EPI_GELU_BWD, true) CASE(EPI_PLAIN, true)
        CASE(EPI_PLAIN_F32, false) CASE(EPI_PLAIN_F32, true)
#undef CASE
    }
    set_error("gemm_bf16: unknown epilogue");
    return REV_EINVAL;
}

}  // namespace rev
