// Weight gradients of a block in 256x256 tiles:  dW[N,K] = sum over tokens m of G[m,n] * A[m,k], up to four of them in one
// launch, for token counts and widths at which such tiles fill the chip (wgrad_plan, gemm_mfma.hip).
//
// One workgroup of 8 wavefronts per CU, 128x64 of the tile per wavefront.  Both operands have the token as their slow
// index: a stage is 64 tokens of 256 columns of each, kept in LDS as it lies in memory and read with the transpose read.
// It travels as four PARTS of 128 columns (16 KB: G columns 0..127 and 128..255, A the same) through two stages of LDS;
// a part is requested again, for the stage after next, as soon as everybody has read it, so seven phases of
// products pass between a request and its use.
//
// A stage is four phases of one quadrant each (G part x A part, 8 products of 32x32x16 per wavefront).  In a phase a
// wavefront first reads the part that the quadrant needs beyond those it holds (A0, A1, G1, next stage's G0), requests
// one, and then multiplies.  The two wavefronts of a SIMD are half a phase apart, so that one multiplies while the other
// reads; the barrier between the halves also orders the reads of a part before its next request.
//
// What bounds it: the matrix cores, busy 57 % of the launch, under this card's power limit (products and barriers alone run at
// 1.65 PFLOP/s).  The four of a block and the QKV bias gradient, with the kernel that adds the pieces, launches back to
// back: 12608 tokens, D = 768: 174 us (1.03 PFLOP/s; in a whole pass 151 and 15 for the pieces), in 128x128 tiles 220.  8224
// tokens, D = 1280: 273 us (1.18 PFLOP/s) against 408.
//
// Columns beyond N or K re-read the last valid ones (never stored).
#include "mfma.h"
#include <type_traits>

namespace rev {

constexpr int WB_PART = 16384, WB_LDS = 8 * WB_PART;
template <int V> using wb_int = std::integral_constant<int, V>;

__global__ __launch_bounds__(512, 2) void wgrad_big_kernel(WgradBig p) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    if ((int)blockIdx.x >= p.tile_blocks) {
        wgrad_tail_sums<8>(p.sums, p.M, blockIdx.x - p.tile_blocks, reinterpret_cast<float*>(smem));
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 2, wm = wave & 1, wn = wave >> 1;      // wavefronts w and w + 4 share a SIMD
    const int g = lane >> 5, fr = lane & 31;

    // ---- which tile, which token range ----
    int t, split = 0, st0 = 0, nst = p.stages, slot = -1;
    if ((int)blockIdx.x < p.full) {
        t = (blockIdx.x & ~255) + xcd_remap(blockIdx.x & 255, 256);
    } else {
        const int rem = p.tiles - p.full;
        const int lin = xcd_remap(blockIdx.x - p.full, rem * p.splits);
        split = __builtin_amdgcn_readfirstlane(lin / rem);             // the quotients come from vector registers
        t = p.full + lin - split * rem;
        st0 = split * p.stages_per_split;
        nst = min(p.stages_per_split, p.stages - st0);
        if (p.splits > 1) slot = (t - p.full) * p.splits + split;
    }
    int pi = 0;
#pragma unroll
    for (int k = 1; k < WGRAD_GROUP_MAX; ++k)
        if (k < p.count && t >= p.p[k].tile0) pi = k;
    const WgradBigProblem& q = p.p[pi];
    const bf16* G = q.G; const bf16* A = q.A;
    const int64_t ldg = q.ldg, lda = q.lda;
    const int N = q.N, K = q.K, M = p.M;
    // the slow tile index is the one along the wider output dimension
    const int tiles_k = (K + 255) / 256, tiles_n = (N + 255) / 256, lt = t - q.tile0;
    const int tn = __builtin_amdgcn_readfirstlane(K > N ? lt % tiles_n : lt / tiles_k);
    const int tk = __builtin_amdgcn_readfirstlane(K > N ? lt / tiles_n : lt % tiles_k);
    const int n0 = tn * 256, k0 = tk * 256;

    // ---- sources: two wavefront-wide loads of 4 token rows per part, 32 rows apart.  A stage that reaches beyond the last
    // token takes the last 64 tokens instead; those of them that belong to the stages before it are masked out of G
    // when they are multiplied (mask_g) ----
    unsigned vg[2], va[2];
    {
        const int krow = wave * 4 + (lane >> 4);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = h * 128 + ((lane & 15) ^ (4 * (krow & 3))) * 8;
            vg[h] = (unsigned)(krow * ldg * 2 + min(c, N - 8 - n0) * 2);
            va[h] = (unsigned)(krow * lda * 2 + min(c, K - 8 - k0) * 2);
        }
    }
    const char* g_base = reinterpret_cast<const char*>(G + (int64_t)st0 * 64 * ldg + n0);
    const char* a_base = reinterpret_cast<const char*>(A + (int64_t)st0 * 64 * lda + k0);
    const unsigned lds0 = (unsigned)(uintptr_t)LDS_PTR(unsigned char, smem), lds_w = lds0 + wave * 1024;
    const int last_row = M - st0 * 64 - 64;                        // first token of the last full stage, from this range's start
    // parts: 0 G0, 1 G1, 2 A0, 3 A1; in LDS G0 G1 of stage 0, G0 G1 of stage 1, then the same of A
    auto issue = [&](auto part_tag, int kt) {
        constexpr int part = decltype(part_tag)::value;
        const unsigned sb = lds_w + (part >> 1) * (4 * WB_PART) + (kt & 1) * (2 * WB_PART) + (part & 1) * WB_PART;
        const int64_t ld = part < 2 ? ldg : lda;
        const char* src = (part < 2 ? g_base : a_base) + min(kt * 64, last_row) * ld * 2;
        dma16_sbase(src, part < 2 ? vg[part & 1] : va[part & 1], sb);
        dma16_sbase(src + 64 * ld, part < 2 ? vg[part & 1] : va[part & 1], sb + 8192);
    };
    using PG0 = wb_int<0>; using PG1 = wb_int<1>; using PA0 = wb_int<2>; using PA1 = wb_int<3>;
    issue(PG0{}, 0); issue(PA0{}, 0); issue(PA1{}, 0); issue(PG1{}, 0);
    issue(PG0{}, 1); issue(PA0{}, 1); issue(PA1{}, 1); issue(PG1{}, 1);

    unsigned g_addr[2], a_addr;
    {
        const int jj = lane & 15, qq = lane >> 4;
        const int r = (qq >> 1) * 8 + (jj >> 2);
        auto at = [&](int c) { return lds0 + r * 256 + (((c >> 3) ^ (4 * (r & 3))) << 4) + (c & 7) * 2; };
        const int c = (qq & 1) * 16 + 4 * (jj & 3);
        g_addr[0] = at(wm * 64 + c);
        g_addr[1] = at(wm * 64 + 32 + c);
        a_addr = at(wn * 32 + c) + 4 * WB_PART;
    }
    u32x4_t g0[4][2], g1[4][2], a0[4], a1[4];
    auto read_frag = [&](unsigned addr, auto off_tag) {
        constexpr int off = decltype(off_tag)::value;
        return join64(lds_read_tr16_b64(addr, off), lds_read_tr16_b64(addr, off + 1024));
    };
    auto read_g = [&](u32x4_t (&f)[4][2], auto half_tag, auto par_tag) {
        constexpr int off = decltype(half_tag)::value * WB_PART + decltype(par_tag)::value * (2 * WB_PART);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            f[0][i] = read_frag(g_addr[i], wb_int<off>{});
            f[1][i] = read_frag(g_addr[i], wb_int<off + 4096>{});
            f[2][i] = read_frag(g_addr[i], wb_int<off + 8192>{});
            f[3][i] = read_frag(g_addr[i], wb_int<off + 12288>{});
        }
    };
    auto read_a = [&](u32x4_t (&f)[4], auto half_tag, auto par_tag) {
        constexpr int off = decltype(half_tag)::value * WB_PART + decltype(par_tag)::value * (2 * WB_PART);
        f[0] = read_frag(a_addr, wb_int<off>{});
        f[1] = read_frag(a_addr, wb_int<off + 4096>{});
        f[2] = read_frag(a_addr, wb_int<off + 8192>{});
        f[3] = read_frag(a_addr, wb_int<off + 12288>{});
    };
    auto pin_g = [&](u32x4_t (&f)[4][2]) {
        asm volatile("" : "+v"(f[0][0]), "+v"(f[0][1]), "+v"(f[1][0]), "+v"(f[1][1]), "+v"(f[2][0]), "+v"(f[2][1]), "+v"(f[3][0]), "+v"(f[3][1]));
    };
    auto pin_a = [&](u32x4_t (&f)[4]) { asm volatile("" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3])); };

    f32x16_t acc[2][2][2];                                         // [G half][A half][32-column tile of G]
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
    auto products = [&](u32x4_t (&fg)[4][2], u32x4_t (&fa)[4], f32x16_t (&c)[2]) {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int i = 0; i < 2; ++i) c[i] = mfma32(as_bf16x8(fg[kk][i]), as_bf16x8(fa[kk]), c[i]);
        __builtin_amdgcn_s_setprio(0);
    };
    // clears the first `skip` tokens of a stage in the fragments of G
    auto mask_g = [&](u32x4_t (&f)[4][2], int skip) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int t = kk * 16 + 8 * g + 2 * e;
                const unsigned keep = (t >= skip ? 0xFFFFu : 0u) | (t + 1 >= skip ? 0xFFFF0000u : 0u);
#pragma unroll
                for (int i = 0; i < 2; ++i) f[kk][i][e] &= keep;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // kind 0 requests as it goes; kind 1 is the last stage but one, kind 2 the last
    auto stage = [&](auto par_tag, auto kind_tag, int kt) {
        constexpr int par = decltype(par_tag)::value, kind = decltype(kind_tag)::value;
        using SP = wb_int<par>; using NP = wb_int<1 - par>;
        if (kind != 0) mask_g(g0, kt * 64 - last_row);             // none of them, unless the stage is beyond the last full one
        read_a(a0, wb_int<0>{}, SP{});
        if (kind == 0) issue(PG0{}, kt + 2);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kind == 0 ? 12 : kind == 1 ? 10 : 2) : "memory");
        pin_a(a0);
        barrier();
        products(g0, a0, acc[0][0]);
        barrier();

        read_a(a1, wb_int<1>{}, SP{});
        if (kind == 0) issue(PA0{}, kt + 2);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kind == 0 ? 12 : kind == 1 ? 8 : 0) : "memory");
        pin_a(a1);
        barrier();
        products(g0, a1, acc[0][1]);
        barrier();

        read_g(g1, wb_int<1>{}, SP{});
        if (kind == 0) issue(PA1{}, kt + 2);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kind == 0 ? 12 : kind == 1 ? 6 : 0) : "memory");
        pin_g(g1);
        if (kind != 0) mask_g(g1, kt * 64 - last_row);
        barrier();
        products(g1, a1, acc[1][1]);
        barrier();

        if (kind != 2) read_g(g0, wb_int<0>{}, NP{});
        if (kind == 0) issue(PG1{}, kt + 2);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kind == 0 ? 12 : kind == 1 ? 4 : 0) : "memory");
        if (kind != 2) pin_g(g0);
        barrier();
        products(g1, a0, acc[1][0]);
        barrier();
    };
    wait_vm<12>();                                                 // G0 and A0 of stage 0 have landed
    barrier();
    read_g(g0, wb_int<0>{}, wb_int<0>{});
    wait_lds();
    pin_g(g0);
    barrier();
    if (grp) barrier();                                            // half a phase behind
    int kt = 0;
    for (; kt + 3 < nst; kt += 2) {                                // an even number of stages, at least two
        stage(wb_int<0>{}, wb_int<0>{}, kt);
        stage(wb_int<1>{}, wb_int<0>{}, kt + 1);
    }
    stage(wb_int<0>{}, wb_int<1>{}, kt);
    stage(wb_int<1>{}, wb_int<2>{}, kt + 1);
    if (!grp) barrier();

    // ---- out: lane (fr, g) holds column k = fr of a 32x32 tile, rows n = 8 (v / 4) + 4 g + v % 4 ----
    float* out = slot < 0 ? q.dW + (int64_t)n0 * K + k0 : p.partial + (int64_t)slot * 65536;
    const int64_t ldo = slot < 0 ? K : 256;
    const int nlim = slot < 0 ? N - n0 : 256, klim = slot < 0 ? K - k0 : 256;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int k = j * 128 + wn * 32 + fr, nb = h * 128 + wm * 64 + i * 32 + 4 * g;
                if (k < klim) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int n = nb + 8 * (v >> 2) + (v & 3);
                        if (n < nlim) out[n * ldo + k] = acc[h][j][i][v];
                    }
                }
            }
}

// Tiles whose tokens were cut into ranges: the ranges' tiles are added in range order, 64 blocks of 4 rows per tile.  The
// blocks after them add the chunks of the column sums.
__global__ __launch_bounds__(256) void wgrad_big_reduce_kernel(WgradBig p) {
    const int ti = blockIdx.x >> 6, part = blockIdx.x & 63, t = p.full + ti;
    if (p.splits == 1 || t >= p.tiles) {
        int n = (blockIdx.x - (p.splits == 1 ? 0 : (p.tiles - p.full) * 64)) * 256 + threadIdx.x;
        const WgradSums& q = n >= p.sums[0].n ? p.sums[1] : p.sums[0];
        if (n >= p.sums[0].n) n -= p.sums[0].n;
        if (n >= q.n) return;
        float s = 0.f;
        int c = 0;
        for (; c + 8 <= q.chunks; c += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = q.out[(int64_t)(c + u) * q.n + n];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; c < q.chunks; ++c) s += q.out[(int64_t)c * q.n + n];
        q.total[n] = s;
        return;
    }
    int pi = 0;
#pragma unroll
    for (int k = 1; k < WGRAD_GROUP_MAX; ++k)
        if (k < p.count && t >= p.p[k].tile0) pi = k;
    const WgradBigProblem& q = p.p[pi];
    const int tiles_k = (q.K + 255) / 256, tiles_n = (q.N + 255) / 256, lt = t - q.tile0;
    const int tn = q.K > q.N ? lt % tiles_n : lt / tiles_k, tk = q.K > q.N ? lt / tiles_n : lt % tiles_k;
    const int n = tn * 256 + part * 4 + (threadIdx.x >> 6), k = tk * 256 + (threadIdx.x & 63) * 4;
    if (n < q.N && k < q.K) {
        const float* src = p.partial + (int64_t)ti * p.splits * 65536 + part * 1024 + threadIdx.x * 4;
        float4 s = *reinterpret_cast<const float4*>(src);
        for (int r = 1; r < p.splits; ++r) {
            const float4 v = *reinterpret_cast<const float4*>(src + (int64_t)r * 65536);
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
        *reinterpret_cast<float4*>(q.dW + (int64_t)n * q.K + k) = s;
    }
}

int launch_wgrad_big(hipStream_t s, const WgradBig& p) {
    static LdsLimit lim;
    if (int rc = lim.ensure(reinterpret_cast<const void*>(wgrad_big_kernel), WB_LDS)) return rc;
    hipLaunchKernelGGL(wgrad_big_kernel, dim3(p.tile_blocks + p.sum_blocks), dim3(512), WB_LDS, s, p);
    REV_HIP(hipGetLastError());
    const int red = (p.splits > 1 ? (p.tiles - p.full) * 64 : 0) + (p.sums[0].n + p.sums[1].n + 255) / 256;
    if (red > 0) {
        hipLaunchKernelGGL(wgrad_big_reduce_kernel, dim3(red), dim3(256), 0, s, p);
        REV_HIP(hipGetLastError());
    }
    return REV_OK;
}

}  // namespace rev
