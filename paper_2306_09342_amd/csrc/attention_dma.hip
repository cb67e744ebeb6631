// bf16 softmax attention for heads of 32, 64 or 80 features.  What a workgroup walks over travels to LDS with direct-to-LDS
// loads in 64-row tiles; a wavefront owns 32 rows and keeps their operands and sums in registers.
//
//   attn_fwd_dma       owns query rows, walks over K and V:    O, log-sum-exp
//   attn_bwd_dq_dma    owns query rows, walks over K and V:    dQ, delta
//   attn_bwd_dkv_dma   owns key rows, walks over Q and dO:     dK, dV
//   attn_bwd_pair_dma  the two passes in one launch, for launches that leave the chip partly idle
//   attn_bwd_fused     the two passes in one workgroup per head, for 32 or 64 features and up to 256 tokens
//
// A wavefront's sums have the same order in all of them, so which one a launch takes (attention_backward_dma) does not
// change a bit of its results.
//
// What bounds them: vector ALU and latency (one exp2 and about ten other instructions per score, softmax statistics in the middle of
// the chain); the tiles come from L2.  The ring kernels keep two tiles in flight and have workgroups of up to four wavefronts,
// one per SIMD, so that several share a CU and their phases overlap.  KB of LDS of a workgroup, beyond 64 tokens, and how
// many share a CU (LDS, or registers), for 32, 64 and 80 features: forward and dQ 16, 33, 41 KB and 4, 4, 3 of them; dK and dV 17,
// 34, 42 KB and 3, 3, 2; the pair 26, 50, 62 KB and 3, 2, 2.  (Half of it up to 64 tokens.)  Three or four tiles in flight
// cost occupancy and time everywhere (197 tokens, 64 features: 27 -> 31 us).  attn_bwd_fused holds a whole head, 16 to 133 KB, in a
// workgroup of up to eight wavefronts, two per SIMD.
// Measured, us, before (padded LDS rows, a whole head loaded per workgroup or the next tile fetched through registers, 80
// features padded to 96) and now.  Forward: 768 heads of 197 tokens, 64 features: 34 -> 27; 384 heads of 512: 66 -> 45;
// 512 heads of 257, 80 features: 84 -> 37; 12288 windows of 49, 32 features: 53 -> 42.  Backward: 384 heads of 512 tokens: 148 ->
// 126; 512 heads of 257, 80 features: 146 -> 108; one image of 12 heads, 197 tokens: 18.0 -> 12.0.
#include "attention.h"
#include "gemm_wgrad_dma.h"

namespace rev {

// ---- LDS tiles ---------------------------------------------------------------------------------------------------------
// Rows are dense (2 * DH bytes); the 16-byte chunk c of row r sits at position c ^ rsw<DH>(r), which serves both access
// patterns without padding: 16 consecutive rows of one chunk (operand fragments read row-wise) hit 16 distinct bank
// groups, and the rows of a transpose read spread over the banks (128-byte rows: 8 rows x 64 B; 64-byte rows: 8 whole rows,
// contiguous).
template <int DH> __device__ __forceinline__ int rsw(int r);
template <> __device__ __forceinline__ int rsw<64>(int r) {
    const int p = (r >> 1) & 7;
    return ((p & 1) << 2) | (p >> 1);
}
template <> __device__ __forceinline__ int rsw<32>(int r) { return (r >> 2) & 3; }
// 160-byte rows: 8 rows start in 8 different bank groups of 32 bytes, the next 8 in the same ones
template <> __device__ __forceinline__ int rsw<80>(int r) { return (r >> 3) & 1; }
// wavefront-wide load number i of a [nrows, ld] matrix with DH columns: rows RPL*i .. RPL*i + RPL-1 (RPL = 512 / DH
// rows of 2 * DH bytes, clamped to the last row) to the dense tile at dst
template <int DH>
__device__ __forceinline__ void res_dma8(unsigned char* dst, const bf16* __restrict__ base, int64_t ld, int nrows, int i, int lane) {
    constexpr int CPR = DH / 8, RPL = 64 / CPR;
    const int row = i * RPL + lane / CPR;
    const int c = (lane % CPR) ^ rsw<DH>(row);
    const unsigned voff = (unsigned)(min(row, nrows - 1) * (int)ld * 2 + c * 16);
    dma16_sbase(base, voff, (unsigned)(uintptr_t)LDS_PTR(unsigned char, dst) + i * 1024);
}
// Loads issued as inline assembly (the compiler's wait insertion neither sees them nor waits for the direct-to-LDS
// loads on their behalf); the caller waits with res_wait and then passes the registers through res_pin.
__device__ __forceinline__ u32x4_t res_load16(const void* p) {
    u32x4_t r;
    asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(r) : "v"(p) : "memory");
    return r;
}
__device__ __forceinline__ float res_load4(const void* p) {
    float r;
    asm volatile("global_load_dword %0, %1, off" : "=v"(r) : "v"(p) : "memory");
    return r;
}
// owned-row fragments of a head: lane (r = l%32, g) takes X[row0 + r][16*ks + 8g .. +7], rows clamped
template <int KS>
__device__ __forceinline__ void res_load_owned(const bf16* __restrict__ base, int64_t ld, int row0, int nrows, int lane,
                                               u32x4_t (&frag)[KS]) {
    const int r = min(row0 + (lane & 31), nrows - 1);
    const bf16* p = base + (int64_t)r * ld + 8 * (lane >> 5);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) frag[ks] = res_load16(p + 16 * ks);
}
template <int KS> __device__ __forceinline__ void res_pin(u32x4_t (&f)[KS]) {
    if constexpr (KS == 2) asm volatile("" : "+v"(f[0]), "+v"(f[1]));
    else if constexpr (KS == 4) asm volatile("" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]));
    else asm volatile("" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]), "+v"(f[4]));
}
__device__ __forceinline__ void res_pin(float& a) { asm volatile("" : "+v"(a)); }
template <int KS>
__device__ __forceinline__ void res_frags(const u32x4_t (&f)[KS], bf16x8_t (&b)[KS]) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) b[ks] = as_bf16x8(f[ks]);
}
// Requests rows [0, tp) of two matrices, 64-row tile by tile; returns through rem[j] how many of THIS wavefront's
// loads are younger than those of tile j (what may still be outstanding when tile j is consumed).
template <int DH>
__device__ __forceinline__ void res_request(unsigned char* d0, const bf16* b0, int64_t ld0, unsigned char* d1, const bf16* b1,
                                            int64_t ld1, int nrows, int tp, int wave, int nw, int lane, int (&rem)[4], int& total_out) {
    constexpr int RPL = 512 / DH, LPT = 64 / RPL;          // rows per wavefront-wide load, loads per 64-row tile
    int issued[4] = {0, 0, 0, 0}, total = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int i1 = min(LPT * j + LPT, tp / RPL);
        for (int i = LPT * j + wave; i < i1; i += nw) {
            res_dma8<DH>(d0, b0, ld0, nrows, i, lane);
            res_dma8<DH>(d1, b1, ld1, nrows, i, lane);
            total += 2;
        }
        issued[j] = total;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) rem[j] = total - issued[j];
    total_out = total;
}
// waits until at most n (wavefront-uniform) vector-memory loads of the wavefront are outstanding, or fewer where there is no step
// for n, and for all LDS operations
__device__ __forceinline__ void res_wait(int n) {
#define RES_WAIT(N) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(N))
    if (n >= 16) {
        if (n >= 40) RES_WAIT(40);
        else if (n >= 24) RES_WAIT(24);
        else RES_WAIT(16);
        return;
    }
    switch (n >> 1) {
        case 1: RES_WAIT(2); break;
        case 2: RES_WAIT(4); break;
        case 3: RES_WAIT(6); break;
        case 4: RES_WAIT(8); break;
        case 5: RES_WAIT(10); break;
        case 6: RES_WAIT(12); break;
        case 7: RES_WAIT(14); break;
        default: RES_WAIT(0); break;
    }
#undef RES_WAIT
}
// per-lane byte offsets of the two transpose reads of tr_frag<4, 8> in a resident tile, for r0 = 0 (any r0 that is a
// multiple of 16 adds r0 * 2 * DH) and feature tile dt
template <int DH>
__device__ __forceinline__ void res_tr_offsets(int lane, int dt, int& o1, int& o2) {
    const int j = lane & 15, q = lane >> 4;
    const int c = dt * 32 + (q & 1) * 16 + 4 * (j & 3);
    const int r = (q >> 1) * 4 + (j >> 2);
    o1 = r * (2 * DH) + (((c >> 3) ^ rsw<DH>(r)) << 4) + (c & 7) * 2;
    o2 = (r + 8) * (2 * DH) + (((c >> 3) ^ rsw<DH>(r + 8)) << 4) + (c & 7) * 2;
}
__device__ __forceinline__ bf16x8_t res_tr_frag(const unsigned char* tile_r0, int o1, int o2) {
    union { struct { s16x4_t lo, hi; } s; bf16x8_t v; } u;
    u.s.lo = lds_tr16(reinterpret_cast<const uint16_t*>(tile_r0 + o1));
    u.s.hi = lds_tr16(reinterpret_cast<const uint16_t*>(tile_r0 + o2));
    return u.v;
}

// What a workgroup walks over: NM matrices of one head in 64-row tiles, two tiles in flight.  Every wavefront requests its
// share of a tile; a tile is used after each wavefront has waited for its own share and all have met at a barrier, which
// is also where the tile before it is known to be free for the next request.  Rows from `rows` on are zeros.
// NS: 64 floats each of NS row statistics come along (clamped to the last row).
// TR: rows a tile has room for (32: only for sequences that are no longer).
template <int DH, int NM, int NS, int TR = 64>
struct TileRing {
    static constexpr int ROWB = 2 * DH, CPR = DH / 8, LPT = DH / 8, TILE = TR * ROWB, SLOT = NM * TILE + NS * 256;
    const bf16* base[NM];
    const float* stat[NS > 0 ? NS : 1];
    int64_t ld[NM];
    unsigned lds;
    int rows, nt, nw, wave, lane, issued, nfull, nlast;

    __device__ __forceinline__ static int loads_of(int n, int wave, int nw) { return wave < n ? (n - wave + nw - 1) / nw : 0; }
    __device__ __forceinline__ void init(unsigned char* smem, int rows_) {
        lds = (unsigned)(uintptr_t)LDS_PTR(unsigned char, smem);
        lane = threadIdx.x & 63; wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); nw = blockDim.x >> 6;
        rows = rows_; nt = (rows + 63) >> 6; issued = 0;
        const bool half = rows - (nt - 1) * 64 <= 32;               // the last tile holds 32 rows at most
        nfull = NM * loads_of(LPT, wave, nw) + (wave == 0 ? NS : 0);
        nlast = half ? NM * loads_of(LPT / 2, wave, nw) + (wave == 0 ? NS : 0) : nfull;
    }
    __device__ __forceinline__ void request() {
        const int j = issued++;
        const unsigned slot = lds + (unsigned)(j & 1) * SLOT;
        const int row0 = j * 64, left = rows - row0, n = left <= 32 ? LPT / 2 : LPT;
        for (int i = wave; i < n; i += nw) {
            const int idx = i * 64 + lane, row = idx / CPR, c = (idx - row * CPR) ^ rsw<DH>(row);
            const unsigned d = slot + i * 1024;
#pragma unroll
            for (int k = 0; k < NM; ++k) {
                if (left >= 64) {
                    dma16_sbase(base[k] + (int64_t)row0 * ld[k], (unsigned)(row * (int)ld[k] * 2 + c * 16), d + k * TILE);
                } else {
                    const bf16* z = reinterpret_cast<const bf16*>(g_zero_chunk);
                    dma16_ptr(row < left ? base[k] + (int64_t)(row0 + row) * ld[k] + c * 8 : z, d + k * TILE);
                }
            }
        }
        if (NS > 0 && wave == 0) {
            const unsigned off = (unsigned)min(row0 + lane, rows - 1) * 4;
#pragma unroll
            for (int k = 0; k < NS; ++k) dma4_sbase(stat[k], off, slot + NM * TILE + k * 256);
        }
    }
    // this wavefront's loads of tiles younger than j (all requested ones for j = -1)
    __device__ __forceinline__ int younger(int j) const {
        const int n = issued - 1 - j;
        return n <= 0 ? 0 : n * nfull - (issued == nt ? nfull - nlast : 0);
    }
    __device__ __forceinline__ void start() {
        request();
        if (nt > 1) request();
    }
    // tile j is in LDS for everybody when this returns; its byte offset
    __device__ __forceinline__ int get(int j) {
        asm volatile("" ::: "memory");
        res_wait(younger(j));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (j > 0 && issued < nt) request();
        return (j & 1) * SLOT;
    }
};

// ---- forward ----------------------------------------------------------------------------------------------------------
struct FwdArgs {
    const bf16* qkv;
    bf16* o;
    float* lse;
    const int* key_len;
    int T, H, nblk;              // nblk workgroups per head
};
template <int DH, int TR>
__device__ __forceinline__ void fwd_rows(const FwdArgs& a, unsigned char* smem, int blk) {
    constexpr int KS = DH / 16, DT = (DH + 31) / 32, ROWB = 2 * DH, NT = TR / 32;
    const bf16* __restrict__ qkv = a.qkv;
    bf16* __restrict__ o = a.o;
    float* __restrict__ lse = a.lse;
    const int* __restrict__ key_len = a.key_len;
    const int T = a.T, H = a.H, nblk = a.nblk;
    const int lane = threadIdx.x & 63, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int bh = blk / nblk, b = bh / H, h = bh - b * H;
    const int D = H * DH;
    const int64_t ld = 3 * (int64_t)D;
    const bf16* base = qkv + (int64_t)b * T * ld + h * DH;
    const int q0 = ((blk - bh * nblk) * nw + wave) * 32;
    const float c2 = rsqrtf((float)DH) * 1.4426950408889634f;
    const int Tk = key_len ? min(max(key_len[b], 1), T) : T;

    u32x4_t fq[KS];
    res_load_owned<KS>(base, ld, q0, T, lane, fq);
    TileRing<DH, 2, 0, TR> ring;
    ring.base[0] = base + D; ring.base[1] = base + 2 * D; ring.ld[0] = ring.ld[1] = ld;
    ring.init(smem, Tk);
    ring.start();
    res_wait(ring.younger(-1));
    res_pin<KS>(fq);
    bf16x8_t bq[KS];
    res_frags<KS>(fq, bq);

    int rowoff[KS], o1[DT], o2[DT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rowoff[ks] = (lane & 31) * ROWB + (((2 * ks + g) ^ rsw<DH>(lane & 31)) << 4);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) res_tr_offsets<DH>(lane, dt, o1[dt], o2[dt]);

    f32x16_t accO[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) accO[dt][v] = 0.f;
    float m = -INFINITY, l = 0.f;
    for (int j = 0; j < ring.nt; ++j) {
        const unsigned char* Ks = smem + ring.get(j);
        const unsigned char* Vs = Ks + TR * ROWB;
        const int left = Tk - j * 64;
        if (q0 >= T) continue;
        f32x16_t s[NT];
        float mloc = -INFINITY;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if (t == 0 || left > 32) {
#pragma unroll
                for (int v = 0; v < 16; ++v) s[t][v] = 0.f;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    s[t] = mfma32(*reinterpret_cast<const bf16x8_t*>(Ks + t * 32 * ROWB + rowoff[ks]), bq[ks], s[t]);
                if (t * 32 + 32 > left) {
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        if (t * 32 + 8 * (v >> 2) + 4 * g + (v & 3) >= left) s[t][v] = -INFINITY;
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) mloc = fmaxf(mloc, s[t][v]);
            }
        }
        mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64)) * c2;
        const float mn = fmaxf(m, mloc);
        const float corr = __builtin_amdgcn_exp2f(m - mn);
        float lsum = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (t == 0 || left > 32) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    s[t][v] = __builtin_amdgcn_exp2f(fmaf(s[t][v], c2, -mn));
                    lsum += s[t][v];
                }
            }
        lsum += __shfl_xor(lsum, 32, 64);
        l = l * corr + lsum;
        m = mn;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) accO[dt][v] *= corr;
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (t == 0 || left > 32) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    float p[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) p[e] = s[t][8 * c + e];
                    const bf16x8_t pb = pack8(p);
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt)
                        accO[dt] = mfma32(res_tr_frag(Vs + (t * 32 + 16 * c) * ROWB, o1[dt], o2[dt]), pb, accO[dt]);
                }
            }
    }
    // O^T tile: lane holds query q0 + l%32, features dt*32 + 8*(v/4) + 4g + v%4
    const int q = q0 + (lane & 31);
    if (q < T) {
        const float inv = 1.f / l;
        bf16* orow = o + ((int64_t)b * T + q) * D + h * DH;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const int d = dt * 32 + 8 * v4 + 4 * g;
                if (dt * 32 + 8 * v4 < DH)
                    store4_bf16(orow + d, accO[dt][4 * v4] * inv, accO[dt][4 * v4 + 1] * inv,
                                accO[dt][4 * v4 + 2] * inv, accO[dt][4 * v4 + 3] * inv);
            }
        if (g == 0) lse[(int64_t)bh * T + q] = (m + __log2f(l)) * 0.6931471805599453f;   // back to natural log
    }
}

template <int DH, int TR>
__global__ __launch_bounds__(256, DH == 80 ? 3 : 4) void attn_fwd_dma(FwdArgs a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    fwd_rows<DH, TR>(a, smem, xcd_remap(blockIdx.x, gridDim.x));
}

// ---- backward pass 1: dQ and delta ----------------------------------------------------------------------------------------
struct BwdArgs {
    const bf16 *qkv, *o, *dout;
    const float* lse;
    bf16* dqkv;
    float* delta;                // written by the dQ rows unless null
    const int* key_len;
    int T, H, nblk;              // nblk workgroups per head
};
template <int DH>
__device__ __forceinline__ void bwd_dq_rows(const BwdArgs& a, unsigned char* smem, int blk) {
    constexpr int KS = DH / 16, DT = (DH + 31) / 32, ROWB = 2 * DH;
    const bf16 *qkv = a.qkv, *o = a.o, *dout = a.dout;
    const float* lse = a.lse;
    const int* key_len = a.key_len;
    const int T = a.T, H = a.H, nblk = a.nblk;
    const int lane = threadIdx.x & 63, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int bh = blk / nblk, b = bh / H, h = bh - b * H;
    const int D = H * DH;
    const int64_t ld = 3 * (int64_t)D;
    const bf16* base = qkv + (int64_t)b * T * ld + h * DH;
    const bf16* dob = dout + (int64_t)b * T * D + h * DH;
    const bf16* ob = o + (int64_t)b * T * D + h * DH;
    const int q0 = ((blk - bh * nblk) * nw + wave) * 32;
    const int q = q0 + (lane & 31), qc = min(q, T - 1);
    const float scale = rsqrtf((float)DH), c2 = scale * 1.4426950408889634f;
    const int Tk = key_len ? min(max(key_len[b], 1), T) : T;

    u32x4_t fq[KS], fdo[KS], fo[KS];
    res_load_owned<KS>(base, ld, q0, T, lane, fq);
    res_load_owned<KS>(dob, D, q0, T, lane, fdo);
    res_load_owned<KS>(ob, D, q0, T, lane, fo);
    float Lraw = res_load4(lse + (int64_t)bh * T + qc);
    TileRing<DH, 2, 0> ring;
    ring.base[0] = base + D; ring.base[1] = base + 2 * D; ring.ld[0] = ring.ld[1] = ld;
    ring.init(smem, Tk);
    ring.start();
    res_wait(ring.younger(-1));
    res_pin<KS>(fq); res_pin<KS>(fdo); res_pin<KS>(fo); res_pin(Lraw);

    bf16x8_t bq[KS], bdo[KS];
    res_frags<KS>(fq, bq); res_frags<KS>(fdo, bdo);
    // delta_q = sum_d dO[q,d] * O[q,d]; the two half-wavefronts hold complementary feature slots
    float dl = 0.f;
    {
        bf16x8_t bo[KS];
        res_frags<KS>(fo, bo);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int e = 0; e < 8; ++e) dl += (float)bdo[ks][e] * (float)bo[ks][e];
        dl += __shfl_xor(dl, 32, 64);
    }
    const float L2 = Lraw * 1.4426950408889634f;

    int rowoff[KS], o1[DT], o2[DT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rowoff[ks] = (lane & 31) * ROWB + (((2 * ks + g) ^ rsw<DH>(lane & 31)) << 4);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) res_tr_offsets<DH>(lane, dt, o1[dt], o2[dt]);

    f32x16_t accQ[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) accQ[dt][v] = 0.f;
    for (int j = 0; j < ring.nt; ++j) {
        const unsigned char* Ks = smem + ring.get(j);
        const unsigned char* Vs = Ks + 64 * ROWB;
        const int left = Tk - j * 64;
        if (q0 >= T) continue;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (t == 0 || left > 32) {
                f32x16_t aS, aP;
#pragma unroll
                for (int v = 0; v < 16; ++v) { aS[v] = 0.f; aP[v] = 0.f; }
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    aS = mfma32(*reinterpret_cast<const bf16x8_t*>(Ks + t * 32 * ROWB + rowoff[ks]), bq[ks], aS);
                    aP = mfma32(*reinterpret_cast<const bf16x8_t*>(Vs + t * 32 * ROWB + rowoff[ks]), bdo[ks], aP);
                }
                // dS without its 1/sqrt(head_dim): that factor is applied once to the finished dQ
                float ds[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) ds[v] = __builtin_amdgcn_exp2f(aS[v] * c2 - L2) * (aP[v] - dl);
                if (t * 32 + 32 > left) {
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        if (t * 32 + 8 * (v >> 2) + 4 * g + (v & 3) >= left) ds[v] = 0.f;
                }
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const bf16x8_t dsb = pack8(&ds[8 * c]);
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt)
                        accQ[dt] = mfma32(res_tr_frag(Ks + (t * 32 + 16 * c) * ROWB, o1[dt], o2[dt]), dsb, accQ[dt]);
                }
            }
        }
    }
    if (q < T) {
        if (g == 0 && a.delta) a.delta[(int64_t)bh * T + q] = dl;
        bf16* dq = a.dqkv + ((int64_t)b * T + q) * ld + h * DH;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const int d = dt * 32 + 8 * v4 + 4 * g;
                if (dt * 32 + 8 * v4 < DH)
                    store4_bf16(dq + d, accQ[dt][4 * v4] * scale, accQ[dt][4 * v4 + 1] * scale,
                                accQ[dt][4 * v4 + 2] * scale, accQ[dt][4 * v4 + 3] * scale);
            }
    }
}

// ---- backward pass 2: dK and dV --------------------------------------------------------------------------------------------
// OWN_DELTA: delta of the streamed rows is formed here, from a third tile with their O, in the order of the dQ rows.
template <int DH, bool OWN_DELTA>
__device__ __forceinline__ void bwd_dkv_rows(const BwdArgs& a, unsigned char* smem, int blk) {
    constexpr int KS = DH / 16, DT = (DH + 31) / 32, ROWB = 2 * DH, TILE = 64 * ROWB;
    const bf16 *qkv = a.qkv, *dout = a.dout;
    const int* key_len = a.key_len;
    const int T = a.T, H = a.H, nblk = a.nblk;
    const int lane = threadIdx.x & 63, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int bh = blk / nblk, b = bh / H, h = bh - b * H;
    const int D = H * DH;
    const int64_t ld = 3 * (int64_t)D;
    const bf16* base = qkv + (int64_t)b * T * ld + h * DH;
    const bf16* dob = dout + (int64_t)b * T * D + h * DH;
    const int j0 = ((blk - bh * nblk) * nw + wave) * 32;
    const float scale = rsqrtf((float)DH), c2 = scale * 1.4426950408889634f;
    const int Tk = key_len ? min(max(key_len[b], 1), T) : T;      // keys beyond Tk are masked: their dK, dV are zero

    u32x4_t fk[KS], fv[KS];
    res_load_owned<KS>(base + D, ld, j0, T, lane, fk);
    res_load_owned<KS>(base + 2 * D, ld, j0, T, lane, fv);
    constexpr int NM = OWN_DELTA ? 3 : 2;
    TileRing<DH, NM, OWN_DELTA ? 1 : 2> ring;
    ring.base[0] = base; ring.base[1] = dob; ring.ld[0] = ld; ring.ld[1] = D;
    ring.stat[0] = a.lse + (int64_t)bh * T;
    if constexpr (OWN_DELTA) { ring.base[2] = a.o + (int64_t)b * T * D + h * DH; ring.ld[2] = D; }
    else ring.stat[1] = a.delta + (int64_t)bh * T;
    ring.init(smem, T);
    ring.start();
    res_wait(ring.younger(-1));
    res_pin<KS>(fk); res_pin<KS>(fv);
    bf16x8_t bk[KS], bv[KS];
    res_frags<KS>(fk, bk); res_frags<KS>(fv, bv);

    int rowoff[KS], o1[DT], o2[DT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rowoff[ks] = (lane & 31) * ROWB + (((2 * ks + g) ^ rsw<DH>(lane & 31)) << 4);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) res_tr_offsets<DH>(lane, dt, o1[dt], o2[dt]);

    // OWN_DELTA: 32 floats per wavefront behind the ring
    float* del_w = reinterpret_cast<float*>(smem + (ring.nt > 1 ? 2 : 1) * ring.SLOT + 64) + wave * 32;
    f32x16_t accK[DT], accV[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) { accK[dt][v] = 0.f; accV[dt][v] = 0.f; }
    for (int it = 0; it < ring.nt; ++it) {
        const unsigned char* Qs = smem + ring.get(it);
        const unsigned char* Os = Qs + 64 * ROWB;
        const float* lse_s = reinterpret_cast<const float*>(Qs + NM * TILE);
        const int left = T - it * 64;
        if (j0 >= Tk) continue;                              // nobody looked at these keys
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (t == 0 || left > 32) {
                f32x16_t aS, aP;
#pragma unroll
                for (int v = 0; v < 16; ++v) { aS[v] = 0.f; aP[v] = 0.f; }
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    aS = mfma32(*reinterpret_cast<const bf16x8_t*>(Qs + t * 32 * ROWB + rowoff[ks]), bk[ks], aS);
                    aP = mfma32(*reinterpret_cast<const bf16x8_t*>(Os + t * 32 * ROWB + rowoff[ks]), bv[ks], aP);
                }
                const float* del_s = lse_s + 64 + t * 32;
                if constexpr (OWN_DELTA) {
                    float dl = 0.f;
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        const bf16x8_t x = *reinterpret_cast<const bf16x8_t*>(Os + t * 32 * ROWB + rowoff[ks]);
                        const bf16x8_t y = *reinterpret_cast<const bf16x8_t*>(Os + TILE + t * 32 * ROWB + rowoff[ks]);
#pragma unroll
                        for (int e = 0; e < 8; ++e) dl += (float)x[e] * (float)y[e];
                    }
                    dl += __shfl_xor(dl, 32, 64);
                    del_w[lane & 31] = dl;                       // both halves hold the same value
                    del_s = del_w;
                }
                // lane: key j0 + l%32; rows i = 64 it + 32 t + 8*(v/4) + 4g + v%4
                float p[16], ds[16];
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) {
                    const float4 Lr = *reinterpret_cast<const float4*>(lse_s + t * 32 + 8 * v4 + 4 * g);
                    const float4 Dr = *reinterpret_cast<const float4*>(del_s + 8 * v4 + 4 * g);
                    const float Lv[4] = {Lr.x, Lr.y, Lr.z, Lr.w};
                    const float Dv[4] = {Dr.x, Dr.y, Dr.z, Dr.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int v = 4 * v4 + e;
                        p[v] = __builtin_amdgcn_exp2f(aS[v] * c2 - Lv[e] * 1.4426950408889634f);
                        ds[v] = p[v] * (aP[v] - Dv[e]);          // 1/sqrt(head_dim) applied to the finished dK
                    }
                }
                if (t * 32 + 32 > left) {
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        if (t * 32 + 8 * (v >> 2) + 4 * g + (v & 3) >= left) { p[v] = 0.f; ds[v] = 0.f; }
                }
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const bf16x8_t pb = pack8(&p[8 * c]);
                    const bf16x8_t dsb = pack8(&ds[8 * c]);
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt) {
                        accV[dt] = mfma32(res_tr_frag(Os + (t * 32 + 16 * c) * ROWB, o1[dt], o2[dt]), pb, accV[dt]);
                        accK[dt] = mfma32(res_tr_frag(Qs + (t * 32 + 16 * c) * ROWB, o1[dt], o2[dt]), dsb, accK[dt]);
                    }
                }
            }
        }
    }
    const int j = j0 + (lane & 31);
    if (j >= Tk) {                       // a masked key: no query looked at it
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) { accK[dt][v] = 0.f; accV[dt][v] = 0.f; }
    }
    if (j < T) {
        bf16* dk = a.dqkv + ((int64_t)b * T + j) * ld + D + h * DH;
        bf16* dv = dk + D;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const int d = dt * 32 + 8 * v4 + 4 * g;
                if (dt * 32 + 8 * v4 < DH) {
                    store4_bf16(dk + d, accK[dt][4 * v4] * scale, accK[dt][4 * v4 + 1] * scale,
                                accK[dt][4 * v4 + 2] * scale, accK[dt][4 * v4 + 3] * scale);
                    store4_bf16(dv + d, accV[dt][4 * v4], accV[dt][4 * v4 + 1], accV[dt][4 * v4 + 2], accV[dt][4 * v4 + 3]);
                }
            }
    }
}

template <int DH>
__global__ __launch_bounds__(256, DH == 80 ? 3 : 4) void attn_bwd_dq_dma(BwdArgs a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    bwd_dq_rows<DH>(a, smem, xcd_remap(blockIdx.x, gridDim.x));
}
template <int DH>
__global__ __launch_bounds__(256, DH == 80 ? 2 : 3) void attn_bwd_dkv_dma(BwdArgs a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    bwd_dkv_rows<DH, false>(a, smem, xcd_remap(blockIdx.x, gridDim.x));
}
// Both passes in one launch, half of the workgroups each: for launches that are too small to fill the chip.
template <int DH>
__global__ __launch_bounds__(256, 2) void attn_bwd_pair_dma(BwdArgs a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int n = gridDim.x >> 1, blk = blockIdx.x;
    if (blk < n) bwd_dq_rows<DH>(a, smem, xcd_remap(blk, n));
    else bwd_dkv_rows<DH, true>(a, smem, xcd_remap(blk - n, n));
}

// The pair and, in the workgroups behind its `attn_blocks`, weight gradients over the same rows: the pair leaves most of the chip idle
// for as long as they take.  12 heads of 197 tokens: 13.0 us, 17.0 with the three weight gradients of an MLP and a projection 768 wide, which
// take 10.4 by themselves.  FWD: the attention forward of the other chain (rev_stack.hip), in `fwd_blocks` before the weight gradients:
// 9.3 us by itself, here 16.7 -> 16.5.
template <int DH, bool FWD>
__global__ __launch_bounds__(256, 2) void attn_bwd_pair_wgrad(BwdArgs a, WgradTail w, int attn_blocks, FwdArgs f, int fwd_blocks) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int n = attn_blocks >> 1;
    int blk = blockIdx.x;
    if (blk < n) bwd_dq_rows<DH>(a, smem, xcd_remap(blk, n));
    else if (blk < attn_blocks) bwd_dkv_rows<DH, true>(a, smem, xcd_remap(blk - n, n));
    else if (FWD && (blk -= attn_blocks) < fwd_blocks) fwd_rows<DH, 64>(f, smem, xcd_remap(blk, fwd_blocks));
    else wgrad_small_block(w.grp, w.M, w.steps, blk - (FWD ? fwd_blocks : attn_blocks));
}

#define RES_BARRIER(n) do { asm volatile("" ::: "memory"); res_wait(n); __builtin_amdgcn_s_barrier(); asm volatile("" ::: "memory"); } while (0)

// ----------------------------------------------------------------------------------------
// backward, both passes in one workgroup per head (DH = 64 or 32, up to 256 tokens): Q, K, V and dO of the head are requested
// at once, tile by tile, and used as they land; every wavefront first runs pass 1 for its 32 query rows (dQ, delta), then, after one
// barrier, pass 2 for its 32 key rows (dK, dV) with the row statistics of pass 1 read from LDS.
// ----------------------------------------------------------------------------------------
template <int DH>
__global__ __launch_bounds__(512) void attn_bwd_fused(const bf16* __restrict__ qkv, const bf16* __restrict__ o,
                                                        const bf16* __restrict__ dout, const float* __restrict__ lse,
                                                        bf16* __restrict__ dqkv, float* __restrict__ delta,
                                                        const int* __restrict__ key_len, int T, int H) {
    constexpr int KS = DH / 16, DT = DH / 32, dh = DH, ROWB = 2 * DH;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tp = (T + 31) / 32 * 32;               // == 32 * wavefronts of the workgroup
    unsigned char* Ks0 = smem;
    unsigned char* Vs0 = Ks0 + tp * ROWB;
    unsigned char* Qs0 = Vs0 + tp * ROWB;
    unsigned char* Os0 = Qs0 + tp * ROWB;             // dO
    float* lse_s0 = reinterpret_cast<float*>(Os0 + tp * ROWB);
    float* del_s0 = lse_s0 + tp;
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 5;
    // two heads of 32 features share a cache line: neighbours go to one XCD's L2 (a stage of 49-token windows: 1886 -> 1869 us)
    const int bh = DH == 32 ? xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x, b = bh / H, h = bh % H;
    const int D = H * dh;
    const int64_t ld = 3 * (int64_t)D;
    const bf16* base = qkv + (int64_t)b * T * ld + h * dh;
    const bf16* dob = dout + (int64_t)b * T * D + h * dh;
    const bf16* ob = o + (int64_t)b * T * D + h * dh;
    const int r0 = wave * 32;                        // this wavefront's query rows (pass 1) and key rows (pass 2)
    const int q = r0 + (lane & 31), qc = min(q, T - 1);
    const float scale = rsqrtf((float)dh);
    const float c2 = scale * 1.4426950408889634f;
    const int Tk = key_len ? min(max(key_len[b], 1), T) : T;
    // ---- requests: owned rows of pass 1 to registers, then K and V (tile by tile), then Q and dO ----
    u32x4_t fq[KS], fdo[KS], fo[KS];
    res_load_owned<KS>(base, ld, r0, T, lane, fq);
    res_load_owned<KS>(dob, D, r0, T, lane, fdo);
    res_load_owned<KS>(ob, D, r0, T, lane, fo);
    float Lraw = res_load4(lse + (int64_t)bh * T + qc);
    int rem[4], nkv, nqo;
    res_request<DH>(Ks0, base + D, ld, Vs0, base + 2 * D, ld, Tk, tp, wave, nw, lane, rem, nkv);   // masked rows: the last valid one
    {
        int rem2[4];
        res_request<DH>(Qs0, base, ld, Os0, dob, D, T, tp, wave, nw, lane, rem2, nqo);
    }
    res_wait(min(nkv + nqo, 16));                    // the owned rows are older than every direct-to-LDS load
    res_pin(fq); res_pin(fdo); res_pin(fo); res_pin(Lraw);

    int rowoff[KS], o1[DT], o2[DT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rowoff[ks] = (lane & 31) * ROWB + (((2 * ks + g) ^ rsw<DH>(lane & 31)) << 4);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) res_tr_offsets<DH>(lane, dt, o1[dt], o2[dt]);

    // ---- pass 1: dQ, delta ----
    {
        bf16x8_t bq[KS], bdo[KS], bo[KS];
        res_frags<KS>(fq, bq); res_frags<KS>(fdo, bdo); res_frags<KS>(fo, bo);
        const float L2 = Lraw * 1.4426950408889634f;
        float dl = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int e = 0; e < 8; ++e) dl += (float)bdo[ks][e] * (float)bo[ks][e];
        dl += __shfl_xor(dl, 32, 64);
        if (g == 0) {
            if (q < T) delta[(int64_t)bh * T + q] = dl;
            // statistics for pass 2; +inf masks rows beyond the sequence (exp2(. - inf) = 0)
            lse_s0[q] = (q < T) ? L2 : INFINITY;
            del_s0[q] = (q < T) ? dl : 0.f;
        }

        f32x16_t accQ[DT];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) accQ[dt][v] = 0.f;

#pragma unroll
        for (int jt = 0; jt < 4; ++jt) {
            const int k0 = jt * 64;
            if (k0 < Tk) {
            RES_BARRIER(min(rem[jt] + nqo, 16));
            const unsigned char* Ks = Ks0 + k0 * ROWB;
            const unsigned char* Vs = Vs0 + k0 * ROWB;
            const int nt = (Tk - k0 > 32) ? 2 : 1;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (t < nt) {
                    f32x16_t aS, aP;
#pragma unroll
                    for (int v = 0; v < 16; ++v) { aS[v] = 0.f; aP[v] = 0.f; }
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        aS = mfma32(*reinterpret_cast<const bf16x8_t*>(Ks + t * 32 * ROWB + rowoff[ks]), bq[ks], aS);
                        aP = mfma32(*reinterpret_cast<const bf16x8_t*>(Vs + t * 32 * ROWB + rowoff[ks]), bdo[ks], aP);
                    }
                    float ds[16];
                    if (k0 + t * 32 + 32 <= Tk) {
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            ds[v] = __builtin_amdgcn_exp2f(aS[v] * c2 - L2) * (aP[v] - dl);
                    } else {
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const int key = k0 + t * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
                            ds[v] = (key < Tk) ? __builtin_amdgcn_exp2f(aS[v] * c2 - L2) * (aP[v] - dl) : 0.f;
                        }
                    }
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const bf16x8_t dsb = pack8(&ds[8 * c]);
#pragma unroll
                        for (int dt = 0; dt < DT; ++dt) {
                            const bf16x8_t a = res_tr_frag(Ks + (t * 32 + 16 * c) * ROWB, o1[dt], o2[dt]);
                            accQ[dt] = mfma32(a, dsb, accQ[dt]);
                        }
                    }
                }
            }
            }
        }
        if (q < T) {
            bf16* dq = dqkv + ((int64_t)b * T + q) * ld + h * dh;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) {
                    const int d = dt * 32 + 8 * v4 + 4 * g;
                    store4_bf16(dq + d, accQ[dt][4 * v4] * scale, accQ[dt][4 * v4 + 1] * scale,
                                accQ[dt][4 * v4 + 2] * scale, accQ[dt][4 * v4 + 3] * scale);
                }
        }
    }
    // ---- every load has landed, every wavefront has left its statistics ----
    RES_BARRIER(0);

    // ---- pass 2: dK, dV ----
    {
        bf16x8_t bk[KS], bv[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            bk[ks] = *reinterpret_cast<const bf16x8_t*>(Ks0 + r0 * ROWB + rowoff[ks]);
            bv[ks] = *reinterpret_cast<const bf16x8_t*>(Vs0 + r0 * ROWB + rowoff[ks]);
        }
        f32x16_t accK[DT], accV[DT];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) { accK[dt][v] = 0.f; accV[dt][v] = 0.f; }

        for (int i0 = 0; i0 < T; i0 += 64) {
            const unsigned char* Qs = Qs0 + i0 * ROWB;
            const unsigned char* Os = Os0 + i0 * ROWB;
            const float* lse_s = lse_s0 + i0;
            const float* del_s = del_s0 + i0;
            const int nt = (T - i0 > 32) ? 2 : 1;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (t < nt) {
                    f32x16_t aS, aP;
#pragma unroll
                    for (int v = 0; v < 16; ++v) { aS[v] = 0.f; aP[v] = 0.f; }
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        aS = mfma32(*reinterpret_cast<const bf16x8_t*>(Qs + t * 32 * ROWB + rowoff[ks]), bk[ks], aS);
                        aP = mfma32(*reinterpret_cast<const bf16x8_t*>(Os + t * 32 * ROWB + rowoff[ks]), bv[ks], aP);
                    }
                    float p[16], ds[16];
#pragma unroll
                    for (int v4 = 0; v4 < 4; ++v4) {
                        const int r = t * 32 + 8 * v4 + 4 * g;
                        const float4 Lr = *reinterpret_cast<const float4*>(lse_s + r);
                        const float4 Dr = *reinterpret_cast<const float4*>(del_s + r);
                        const float Lv[4] = {Lr.x, Lr.y, Lr.z, Lr.w};
                        const float Dv[4] = {Dr.x, Dr.y, Dr.z, Dr.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int v = 4 * v4 + e;
                            p[v] = __builtin_amdgcn_exp2f(aS[v] * c2 - Lv[e]);
                            ds[v] = p[v] * (aP[v] - Dv[e]);
                        }
                    }
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const bf16x8_t pb = pack8(&p[8 * c]);
                        const bf16x8_t dsb = pack8(&ds[8 * c]);
#pragma unroll
                        for (int dt = 0; dt < DT; ++dt) {
                            const bf16x8_t ao = res_tr_frag(Os + (t * 32 + 16 * c) * ROWB, o1[dt], o2[dt]);
                            accV[dt] = mfma32(ao, pb, accV[dt]);
                            const bf16x8_t aq = res_tr_frag(Qs + (t * 32 + 16 * c) * ROWB, o1[dt], o2[dt]);
                            accK[dt] = mfma32(aq, dsb, accK[dt]);
                        }
                    }
                }
            }
        }
        const int j = r0 + (lane & 31);
        if (j >= Tk) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int v = 0; v < 16; ++v) { accK[dt][v] = 0.f; accV[dt][v] = 0.f; }
        }
        if (j < T) {
            bf16* dk = dqkv + ((int64_t)b * T + j) * ld + D + h * dh;
            bf16* dv = dk + D;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) {
                    const int d = dt * 32 + 8 * v4 + 4 * g;
                    store4_bf16(dk + d, accK[dt][4 * v4] * scale, accK[dt][4 * v4 + 1] * scale,
                                accK[dt][4 * v4 + 2] * scale, accK[dt][4 * v4 + 3] * scale);
                    store4_bf16(dv + d, accV[dt][4 * v4], accV[dt][4 * v4 + 1], accV[dt][4 * v4 + 2], accV[dt][4 * v4 + 3]);
                }
        }
    }
}

// ---- launchers -------------------------------------------------------------------------------------------------------------
// Row tiles of a head are split evenly over workgroups of at most `most` wavefronts.
static void split_rows(int T, int most, int* nblk, int* nw) {
    const int tiles = (T + 31) / 32;
    *nblk = (tiles + most - 1) / most;
    *nw = (tiles + *nblk - 1) / *nblk;
}
// 64 bytes more than the tiles: the last transpose reads of 80-wide rows run past the row
template <typename Ring> static size_t ring_lds(int T) { return (size_t)(T > 64 ? 2 : 1) * Ring::SLOT + 64; }

template <int DH, int TR>
static int fwd_dma(hipStream_t s, const bf16* qkv, bf16* o, float* lse, int B, int T, int H, const int* key_len) {
    int nblk, nw;
    split_rows(T, 4, &nblk, &nw);
    const size_t lds = ring_lds<TileRing<DH, 2, 0, TR>>(T);
    hipLaunchKernelGGL((attn_fwd_dma<DH, TR>), dim3(nblk * B * H), dim3(nw * 64), lds, s, FwdArgs{qkv, o, lse, key_len, T, H, nblk});
    REV_HIP(hipGetLastError());
    return REV_OK;
}

// Which backward kernels a launch takes.  Measured (us; one workgroup per head, one launch per pass, both passes in one launch),
// features, tokens, heads, with the workgroups of the last:
//   64, 197:  64 (256) 19.2 21.5 13.1;  128 (512) 20.2 23.0 17.7;  192 (768) 21.4 29.0 24.4;  256 23.6 31.8 30.3;  768 68 75 97
//   64, 128:  128 (256) 12.3 16.4 10.3;  192 (384) 13.1 17.0 13.3;  256 (512) 14.7 18.4 14.7
//   32, 197:  128 (512) 14.8 15.3 11.7;  192 (768) 15.9 19.5 14.5;  256 (1024) 17.2 19.9 18.3
//   64, 512:  64 (512) - 38.5 29.2;  96 (768) - 45.8 42.3;  192 (1536) - 68.0 73.0
//   80, 1000: 32 (512) - 74.2 61.8;  48 (768) - 92.1 89.9;  64 (1024) - 101 106
//   80, 257:  64 (384) - 28.6 23.1;  128 (768) - 37.9 33.1;  384 (2304) - 87.4 84.7
// So heads of 64 features up to 256 tokens take the pair up to 128 heads (up to 64 tokens, one workgroup of two wavefronts a pass, up to
// 256), everything else up to 768 workgroups.  (96 to 128 tokens, 192 heads, with the pair 2 to 5 % slower.)
// Workgroups of two wavefronts instead of four as long as every CU gets at most one of them (12 heads of 197 tokens: 12.0
// against 12.3; 24 of 128, 64 features: 8.1 against 8.8; where a CU gets two, both use the same two SIMDs: 48 of 197, 14.5
// against 12.7).
static bool bwd_pair_pays(int heads, int T, int dh) {
    const int tiles = (T + 31) / 32;
    return dh == 64 && T <= 256 ? heads <= (tiles > 2 ? 128 : 256) : 2 * heads * ((tiles + 3) / 4) <= 768;
}
template <int DH>
static int bwd_dma(hipStream_t s, BwdArgs a, int B) {
    const int heads = B * a.H, tiles = (a.T + 31) / 32;
    int nw;
    const bool fits = DH <= 64 && a.T <= 256;
    if (bwd_pair_pays(heads, a.T, DH)) {
        split_rows(a.T, 2 * heads * ((tiles + 1) / 2) <= 256 ? 2 : 4, &a.nblk, &nw);
        a.delta = nullptr;
        const size_t lds = ring_lds<TileRing<DH, 3, 1>>(a.T) + nw * 128;
        hipLaunchKernelGGL(attn_bwd_pair_dma<DH>, dim3(2 * heads * a.nblk), dim3(nw * 64), lds, s, a);
        REV_HIP(hipGetLastError());
        return REV_OK;
    }
    if constexpr (DH <= 64) {
        if (fits) {
            const size_t lds = (size_t)tiles * 32 * (4 * 2 * DH + 8);
            static LdsLimit lim;
            if (int rc = lim.ensure(reinterpret_cast<const void*>(attn_bwd_fused<DH>), 160 * 1024)) return rc;
            hipLaunchKernelGGL(attn_bwd_fused<DH>, dim3(heads), dim3(tiles * 64), lds, s, a.qkv, a.o, a.dout, a.lse, a.dqkv, a.delta, a.key_len, a.T, a.H);
            REV_HIP(hipGetLastError());
            return REV_OK;
        }
    }
    split_rows(a.T, 4, &a.nblk, &nw);
    const size_t lds1 = ring_lds<TileRing<DH, 2, 0>>(a.T), lds2 = ring_lds<TileRing<DH, 2, 2>>(a.T);
    hipLaunchKernelGGL(attn_bwd_dq_dma<DH>, dim3(heads * a.nblk), dim3(nw * 64), lds1, s, a);
    hipLaunchKernelGGL(attn_bwd_dkv_dma<DH>, dim3(heads * a.nblk), dim3(nw * 64), lds2, s, a);
    REV_HIP(hipGetLastError());
    return REV_OK;
}

// with weight gradients: workgroups of four wavefronts, as theirs
template <int DH>
static int bwd_wgrad_dma(hipStream_t s, BwdArgs a, int B, const WgradTail& w, const AttnFwdCall<bf16>* beside) {
    const int heads = B * a.H;
    a.nblk = ((a.T + 31) / 32 + 3) / 4;
    const int lds = std::max((int)(ring_lds<TileRing<DH, 3, 1>>(a.T) + 4 * 128), 2 * WD_STAGE), attn_blocks = 2 * heads * a.nblk;
    static_assert(2 * TileRing<DH, 2, 0, 64>::SLOT + 64 <= 2 * WD_STAGE, "the forward's ring");
    auto go = [&](auto kern, const FwdArgs& f, int fwd_blocks, LdsLimit& lim) -> int {
        if (int rc = lim.ensure(reinterpret_cast<const void*>(kern), 2 * WD_STAGE)) return rc;
        hipLaunchKernelGGL(kern, dim3(attn_blocks + fwd_blocks + w.grp.tile_blocks), dim3(256), lds, s, a, w, attn_blocks, f, fwd_blocks);
        REV_HIP(hipGetLastError());
        return REV_OK;
    };
    static LdsLimit lim, lim_fwd;
    if (!beside) return go(attn_bwd_pair_wgrad<DH, false>, FwdArgs{}, 0, lim);
    return go(attn_bwd_pair_wgrad<DH, true>, FwdArgs{beside->qkv, beside->o, beside->lse, a.key_len, a.T, a.H, a.nblk}, heads * a.nblk, lim_fwd);
}
bool attention_takes_wgrad(int B, int T, int H, int dh) { return attention_dma_takes(dh) && bwd_pair_pays(B * H, T, dh); }
int attention_backward_wgrad(hipStream_t s, const bf16* qkv, const bf16* o, const bf16* dout, const float* lse, bf16* dqkv, int B, int T,
                             int H, int dh, const int* key_len, const WgradItem* items, int count, const AttnFwdCall<bf16>* beside) {
    const BwdArgs a = {qkv, o, dout, lse, dqkv, nullptr, key_len, T, H, 0};
    WgradTail w;
    double flops = (beside ? 12.0 : 8.0) * B * H * (double)T * T * dh;
    if (int rc = gemm_wgrad_bf16_beside(items, count, B * T, &w, &flops)) return rc;
    ProfScope ps(K_MIXED, s, flops);
    if (dh == 32) return bwd_wgrad_dma<32>(s, a, B, w, beside);
    if (dh == 64) return bwd_wgrad_dma<64>(s, a, B, w, beside);
    return bwd_wgrad_dma<80>(s, a, B, w, beside);
}

bool attention_dma_takes(int dh) { return dh == 32 || dh == 64 || dh == 80; }
int attention_forward_dma(hipStream_t s, const bf16* qkv, bf16* o, float* lse, int B, int T, int H, int dh, const int* key_len) {
    // Tiles of 32 rows hold half the LDS, so twice as many one-wavefront workgroups share a CU.  64 rows / 32, us: 64 features, T = 1, 6144
    // heads 11.5 / 8.5, 49152 69 / 47; T = 16, 3072 heads 8.9 / 7.6, 6144 13.8 / 12.4; but where the rows come from HBM more of
    // them in flight are slower: T = 16, 49152 heads 108 / 115; T = 24, 12288 heads 41.7 / 46.0; T = 32, 6144 heads 28.4 / 30.7.
    const bool half = T <= 8 || (T <= 16 && (int64_t)B * H * T <= 131072);
#define FWD(DH) return half ? fwd_dma<DH, 32>(s, qkv, o, lse, B, T, H, key_len) : fwd_dma<DH, 64>(s, qkv, o, lse, B, T, H, key_len)
    if (dh == 32) FWD(32);
    if (dh == 64) FWD(64);
    FWD(80);
#undef FWD
}
int attention_backward_dma(hipStream_t s, const bf16* qkv, const bf16* o, const bf16* dout, const float* lse, bf16* dqkv, float* delta,
                           int B, int T, int H, int dh, const int* key_len) {
    const BwdArgs a = {qkv, o, dout, lse, dqkv, delta, key_len, T, H, 0};
    if (dh == 32) return bwd_dma<32>(s, a, B);
    if (dh == 64) return bwd_dma<64>(s, a, B);
    return bwd_dma<80>(s, a, B);
}

}  // namespace rev
