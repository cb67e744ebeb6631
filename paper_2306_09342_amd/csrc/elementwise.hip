// Memory-bound kernels: LayerNorm forward / backward, column sums, fixed-order
// reductions, dtype conversion.  One wavefront (64 lanes) owns one
// row at a time and keeps it in registers; row statistics are wavefront
// reductions; column statistics (d gamma, d beta, bias gradients) are summed in
// a fixed order so that results do not depend on scheduling.
#include "common.h"
#include "rowwise.h"
#include "sums.h"

namespace rev {

// A chunk's products, with the rounding spelled out: left to the compiler, which products it fuses into the sums behind them changes
// from kernel to kernel, and a row must have the same bits in all of them.
__device__ __forceinline__ f4 mul4(const f4& a, const f4& b) {
#pragma clang fp contract(off)
    return {a.x * b.x, a.y * b.y, a.z * b.z, a.w * b.w};
}
__device__ __forceinline__ float dot4(const f4& a, const f4& b) { return fmaf(a.x, b.x, a.y * b.y) + fmaf(a.z, b.z, a.w * b.w); }

// ---- LayerNorm forward -----------------------------------------------------------
// LPR lanes hold a row: lane l of them the 4-element chunks l, l + LPR, ... (MAXJ of them).  Rows of up to 256 floats share a
// wavefront (pick_row), wider ones have it to themselves.  Every lane handles two rows, half of all rows apart and both
// requested before either is reduced, so it has two independent memory round trips in flight.  Bound by HBM.  200704 rows
// of 96: 49 us with a wavefront per row (24 of 64 lanes at work), now 28; 100000 rows of 64: 22 -> 9.6.
template <typename TA, typename TP, int LPR, int MAXJ>
__device__ __forceinline__ void ln_fwd_rows(const float* __restrict__ x, const TP* __restrict__ g, const TP* __restrict__ b, float eps,
                                            TA* __restrict__ y, float* __restrict__ stats, int M, int D, int thread) {
    const int lane = thread & (LPR - 1);
    const int half = (M + 1) >> 1;
    const int r0 = thread / LPR;                                   // rows r0 and r0 + half
    if (r0 >= half) return;
    const int nch = D >> 2;
    int rows[2] = {r0, r0 + half};
    const bool live1 = rows[1] < M;
    f4 v[2][MAXJ];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const float* xr = x + (int64_t)rows[k] * D;
        if (k == 1 && !live1) break;
#pragma unroll
        for (int j = 0; j < MAXJ; ++j) {
            int c = lane + LPR * j;
            if (c < nch) v[k][j] = load4(xr + 4 * c);
        }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (k == 1 && !live1) break;
        float s[MAXJ], q[MAXJ];
#pragma unroll
        for (int j = 0; j < MAXJ; ++j) {
            int c = lane + LPR * j;
            s[j] = c < nch ? (v[k][j].x + v[k][j].y) + (v[k][j].z + v[k][j].w) : 0.f;
        }
        const float mean = row_sum<LPR, MAXJ>(s) / (float)D;
#pragma unroll
        for (int j = 0; j < MAXJ; ++j) {
            int c = lane + LPR * j;
            const f4 a = {v[k][j].x - mean, v[k][j].y - mean, v[k][j].z - mean, v[k][j].w - mean};
            const float d = dot4(a, a);
            q[j] = c < nch ? d : 0.f;
        }
        const float rstd = 1.0f / sqrtf(row_sum<LPR, MAXJ>(q) / (float)D + eps);
        TA* yr = y + (int64_t)rows[k] * D;
#pragma unroll
        for (int j = 0; j < MAXJ; ++j) {
            int c = lane + LPR * j;
            if (c < nch) {
                f4 gg = load4(g + 4 * c), bb = load4(b + 4 * c), o;
                o.x = (v[k][j].x - mean) * rstd * gg.x + bb.x;
                o.y = (v[k][j].y - mean) * rstd * gg.y + bb.y;
                o.z = (v[k][j].z - mean) * rstd * gg.z + bb.z;
                o.w = (v[k][j].w - mean) * rstd * gg.w + bb.w;
                store4(yr + 4 * c, o);
            }
        }
        if (lane == 0) {
            stats[2 * (int64_t)rows[k]] = mean;
            stats[2 * (int64_t)rows[k] + 1] = rstd;
        }
    }
}

template <typename TA, typename TP, int LPR, int MAXJ>
__global__ __launch_bounds__(256) void ln_fwd_kernel(const float* __restrict__ x, const TP* __restrict__ g,
                                                     const TP* __restrict__ b, float eps,
                                                     TA* __restrict__ y, float* __restrict__ stats,
                                                     int M, int D) {
    ln_fwd_rows<TA, TP, LPR, MAXJ>(x, g, b, eps, y, stats, M, D, blockIdx.x * 256 + threadIdx.x);
}

template <typename TA, typename TP>
int ln_forward(hipStream_t s, const float* x, const TP* g, const TP* b, float eps,
               TA* y, float* stats, int M, int D) {
    ProfScope ps(K_LN_FWD, s, (double)M * D * (4 + sizeof(TA)));
    const RowSplit rs = pick_row(D, M >= 16384);       // shared wavefronts only where there are enough of them
    dim3 grid((unsigned)(((int64_t)((M + 1) / 2) * rs.lpr + 255) / 256)), block(256);
#define CASE(L, J) if (rs.lpr == L && rs.maxj == J) { hipLaunchKernelGGL((ln_fwd_kernel<TA, TP, L, J>), grid, block, 0, s, x, g, b, eps, y, stats, M, D); } else
    ROW_SPLITS_WIDE(CASE) ROW_SPLITS_8(CASE) ROW_SPLITS_FWD(CASE) { set_error("ln_forward: d_model too large"); return REV_EINVAL; }
#undef CASE
    REV_HIP(hipGetLastError());
    return REV_OK;
}
template int ln_forward<float, float>(hipStream_t, const float*, const float*, const float*, float, float*, float*, int, int);
template int ln_forward<bf16, bf16>(hipStream_t, const float*, const bf16*, const bf16*, float, bf16*, float*, int, int);

// ---- LayerNorm backward + residual-gradient add -----------------------------------------
// out = r + rstd * (dxh - mean(dxh) - xhat * mean(dxh * xhat)),  dxh = dn * g.
// Each block walks LNB_ROWS consecutive rows (4 wavefronts, one row each at a
// time); per-lane column accumulators for d gamma, d beta and the column sums of
// `out` itself (the bias gradient of the linear map that `out` is the cotangent
// of) are folded across the 4 wavefronts in LDS in wavefront order and written
// as one partial row [dgamma | dbeta | colsum(out)] per block.
constexpr int LNB_ROWS = 32;
// Rows per block (a multiple of 4): LNB_ROWS for 32 k rows and more; fewer, down to 8, for shorter
// inputs so that about 1024 blocks (4 per CU) are in flight; more once LNB_ROWS would give above 2048
// partial rows, and for rows of 772 to 2048 floats (2 to 4 blocks share a CU) where that makes one round of blocks: 8224 rows
// of 1280 45.8 -> 41.4 us, 16384 of 1024 54 -> 43.
// Rows of up to 64 floats, and of up to 96 in 100 000 rows and more, share a wavefront (8 lanes each), 32 of a block at a time; beyond,
// the registers of three and more chunks per lane leave too few wavefronts in flight.  A wavefront per row / shared, us: 64
// floats, 8200 rows 5.9 / 5.4, 65 536 19 / 17, 200 704 65 / 44; 96 floats, 8200 6.3 / 7.6, 65 536 27 / 30, 100 000 40 / 38, 200 704
// 75 / 68; 128 floats, 8200 6.4 / 9.8, 65 536 31 / 42, 200 704 88 / 94; rows of 160 to 256 floats, four to a wavefront: 50 176 of
// 192 28 / 31.
static bool ln_bwd_shares(int M, int D) { return M > 8192 && (D <= 64 || (D <= 96 && M >= 100000)); }
static int ln_bwd_rows_per_block(int M, int D) {
    int rpb = LNB_ROWS;
    if ((M + rpb - 1) / rpb > 2048) rpb = (((M + 2047) / 2048) + 3) / 4 * 4;
    else if (M < 1024 * LNB_ROWS) rpb = ((M + 1023) / 1024 + 3) / 4 * 4;
    if (rpb < 8) rpb = 8;
    if (rpb > 8 && D > 768 && D <= 2048) {                          // accumulators in LDS: a second, short round costs a whole one
        const int slots = 256 * (160 * 1024 / (48 * D)), one_round = ((M + slots - 1) / slots + 3) / 4 * 4;
        if (one_round > rpb && one_round <= LNB_ROWS) rpb = one_round;
    }
    if (ln_bwd_shares(M, D)) rpb = (rpb + 31) / 32 * 32;
    return rpb;
}

// Rows of 1024 floats and more (4+ register chunks per lane): the three column accumulators of a
// wavefront live in its own slice of LDS instead of registers (lane-private slots, no synchronisation),
// which roughly halves the register count and doubles the wavefronts in flight.
template <int LPR, int MAXJ> struct LnBwdCfg { static constexpr bool ACC_LDS = (LPR == 64 && MAXJ >= 4 && MAXJ <= 8); };

template <typename TA, typename TP, int LPR, int MAXJ>
__global__ __launch_bounds__(256) void ln_bwd_kernel(const TA* __restrict__ dn, const float* __restrict__ x,
                                                     const float* __restrict__ stats, const TP* __restrict__ g,
                                                     const float* __restrict__ r, float* __restrict__ out,
                                                     TA* __restrict__ outb, float* __restrict__ partial,
                                                     int M, int D, int rows_per_block) {
    constexpr bool ACC_LDS = LnBwdCfg<LPR, MAXJ>::ACC_LDS;
    constexpr int G = 64 / LPR;                                  // rows of a wavefront at a time
    extern __shared__ float lds[];   // [3 * D], or [4][3 * D] with ACC_LDS
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & (LPR - 1), grp = (threadIdx.x & 63) / LPR;
    const int nch = D >> 2;
    constexpr int NACC = ACC_LDS ? 1 : MAXJ;
    // The chunks' sums: added as they come, or kept apart, whichever is faster (1280 floats, 50176 rows: 238 / 252 us;
    // 2048 floats, 8192 rows: 101 / 94).  The order is the same.
    constexpr int NP = MAXJ >= 4 && MAXJ < 8 ? 1 : MAXJ;
    f4 ag[NACC], ab[NACC], ao[NACC], gg[MAXJ];
    float* wacc = lds + (ACC_LDS ? wave * 3 * D : 0);            // [dgamma | dbeta | colsum(out)] of this wavefront
#pragma unroll
    for (int j = 0; j < MAXJ; ++j) {
        int c = lane + LPR * j;
        gg[j] = (c < nch) ? load4(g + 4 * c) : f4{0.f, 0.f, 0.f, 0.f};
        if (ACC_LDS) {
            if (c < nch) {
                const f4 z = {0.f, 0.f, 0.f, 0.f};
                *reinterpret_cast<f4*>(wacc + 4 * c) = z;
                *reinterpret_cast<f4*>(wacc + D + 4 * c) = z;
                *reinterpret_cast<f4*>(wacc + 2 * D + 4 * c) = z;
            }
        } else {
            ag[j % NACC] = {0.f, 0.f, 0.f, 0.f};
            ab[j % NACC] = {0.f, 0.f, 0.f, 0.f};
            ao[j % NACC] = {0.f, 0.f, 0.f, 0.f};
        }
    }
    const int row0 = blockIdx.x * rows_per_block;
    const int row1 = min(M, row0 + rows_per_block);
    for (int row = row0 + wave * G + grp; row < row1; row += 4 * G) {
        const float mean = stats[2 * (int64_t)row], rstd = stats[2 * (int64_t)row + 1];
        const int64_t base = (int64_t)row * D;
        f4 xh[MAXJ], dh[MAXJ], rv[MAXJ];
        float p1[NP] = {}, p2[NP] = {};
        // all three input rows are requested up front: one memory round trip per row, not two
#pragma unroll
        for (int j = 0; j < MAXJ; ++j) {
            int c = lane + LPR * j;
            if (c < nch) rv[j] = load4(r + base + 4 * c);
        }
#pragma unroll
        for (int j = 0; j < MAXJ; ++j) {
            int c = lane + LPR * j;
            if (c < nch) {
                f4 xv = load4(x + base + 4 * c), d = load4(dn + base + 4 * c);
                xh[j] = {(xv.x - mean) * rstd, (xv.y - mean) * rstd, (xv.z - mean) * rstd, (xv.w - mean) * rstd};
                if (ACC_LDS) {
                    f4 b0 = *reinterpret_cast<f4*>(wacc + D + 4 * c), g0 = *reinterpret_cast<f4*>(wacc + 4 * c);
                    b0.x += d.x; b0.y += d.y; b0.z += d.z; b0.w += d.w;
                    g0.x += d.x * xh[j].x; g0.y += d.y * xh[j].y; g0.z += d.z * xh[j].z; g0.w += d.w * xh[j].w;
                    *reinterpret_cast<f4*>(wacc + D + 4 * c) = b0;
                    *reinterpret_cast<f4*>(wacc + 4 * c) = g0;
                } else {
                    ab[j % NACC].x += d.x; ab[j % NACC].y += d.y; ab[j % NACC].z += d.z; ab[j % NACC].w += d.w;
                    ag[j % NACC].x += d.x * xh[j].x; ag[j % NACC].y += d.y * xh[j].y;
                    ag[j % NACC].z += d.z * xh[j].z; ag[j % NACC].w += d.w * xh[j].w;
                }
                dh[j] = mul4(d, gg[j]);
                const float s1 = dot4(d, gg[j]);
                const float s2 = dot4(dh[j], xh[j]);
                p1[j % NP] = NP == 1 ? p1[0] + s1 : s1;
                p2[j % NP] = NP == 1 ? p2[0] + s2 : s2;
            }
        }
        const float c1 = row_sum<LPR, NP>(p1) / (float)D, c2 = row_sum<LPR, NP>(p2) / (float)D;
#pragma unroll
        for (int j = 0; j < MAXJ; ++j) {
            int c = lane + LPR * j;
            if (c < nch) {
                f4 o;
                o.x = rv[j].x + rstd * (dh[j].x - c1 - xh[j].x * c2);
                o.y = rv[j].y + rstd * (dh[j].y - c1 - xh[j].y * c2);
                o.z = rv[j].z + rstd * (dh[j].z - c1 - xh[j].z * c2);
                o.w = rv[j].w + rstd * (dh[j].w - c1 - xh[j].w * c2);
                if (ACC_LDS) {
                    f4 o0 = *reinterpret_cast<f4*>(wacc + 2 * D + 4 * c);
                    o0.x += o.x; o0.y += o.y; o0.z += o.z; o0.w += o.w;
                    *reinterpret_cast<f4*>(wacc + 2 * D + 4 * c) = o0;
                } else {
                    ao[j % NACC].x += o.x; ao[j % NACC].y += o.y; ao[j % NACC].z += o.z; ao[j % NACC].w += o.w;
                }
                store4(out + base + 4 * c, o);
                if (outb) store4(outb + base + 4 * c, o);
            }
        }
    }
    float* prow = partial + (int64_t)blockIdx.x * 3 * D;
    if (ACC_LDS) {
        // fold the 4 wavefronts' slices in wavefront order
        __syncthreads();
        for (int i = threadIdx.x; i < 3 * D; i += 256)
            prow[i] = ((lds[i] + lds[3 * D + i]) + lds[6 * D + i]) + lds[9 * D + i];
        return;
    }
    // the rows that shared the wavefront, by halves
    if constexpr (G > 1) {
#pragma unroll
        for (int j = 0; j < NACC; ++j)
#pragma unroll
            for (int off = 32; off >= LPR; off >>= 1) {
                auto fold = [&](f4& v) {
                    v.x += __shfl_xor(v.x, off, 64); v.y += __shfl_xor(v.y, off, 64);
                    v.z += __shfl_xor(v.z, off, 64); v.w += __shfl_xor(v.w, off, 64);
                };
                fold(ag[j]); fold(ab[j]); fold(ao[j]);
            }
    }
    // fold the 4 wavefronts' column accumulators in wavefront order
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int j = 0; j < MAXJ; ++j) {
                int c = lane + LPR * j;
                if (c < nch && grp == 0) {
                    float* pg = lds + 4 * c;
                    float* pb = lds + D + 4 * c;
                    float* po = lds + 2 * D + 4 * c;
                    if (w == 0) {
                        pg[0] = ag[j % NACC].x; pg[1] = ag[j % NACC].y; pg[2] = ag[j % NACC].z; pg[3] = ag[j % NACC].w;
                        pb[0] = ab[j % NACC].x; pb[1] = ab[j % NACC].y; pb[2] = ab[j % NACC].z; pb[3] = ab[j % NACC].w;
                        po[0] = ao[j % NACC].x; po[1] = ao[j % NACC].y; po[2] = ao[j % NACC].z; po[3] = ao[j % NACC].w;
                    } else {
                        pg[0] += ag[j % NACC].x; pg[1] += ag[j % NACC].y; pg[2] += ag[j % NACC].z; pg[3] += ag[j % NACC].w;
                        pb[0] += ab[j % NACC].x; pb[1] += ab[j % NACC].y; pb[2] += ab[j % NACC].z; pb[3] += ab[j % NACC].w;
                        po[0] += ao[j % NACC].x; po[1] += ao[j % NACC].y; po[2] += ao[j % NACC].z; po[3] += ao[j % NACC].w;
                    }
                }
            }
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < 3 * D; i += 256) prow[i] = lds[i];
}

// The same for short inputs (up to 8192 rows of up to 1280 floats): a row per wavefront, 8 in a block, which leave their
// contributions to the column sums in LDS at once.  A chain of one memory round trip, one barrier and the stores; the kernel above
// takes its rows in turn and adds its wavefronts one after the other.  The kernel above / here, us: 197 rows of 768 6.7 / 3.8; 1000
// of 640 7.4 / 4.4; 4096 of 768 13.0 / 10.6; 8192 of 640 18.9 / 18.2, of 768 23.1 / 23.3, of 1280 43.3 / 39.8.  Rows of 852 to 1024
// floats, of which one block here but three or four above fit a CU, only in one round of blocks (2048 rows): 1024 floats,
// 2000 rows 10.8 / 8.5, 4096 15.2 / 15.7, 6144 24.2 / 25.4, 8192 33.1 / 34.0.
constexpr int LNB_SMALL_MAXD = 1280;
template <typename TA, typename TP, int MAXJ>
__device__ __forceinline__ void ln_bwd_small_rows(const TA* __restrict__ dn, const float* __restrict__ x, const float* __restrict__ stats,
                                                  const TP* __restrict__ g, const float* __restrict__ r, float* __restrict__ out,
                                                  TA* __restrict__ outb, float* __restrict__ partial, int M, int D, int block) {
    extern __shared__ float lds[];   // [8][3 * D]
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nch = D >> 2;
    const int row = block * 8 + wave;
    float* slot = lds + wave * 3 * D;
    const f4 z = {0.f, 0.f, 0.f, 0.f};
    if (row < M) {
        const int64_t base = (int64_t)row * D;
        f4 xv[MAXJ], d[MAXJ], rv[MAXJ], gg[MAXJ];
#pragma unroll
        for (int j = 0; j < MAXJ; ++j) {
            const int c = lane + 64 * j;
            xv[j] = d[j] = rv[j] = gg[j] = z;
            if (c < nch) { xv[j] = load4(x + base + 4 * c); d[j] = load4(dn + base + 4 * c); gg[j] = load4(g + 4 * c); rv[j] = load4(r + base + 4 * c); }
        }
        const float mean = stats[2 * (int64_t)row], rstd = stats[2 * (int64_t)row + 1];
        float c1 = 0.f, c2 = 0.f;
#pragma unroll
        for (int j = 0; j < MAXJ; ++j) {
            const int c = lane + 64 * j;
            xv[j] = {(xv[j].x - mean) * rstd, (xv[j].y - mean) * rstd, (xv[j].z - mean) * rstd, (xv[j].w - mean) * rstd};
            const f4 h = mul4(d[j], gg[j]);
            c1 += dot4(d[j], gg[j]);
            c2 += dot4(h, xv[j]);
            if (c < nch) {
                store4(slot + 4 * c, f4{d[j].x * xv[j].x, d[j].y * xv[j].y, d[j].z * xv[j].z, d[j].w * xv[j].w});
                store4(slot + D + 4 * c, d[j]);
            }
            d[j] = h;
        }
        c1 = wave_sum(c1) / (float)D;
        c2 = wave_sum(c2) / (float)D;
#pragma unroll
        for (int j = 0; j < MAXJ; ++j) {
            const int c = lane + 64 * j;
            if (c < nch) {
                f4 o;
                o.x = rv[j].x + rstd * (d[j].x - c1 - xv[j].x * c2);
                o.y = rv[j].y + rstd * (d[j].y - c1 - xv[j].y * c2);
                o.z = rv[j].z + rstd * (d[j].z - c1 - xv[j].z * c2);
                o.w = rv[j].w + rstd * (d[j].w - c1 - xv[j].w * c2);
                store4(slot + 2 * D + 4 * c, o);
                store4(out + base + 4 * c, o);
                if (outb) store4(outb + base + 4 * c, o);
            }
        }
    } else {
        for (int c = lane; c < 3 * nch; c += 64) store4(slot + 4 * c, z);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < 3 * nch; c += 512) {
        f4 s = z;
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const f4 v = load4(lds + w * 3 * D + 4 * c);
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
        store4(partial + (int64_t)block * 3 * D + 4 * c, s);
    }
}
template <typename TA, typename TP, int MAXJ>
__global__ __launch_bounds__(512) void ln_bwd_small_kernel(const TA* __restrict__ dn, const float* __restrict__ x,
                                                           const float* __restrict__ stats, const TP* __restrict__ g,
                                                           const float* __restrict__ r, float* __restrict__ out,
                                                           TA* __restrict__ outb, float* __restrict__ partial, int M, int D) {
    ln_bwd_small_rows<TA, TP, MAXJ>(dn, x, stats, g, r, out, outb, partial, M, D, blockIdx.x);
}
// It and, in the workgroups behind its own, the LayerNorm forward of other rows of the same width: the two chains of a small stack
// side by side (rev_stack.hip).  197 rows of 768: 4.6 and 4.5 us by themselves, 4.8 together.
template <typename TA, typename TP, int MAXJ>
__global__ __launch_bounds__(512) void ln_pair_kernel(LnBwdCall<TA, TP> b, LnFwdCall<TA, TP> f, int M, int D, int bwd_blocks) {
    if ((int)blockIdx.x < bwd_blocks) ln_bwd_small_rows<TA, TP, MAXJ>(b.dn, b.x, b.stats, b.g, b.r, b.out, b.outb, b.partial, M, D, blockIdx.x);
    else ln_fwd_rows<TA, TP, 64, MAXJ>(f.x, f.g, f.b, f.eps, f.y, f.stats, M, D, (blockIdx.x - bwd_blocks) * 512 + threadIdx.x);
}

// ---- several fixed-order reductions in one launch ----------------------------------------------------
__global__ __launch_bounds__(256) void reduce_multi_kernel(RedArgs a) {
    __shared__ float4 sh[256];
    reduce_block(a, blockIdx.x, sh);
}

int reduce_multi(hipStream_t s, const RedSeg* segs, int nseg) {
    if (nseg <= 0) return REV_OK;
    RedArgs a;
    double bytes = 0;
    const int blocks = reduce_args(segs, nseg, &a, &bytes);
    if (blocks < 0) return blocks;
    ProfScope ps(K_REDUCE, s, bytes);
    hipLaunchKernelGGL(reduce_multi_kernel, dim3(blocks), dim3(256), 0, s, a);
    REV_HIP(hipGetLastError());
    return REV_OK;
}

int64_t ln_bwd_partial_elems(int M, int D) {
    const int rpb = ln_bwd_rows_per_block(M, D);
    return (int64_t)((M + rpb - 1) / rpb) * 3 * D;
}

static bool ln_bwd_small(int M, int D) {
    return ln_bwd_rows_per_block(M, D) == 8 && D <= LNB_SMALL_MAXD && !(M > 2048 && D > 848 && D <= 1024);
}
template <typename TA, typename TP>
int ln_backward(hipStream_t s, const TA* dn, const float* x, const float* stats, const TP* g,
                const float* r, float* out, TA* outb, float* dgb, float* dbias,
                float* partial, int M, int D, RedSeg* defer) {
    const int rpb = ln_bwd_rows_per_block(M, D);
    const int nblk = (M + rpb - 1) / rpb;
    {
        ProfScope ps(K_LN_BWD, s, (double)M * D * (sizeof(TA) + 4 + 4 + 4 + (outb ? sizeof(TA) : 0)));
        dim3 grid(nblk), block(256);
        const bool small = ln_bwd_small(M, D);
        const RowSplit rs = pick_row(D, ln_bwd_shares(M, D));
#define SMALL(J) if (rs.maxj == J) {                                                                                   \
            auto kern = ln_bwd_small_kernel<TA, TP, J>;                                                                 \
            static LdsLimit lim;                                                                                        \
            if (int rc = lim.ensure(reinterpret_cast<const void*>(kern), 96 * LNB_SMALL_MAXD)) return rc;               \
            hipLaunchKernelGGL(kern, grid, dim3(512), (size_t)96 * D, s, dn, x, stats, g, r, out, outb, partial, M, D); \
        }
#define CASE(L, J) if (rs.lpr == L && rs.maxj == J) {                                                                  \
            auto kern = ln_bwd_kernel<TA, TP, L, J>;                                                                    \
            constexpr int copies = LnBwdCfg<L, J>::ACC_LDS ? 4 : 1;                                                     \
            const size_t shmem = (size_t)copies * 3 * D * sizeof(float);                                                \
            static LdsLimit lim;                                                                                        \
            if (int rc = lim.ensure(reinterpret_cast<const void*>(kern), copies * 3 * L * J * 16)) return rc;           \
            hipLaunchKernelGGL(kern, grid, block, shmem, s, dn, x, stats, g, r, out, outb, partial, M, D, rpb);         \
        } else
        if (small) { SMALL(2) SMALL(3) SMALL(4) SMALL(5) } else
        ROW_SPLITS_WIDE(CASE) ROW_SPLITS_8(CASE) { set_error("ln_backward: d_model too large"); return REV_EINVAL; }
#undef CASE
#undef SMALL
        REV_HIP(hipGetLastError());
    }
    // partial rows are [dgamma(D) | dbeta(D) | colsum(out)(D)]; gamma and beta gradients are adjacent in dgb
    const RedSeg seg = {partial, dgb, dbias, 3 * (int64_t)D, 3 * (int64_t)D, 2 * (int64_t)D, nblk};
    if (defer) { *defer = seg; return REV_OK; }
    return reduce_multi(s, &seg, 1);
}
template int ln_backward<float, float>(hipStream_t, const float*, const float*, const float*, const float*, const float*, float*, float*, float*, float*, float*, int, int, RedSeg*);
template int ln_backward<bf16, bf16>(hipStream_t, const bf16*, const float*, const float*, const bf16*, const float*, float*, bf16*, float*, float*, float*, int, int, RedSeg*);

template <typename TA, typename TP>
int ln_pair(hipStream_t s, const LnBwdCall<TA, TP>& b, const LnFwdCall<TA, TP>& f, int M, int D, RedSeg* defer) {
    if (!ln_bwd_small(M, D)) {
        if (int rc = ln_backward<TA, TP>(s, b.dn, b.x, b.stats, b.g, b.r, b.out, b.outb, b.dgb, b.dbias, b.partial, M, D, defer)) return rc;
        return ln_forward<TA, TP>(s, f.x, f.g, f.b, f.eps, f.y, f.stats, M, D);
    }
    const int nblk = (M + 7) / 8;
    ProfScope ps(K_LN_PAIR, s, (double)M * D * (16 + sizeof(TA) * (b.outb ? 3 : 2)));
    const dim3 grid(nblk + ((M + 1) / 2 + 7) / 8), block(512);
    switch (pick_maxj(D)) {
#define CASE(J) case J: {                                                                                              \
            auto kern = ln_pair_kernel<TA, TP, J>;                                                                      \
            static LdsLimit lim;                                                                                        \
            if (int rc = lim.ensure(reinterpret_cast<const void*>(kern), 96 * LNB_SMALL_MAXD)) return rc;               \
            hipLaunchKernelGGL(kern, grid, block, (size_t)96 * D, s, b, f, M, D, nblk);                                 \
            break; }
        CASE(2) CASE(3) CASE(4) CASE(5)
#undef CASE
        default: set_error("ln_pair: d_model too large"); return REV_EINVAL;
    }
    REV_HIP(hipGetLastError());
    *defer = {b.partial, b.dgb, b.dbias, 3 * (int64_t)D, 3 * (int64_t)D, 2 * (int64_t)D, nblk};
    return REV_OK;
}
template int ln_pair<float, float>(hipStream_t, const LnBwdCall<float, float>&, const LnFwdCall<float, float>&, int, int, RedSeg*);
template int ln_pair<bf16, bf16>(hipStream_t, const LnBwdCall<bf16, bf16>&, const LnFwdCall<bf16, bf16>&, int, int, RedSeg*);

// ---- column sums (bias gradients) --------------------------------------------------------
// grid (column tiles of 256, row chunks); each wavefront sums a quarter of the
// block's rows for its 256 columns, the 4 wavefronts are folded in order.
template <typename T>
__global__ __launch_bounds__(256) void colsum_kernel(const T* __restrict__ in, int64_t ld, int M, int N,
                                                     int rows_per_block, float* __restrict__ partial) {
    __shared__ float lds[4][256];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int col = blockIdx.x * 256 + lane * 4;
    const int row0 = blockIdx.y * rows_per_block;
    const int row1 = min(M, row0 + rows_per_block);
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    if (col < N) {
        for (int row = row0 + wave; row < row1; row += 4) {
            f4 v = load4(in + (int64_t)row * ld + col);
            acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
        }
    }
    lds[wave][lane * 4 + 0] = acc.x; lds[wave][lane * 4 + 1] = acc.y;
    lds[wave][lane * 4 + 2] = acc.z; lds[wave][lane * 4 + 3] = acc.w;
    __syncthreads();
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c < N) {
        float v = ((lds[0][threadIdx.x] + lds[1][threadIdx.x]) + lds[2][threadIdx.x]) + lds[3][threadIdx.x];
        partial[(int64_t)blockIdx.y * N + c] = v;
    }
}

static int colsum_chunks(int M, int N) {
    int tiles = (N + 255) / 256;
    int P = (2048 + tiles - 1) / tiles;
    int maxP = (M + 15) / 16;
    if (P > maxP) P = maxP;
    if (P < 1) P = 1;
    return P;
}
int64_t colsum_partial_elems(int M, int N) { return (int64_t)colsum_chunks(M, N) * N; }

template <typename T>
int colsum(hipStream_t s, const T* in, int64_t ld, int M, int N, float* out, float* partial, RedSeg* defer) {
    int P = colsum_chunks(M, N);
    int rpb = (M + P - 1) / P;
    P = (M + rpb - 1) / rpb;
    {
        ProfScope ps(K_COLSUM, s, (double)M * N * sizeof(T));
        dim3 grid((N + 255) / 256, P), block(256);
        hipLaunchKernelGGL((colsum_kernel<T>), grid, block, 0, s, in, ld, M, N, rpb, partial);
        REV_HIP(hipGetLastError());
    }
    const RedSeg g = {partial, out, nullptr, (int64_t)N, (int64_t)N, (int64_t)N, P};
    if (defer) { *defer = g; return REV_OK; }
    return reduce_multi(s, &g, 1);
}
template int colsum<float>(hipStream_t, const float*, int64_t, int, int, float*, float*, RedSeg*);

// ---- conversion, with the column sums of what is converted ---------------------------------------------
// grid (column tiles of 4 * lpr floats, row chunks); lpr lanes hold a row's tile, so a narrow row leaves few lanes idle.  The
// rows of a block at a time (256 / lpr) are added in order through LDS at the end.  One pass over the float32 rows instead of one for
// the copy and one for the sums: 12608 x 768 11 + 15 + 14 us with the reduction, now 14 and a segment of a later reduction.
__global__ __launch_bounds__(256) void cvt_colsum_kernel(const float* __restrict__ in, bf16* __restrict__ out, int M, int N,
                                                         int rows_per_block, int lpr, float* __restrict__ partial) {
    __shared__ float4 sh[256];
    const int lane = threadIdx.x & (lpr - 1), grp = threadIdx.x / lpr, groups = 256 / lpr;
    const int col = (blockIdx.x * lpr + lane) * 4;
    const int row1 = min(M, (int)(blockIdx.y + 1) * rows_per_block);
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    if (col < N) {
        int row = blockIdx.y * rows_per_block + grp;
        for (; row < row1; row += 4 * groups) {
            f4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (row + u * groups < row1) v[u] = load4(in + (int64_t)(row + u * groups) * N + col);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (row + u * groups < row1) {
                    acc.x += v[u].x; acc.y += v[u].y; acc.z += v[u].z; acc.w += v[u].w;
                    if (out) store4(out + (int64_t)(row + u * groups) * N + col, v[u]);
                }
        }
    }
    sh[threadIdx.x] = make_float4(acc.x, acc.y, acc.z, acc.w);
    __syncthreads();
    if (grp == 0 && col < N) {
        for (int k = 1; k < groups; ++k) {
            const float4 v = sh[k * lpr + lane];
            acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
        }
        store4(partial + (int64_t)blockIdx.y * N + col, acc);
    }
}
int convert_colsum(hipStream_t s, const float* in, bf16* out, int M, int N, float* sums, float* partial, RedSeg* defer) {
    if (N % 4 != 0) { set_error("convert: the width must be a multiple of 4"); return REV_EINVAL; }
    const int chunks = colsum_chunks(M, N), rpb = (M + chunks - 1) / chunks, P = (M + rpb - 1) / rpb;
    int lpr = 8;
    while (lpr < 64 && lpr * 4 < N) lpr *= 2;
    ProfScope ps(K_CONVERT, s, (double)M * N * (out ? 6 : 4));
    hipLaunchKernelGGL(cvt_colsum_kernel, dim3((N + 4 * lpr - 1) / (4 * lpr), P), dim3(256), 0, s, in, out, M, N, rpb, lpr, partial);
    REV_HIP(hipGetLastError());
    *defer = {partial, sums, nullptr, (int64_t)N, (int64_t)N, (int64_t)N, P};
    return REV_OK;
}

}  // namespace rev
