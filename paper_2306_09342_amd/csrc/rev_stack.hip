// Host side of librevstack: argument checks, workspace layout, the per-block
// recompute (R_i) and gradient (V_i) kernel sequences, and the two schedules
// of the paper's Sec. 3.2 (Reprop: one stream) and Sec. 3.3 (PaReprop: the
// recomputation chain on a second stream, ordered against the gradient chain
// by events and a double-buffered activation slot).
#include "common.h"

#include <mutex>
#include <type_traits>
#include <vector>

namespace rev {

// ---------------------------------------------------------------------------------
// errors
// ---------------------------------------------------------------------------------
static thread_local std::string g_err;
void set_error(const std::string& msg) { g_err = msg; }
int hip_fail(hipError_t e, const char* what, const char* file, int line) {
    g_err = std::string(hipGetErrorString(e)) + " in " + what + " (" + file + ":" + std::to_string(line) + ")";
    return REV_EHIP;
}

// ---------------------------------------------------------------------------------
// per-family timing
// ---------------------------------------------------------------------------------
struct ProfRec { Kind kind; hipEvent_t e0, e1; };
static bool g_prof_on = false;
static std::vector<ProfRec> g_prof_recs;
static double g_prof_ms[K_COUNT];
static int64_t g_prof_n[K_COUNT];
static double g_prof_work[K_COUNT];
static const char* g_kind_names[K_COUNT] = {"gemm_nt", "gemm_wgrad", "attn_fwd", "attn_bwd", "ln_fwd",
                                            "ln_bwd", "colsum", "reduce", "convert", "optimizer", "mixed", "ln_pair"};
static const int g_kind_flops[K_COUNT] = {1, 1, 1, 1, 0, 0, 0, 0, 0, 0, 1, 0};

bool profiling() { return g_prof_on; }

ProfScope::ProfScope(Kind k, hipStream_t s, double work) : kind(k), stream(s), rec(nullptr) {
    if (!g_prof_on) return;
    ProfRec r;
    r.kind = k;
    if (hipEventCreate(&r.e0) != hipSuccess) return;
    if (hipEventCreate(&r.e1) != hipSuccess) { (void)hipEventDestroy(r.e0); return; }
    (void)hipEventRecord(r.e0, s);
    g_prof_recs.push_back(r);
    g_prof_work[k] += work;
    rec = (void*)(uintptr_t)g_prof_recs.size();   // index + 1
}
ProfScope::~ProfScope() {
    if (rec) (void)hipEventRecord(g_prof_recs[(uintptr_t)rec - 1].e1, stream);
}

// ---------------------------------------------------------------------------------
// configuration and packed-parameter layout
// ---------------------------------------------------------------------------------
enum { T_LN1G = 0, T_LN1B, T_WQKV, T_BQKV, T_WPROJ, T_BPROJ, T_LN2G, T_LN2B, T_WFC1, T_BFC1, T_WFC2, T_BFC2, T_COUNT };

static int64_t tensor_count(const rev_cfg& c, int t) {
    const int64_t D = c.d_model, Dm = c.d_mlp;
    switch (t) {
        case T_WQKV: return 3 * D * D;
        case T_BQKV: return 3 * D;
        case T_WPROJ: return D * D;
        case T_WFC1: case T_WFC2: return D * Dm;
        case T_BFC1: return Dm;
        default: return D;
    }
}
static int64_t tensor_offset(const rev_cfg& c, int t) {
    int64_t off = 0;
    for (int i = 0; i < t; ++i) off += tensor_count(c, i);
    return off;
}
static int64_t block_params(const rev_cfg& c) { return tensor_offset(c, T_COUNT); }

static int check_cfg(const rev_cfg* c) {
    if (!c) { set_error("cfg is null"); return REV_EINVAL; }
    if (c->n_blocks <= 0 || c->d_model <= 0 || c->n_heads <= 0 || c->d_mlp <= 0 || c->seq_len <= 0 || c->batch <= 0) {
        set_error("cfg: every size must be positive"); return REV_EINVAL;
    }
    if (c->mode != REV_MODE_FP32 && c->mode != REV_MODE_BF16) { set_error("cfg: unknown mode"); return REV_EINVAL; }
    if (c->d_model % c->n_heads != 0) { set_error("cfg: d_model must be divisible by n_heads"); return REV_EINVAL; }
    const int dh = c->d_model / c->n_heads;
    if (c->d_model % 8 != 0 || c->d_mlp % 8 != 0 || dh % 8 != 0) {
        set_error("cfg: d_model, d_mlp and head_dim must be multiples of 8"); return REV_EINVAL;
    }
    if (dh > 128) { set_error("cfg: head_dim must be <= 128"); return REV_EINVAL; }
    if (c->d_model > 8192 || c->d_mlp > 32768) { set_error("cfg: d_model <= 8192 and d_mlp <= 32768"); return REV_EINVAL; }
    // launch-grid limits: the attention kernels put (sample, head) pairs on the grid's y axis, which holds at most 65535;
    // the token limit keeps tile counts and row offsets of every launch within 32 bits
    if ((int64_t)c->batch * c->seq_len > (int64_t)65535 * 64) {
        set_error("cfg: batch*seq_len must be <= 4194240"); return REV_EINVAL;
    }
    if ((int64_t)c->batch * c->n_heads > 65535) { set_error("cfg: batch*n_heads must be <= 65535"); return REV_EINVAL; }
    if (!(c->ln_eps >= 0.f)) { set_error("cfg: ln_eps must be >= 0"); return REV_EINVAL; }
    return REV_OK;
}

// ---------------------------------------------------------------------------------
// workspace layout (byte offsets, every region 256-byte aligned)
// ---------------------------------------------------------------------------------

struct Layout {
    int64_t slot[2];
    int64_t s_n2, s_h, s_a, s_n1, s_qkv, s_o, s_lse, s_st1, s_st2;   // relative to a slot
    int64_t ring[3][2];
    int64_t cot[2][2];     // float32 cotangent levels
    int64_t cot2b[3];      // act-typed copies of the stream-2 cotangent (bf16 mode), by block index mod 3
    int64_t gy1b[2];       // act-typed copy of gY1 (bf16 mode), by block parity
    int64_t dh[2], dqkv[2]; // by block parity: read by the weight-gradient kernels of the block
    int64_t dn, dO, delta;
    int64_t part_ln[2], part_col[2], part_wg;   // partial sums of the deferred reductions of a block
    int64_t total;
    int64_t part_wg_elems;
    int64_t slot_bytes;
    int ring_levels;
};

// compact = the layout of the sequential schedule (and of the forward map): nothing of block i-1
// is produced while block i is still being consumed, so one activation slot, two residual levels and
// one copy of each per-block gradient temporary are enough.  The full layout doubles those, which is
// the extra memory the parallel schedule pays (Sec. 3.3, Sec. 4.2).
static Layout make_layout(const rev_cfg& c, bool compact) {
    Layout L = {};
    const int64_t M = (int64_t)c.batch * c.seq_len, D = c.d_model, Dm = c.d_mlp;
    const int64_t es = (c.mode == REV_MODE_BF16) ? 2 : 4;
    int64_t off = 0;
    auto take = [&](int64_t bytes) { int64_t o = off; off += (bytes + 255) / 256 * 256; return o; };
    // one activation slot
    {
        int64_t base = off;
        L.s_n2 = take(M * D * es) - base;
        L.s_h = take(M * Dm * es) - base;
        L.s_a = take(M * Dm * es) - base;
        L.s_n1 = take(M * D * es) - base;
        L.s_qkv = take(M * 3 * D * es) - base;
        L.s_o = take(M * D * es) - base;
        L.s_lse = take((int64_t)c.batch * c.n_heads * c.seq_len * 4) - base;
        L.s_st1 = take(M * 2 * 4) - base;
        L.s_st2 = take(M * 2 * 4) - base;
        L.slot_bytes = off - base;
        L.slot[0] = base;
        L.slot[1] = compact ? base : take(L.slot_bytes);
    }
    L.ring_levels = compact ? 2 : 3;
    for (int r = 0; r < L.ring_levels; ++r)
        for (int s = 0; s < 2; ++s) L.ring[r][s] = take(M * D * 4);
    for (int r = 0; r < 2; ++r)
        for (int s = 0; s < 2; ++s) L.cot[r][s] = take(M * D * 4);
    if (c.mode == REV_MODE_BF16) {
        L.cot2b[0] = take(M * D * es);
        L.cot2b[1] = take(M * D * es);
        L.cot2b[2] = take(M * D * es);
        L.gy1b[0] = take(M * D * es);
        L.gy1b[1] = compact ? L.gy1b[0] : take(M * D * es);
    }
    for (int r = 0; r < 2; ++r) {
        L.dh[r] = (compact && r) ? L.dh[0] : take(M * Dm * es);
        L.dqkv[r] = (compact && r) ? L.dqkv[0] : take(M * 3 * D * es);
    }
    L.dn = take(M * D * es);
    L.dO = L.dn;           // dn is consumed by LN2's backward before dO is written, and dO by attention's before dn is again
    // read by the bf16 attention backward (heads up to 96 wide); the float32 products form it in registers
    L.delta = take(c.mode == REV_MODE_BF16 && D / c.n_heads <= 96 ? (int64_t)c.batch * c.n_heads * c.seq_len * 4 : 0);
    L.part_ln[0] = take(ln_bwd_partial_elems((int)M, (int)D) * 4);
    L.part_ln[1] = take(ln_bwd_partial_elems((int)M, (int)D) * 4);
    {
        // [0]: fc1 bias gradient (column-sum strips of the GELU' epilogue); [1]: float32 mode, the QKV bias gradients
        const int64_t e0 = (int64_t)(c.mode == REV_MODE_BF16 ? gemm_colsum_strips((int)M, (int)Dm, (int)D) : gemm_f32_colsum_strips((int)M, (int)Dm)) * Dm;
        const int64_t e1 = c.mode == REV_MODE_BF16 || M <= COLSUM_ROWS ? 0 : colsum_partial_elems((int)M, (int)(3 * D));
        L.part_col[0] = take(e0 * 4);
        L.part_col[1] = take(e1 * 4);
    }
    if (c.mode == REV_MODE_BF16) {
        // scratch for the pieces of the four weight gradients (fc2, fc1, proj, qkv), which go out as one launch: none
        // where their tiles fill the device without cutting the token range
        const int nn[4] = {(int)D, (int)Dm, (int)D, (int)(3 * D)}, kk[4] = {(int)Dm, (int)D, (int)D, (int)D};
        L.part_wg_elems = wgrad_scratch_elems((int)M, nn, kk, 4);
        L.part_wg = take(L.part_wg_elems * 4);
    }
    L.total = off;
    return L;
}

// ---------------------------------------------------------------------------------
// event pool (the only state kept between calls)
// ---------------------------------------------------------------------------------
// A two-stream call leases a set of events that no other call holds while it enqueues, so calls issued
// from several host threads (on their own workspaces and streams) never record or wait on each other's
// events.  The lease ends when the enqueue returns: a wait that is already enqueued refers to the record
// that preceded it, so a later call may record the same event again without disturbing it.
static std::mutex g_ev_mu;
static std::vector<hipEvent_t> g_ev_free;
struct EventLease {
    std::vector<hipEvent_t> ev;
    int take(int n) {
        std::lock_guard<std::mutex> lk(g_ev_mu);
        while ((int)ev.size() < n) {
            hipEvent_t e;
            if (!g_ev_free.empty()) {
                e = g_ev_free.back();
                g_ev_free.pop_back();
            } else {
                REV_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
            }
            ev.push_back(e);
        }
        return REV_OK;
    }
    ~EventLease() {
        std::lock_guard<std::mutex> lk(g_ev_mu);
        g_ev_free.insert(g_ev_free.end(), ev.begin(), ev.end());
    }
};

// ---------------------------------------------------------------------------------
// the per-block kernel sequences
// ---------------------------------------------------------------------------------
#define RC(expr) do { int _rc = (expr); if (_rc != REV_OK) return _rc; } while (0)

static int gemm_nt(hipStream_t s, const float* A, int64_t lda, const float* B, int64_t ldb, int M, int N, int K, const Epi& e) {
    return gemm_nt_f32(s, A, lda, B, ldb, M, N, K, e);
}
static int gemm_nt(hipStream_t s, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K, const Epi& e) {
    return gemm_nt_bf16(s, A, lda, B, ldb, M, N, K, e);
}

// How a backward call issues the two chains of its blocks.
enum Order { IN_TURN = REV_ORDER_IN_TURN, SIDE_BY_SIDE = REV_ORDER_SIDE_BY_SIDE, TWO_STREAMS = REV_ORDER_TWO_STREAMS };

static double forward_flops(const rev_cfg& c) {               // of a block
    const double M = (double)c.batch * c.seq_len, D = c.d_model;
    return 2.0 * M * D * (4.0 * D + 2.0 * c.d_mlp) + 4.0 * M * c.seq_len * D;
}
// Blocks whose launches are mostly latency: on one stream, QKV's input gradient, the weight gradients, the column sums and the
// second stages of the sums that the launches before left are one launch, and where the workspace holds the layout of two streams
// the two chains are issued side by side, each launch of R_{i-1} in one of D_i (grad_d).  Four blocks, us a call: one stream, one chain
// after the other / one stream, side by side / two streams, and in brackets side by side with the fork and the join of the parallel
// schedule, which cost about 45 us:
//                        197 rows                394                     788                     1000
//     D =  256           309 / 201 / 404 (255)   339 / 214 / 418 (267)   344 / 227 / 420 (280)   423 / 278 / 428 (329)
//     D =  768           433 / 305 / 357 (324)   507 / 352 / 439 (400)   601 / 520 / 515 (556)   701 / 597 / 600 (640)
//     D = 1280           706 / 547 / 598 (565)   914 / 736 / 720 (776)   1228 / 1045 / 995 (1090)
//     float32, D = 256   440 / 293 / 412 (349)   476 / 340 / 429 (394)   554 / 444 / 511 (495)   702 / 567 / 658 (615)
// So the parallel schedule takes two streams from about 8e9 FLOP of a block's forward on (float32: 2.2e9; beyond it too much of the
// chip is busy).  Two to 24 blocks: the same lines.  Rows of more than 1280 floats are too wide for the LayerNorm pair, and two streams are
// faster from the first row on; just below, from where 32x32 tiles no longer hold two products of that width (288 of them) on.  Side by side with
// the fork and the join / two streams, us: D = 1280, 32 blocks, 50 rows 3073 / 3223, 100 3725 / 3432, 128 3975 / 3685, 197 (8e9 FLOP) 4095 / 4117;
// 24 blocks, 77 rows (240 tiles) 2376 / 2533; D = 1248, 100 rows (312 tiles) 2828 / 2606; D = 1216, 197 rows 2820 / 2871; three blocks, D = 1344, 16 rows (7e8) 384 / 349, 150 (6.6e9) 470 / 415; D = 1536, 100 rows 543 / 479; D = 4096, 16 rows 1854 / 1742.
static bool side_by_side_is_faster(const rev_cfg& c) {
    if (c.mode != REV_MODE_BF16) return forward_flops(c) < 2.2e9;
    const int rows = c.batch * c.seq_len, pair_tiles = 2 * ((rows + 31) / 32) * ((c.d_model + 31) / 32);
    return forward_flops(c) < 8e9 && c.d_model <= 1280 && (c.d_model <= 1216 || pair_tiles <= 288);
}
// The same without the common launch of the weight gradients, beyond 1024 rows or 512 64x64 tiles of them.  Four blocks, us a call: one
// stream, in turn / side by side / two streams.  bf16, D = 64: 1576 rows 281 / 233 / 364, 12608 423 / 396 / 518; D = 128: 3152 rows 366 / 308 /
// 382, 6304 434 / 396 / 416, 12608 (6e9 FLOP) 578 / 581 / 528; D = 256: 3152 473 / 445 / 424; D = 512: 1576 (1e10) 559 / 534 / 478, 3152 (2e10)
// 767 / 770 / 877.  float32, D = 64: 3152 464 / 402 / 570; D = 256: 1576 824 / 760 / 753; D = 384: 3152 (1.2e10) 2463 / 2424 / 2323; three
// blocks of 16 rows, side by side / two streams: D = 512 331 / 361, D = 640 387 / 374, D = 768 437 / 430.
// Narrow blocks of very many rows have as few FLOP, but what limits them is memory: with the intermediates of two blocks in turn the memory-side
// cache keeps less of either, and two streams fill the chip.  By rows times width, over 550 stacks of 2 to 12 blocks.  One stream, in turn / side by side:
// bf16, 11866 x 128 (1.5e6) 1046 / 1008, 18100 x 96 (1.7e6) 278 / 277, 31552 x 64 (2.0e6) 282 / 298, 34742 x 64 (2.2e6) 1327 / 1416; float32, 9062 x 64
// 974 / 913, 9828 x 128 (1.26e6) 3599 / 3527, 13489 x 128 (1.7e6) 4593 / 4672, 34580 x 64 (2.2e6) 5393 / 5590.  Two streams, two streams / side by
// side: bf16, 8029 x 64 (5.1e5) 222 / 174, 6765 x 80 (5.4e5) 239 / 257, 8680 x 80 (6.9e5) 608 / 699, 11390 x 64 (7.3e5) 481 / 382, 15617 x 64
// (1e6) 600 / 652, 42780 x 32 (1.4e6) 837 / 1043: from 5.2e5 to 1.2e6 the two are even in the mean; float32, 1440 x 64 505 / 459, 1125 x 128 (1.44e5)
// 328 / 286, 2006 x 80 (1.6e5) 728 / 773, 9174 x 32 (2.9e5) 560 / 630.
static bool apart_side_by_side_is_faster(const rev_cfg& c, bool two_streams) {
    const bool bf = c.mode == REV_MODE_BF16;
    const double floats = (double)c.batch * c.seq_len * c.d_model;
    if (two_streams) return c.d_model <= (bf ? 1280 : 512) && forward_flops(c) < (bf ? 2e9 : 5e8) && floats <= (bf ? 5.2e5 : 1.55e5);
    return forward_flops(c) < (bf ? 8e9 : 1.2e10) && floats <= (bf ? 1.8e6 : 1.3e6);
}
// Blocks of 4.5e7 to 1.3e8 weights, which the memory-side cache does not keep from pass to pass, and few rows: a launch of one product in
// 32x32 tiles has as many loads under way as one of two products in the 64x64 tiles that hold both, and the chains take turns.  Three blocks, one
// stream, in turn / side by side, us: D = 2048, 100 rows (1e10 FLOP) 692 / 735, 125 722 / 770, 150 (1.5e10) 821 / 827, 200 852 / 837; D = 2560, 16
// rows 915 / 952, 50 962 / 1039, 75 (1.2e10) 1027 / 1068, 100 (1.6e10) 1186 / 1165; D = 3072, 50 rows 1178 / 1270, 75 (1.7e10) 1382 / 1356.  Smaller
// and larger blocks: D = 1792, 16 rows 552 / 526, 100 609 / 616, 200 772 / 698; D = 3584, 16 rows 1600 / 1513, 50 1656 / 1617.
static bool turns_are_faster(const rev_cfg& c) {
    const double weights = (double)block_params(c);
    return c.mode == REV_MODE_BF16 && weights > 4.5e7 && weights < 1.3e8 && forward_flops(c) < 1.4e10;
}
// Both schedules and any number of blocks must sum the weight gradients in as many pieces: where two streams would be taken, only what
// they sum in one.  A single block has nothing to put side by side, but goes in one stream all the same where the weight gradients
// ride, which costs it nothing: 1000 rows of 512, two streams and two pieces / one stream, 159 / 149 us, of 256 124 / 120.
static bool blocks_ride(const rev_cfg& c) {
    const int M = c.batch * c.seq_len, D = c.d_model, Dm = c.d_mlp;
    const int nn[4] = {D, Dm, D, 3 * D}, kk[4] = {Dm, D, D, D};
    if (c.mode != REV_MODE_BF16) return gemm_wgrad_f32_together(M, D, nn, kk, 4);
    return !turns_are_faster(c) && gemm_wgrad_bf16_together(M, nn, kk, 4, !side_by_side_is_faster(c));
}

// Two streams cost the host three events and three waits per block, so where the line lies depends on the host's speed.
// Measured (us a call, one stream / two, calls back to back) on a slow host, 12 blocks, and on a fast one, 6 blocks, by FLOP
// of a block's forward:
//              slow: bf16         float32         fast: bf16      float32
//    6.6e6       769 / 1018       848 / 1249        450 / 443      537 / 478
//    2.9e7      1047 / 1006      1142 / 1262        538 / 453      616 / 500
//    5.5e7      1039 / 1010      1164 / 1241        522 / 435      608 / 503
//    9.7e7      1202 /  976      1296 / 1270        635 / 460      724 / 546
//    2.0e8      1240 / 1043      1418 / 1241        657 / 465      796 / 618
// From 8e7 on two streams win on both, where the chains cannot be issued side by side on one.  Same kernels in the same order, so
// the same results under every order.
// A sequential pass takes the layout of the parallel one where the workspace holds it and the blocks are small, for it issues both chains
// side by side then.  schedule: 0 = Reprop, 1 = PaReprop, others: one chain alone
static Order issue_order(const rev_cfg& c, int schedule, int64_t ws_bytes) {
    if (schedule > 1) return IN_TURN;
    const bool ride = blocks_ride(c), several = c.n_blocks > 1;
    if (schedule == 0)
        return several && !turns_are_faster(c) && (ride || apart_side_by_side_is_faster(c, false)) && ws_bytes >= make_layout(c, false).total ? SIDE_BY_SIDE : IN_TURN;
    if (forward_flops(c) < 8e7 || (ride ? side_by_side_is_faster(c) : several && apart_side_by_side_is_faster(c, true)))
        return several ? SIDE_BY_SIDE : IN_TURN;
    return TWO_STREAMS;
}

template <typename T>
struct Runner {
    static constexpr bool kBf16 = sizeof(T) == 2;
    rev_cfg c;
    Layout L;
    char* ws;
    const T* params;
    float* dparams;
    int M, D, Dm, H, dh, B, Tn;
    bool solo;      // one stream: every kernel has the device to itself
    Order order;
    const int* key_len = nullptr;   // optional key-padding mask: valid keys per sample (device, [batch])

    Runner(const rev_cfg& cfg, const void* p, float* dp, void* w, bool compact, bool one_stream, Order o)
        : c(cfg), L(make_layout(cfg, compact)), ws((char*)w), params((const T*)p), dparams(dp), solo(one_stream), order(o) {
        M = c.batch * c.seq_len; D = c.d_model; Dm = c.d_mlp; H = c.n_heads; dh = D / H; B = c.batch; Tn = c.seq_len;
    }
    Epi epi0() const { Epi e = {}; e.solo = solo; return e; }
    template <typename U> U* at(int64_t off) const { return reinterpret_cast<U*>(ws + off); }
    const T* P(int blk, int t) const { return params + (int64_t)blk * block_params(c) + tensor_offset(c, t); }
    float* G(int blk, int t) const { return dparams + (int64_t)blk * block_params(c) + tensor_offset(c, t); }
    struct Slot { T *n2, *h, *a, *n1, *qkv, *o; float *lse, *st1, *st2; };
    Slot slot(int i) const {
        int64_t b = L.slot[i & 1];
        return {at<T>(b + L.s_n2), at<T>(b + L.s_h), at<T>(b + L.s_a), at<T>(b + L.s_n1), at<T>(b + L.s_qkv),
                at<T>(b + L.s_o), at<float>(b + L.s_lse), at<float>(b + L.s_st1), at<float>(b + L.s_st2)};
    }

    // ---- the launches of a block's two maps ----
    using Gemm = GemmCall<T>;
    using Ln = LnFwdCall<T, T>;
    Ln ln1(int blk, const float* x2, const Slot& sl) const { return {x2, P(blk, T_LN1G), P(blk, T_LN1B), c.ln_eps, sl.n1, sl.st1}; }
    Ln ln2(int blk, const float* y1, const Slot& sl) const { return {y1, P(blk, T_LN2G), P(blk, T_LN2B), c.ln_eps, sl.n2, sl.st2}; }
    Gemm qkv_map(int blk, const Slot& sl) const {
        Epi e = epi0(); e.kind = EPI_BIAS; e.out = sl.qkv; e.bias = P(blk, T_BQKV); e.ldo = 3 * D;
        return {sl.n1, D, P(blk, T_WQKV), D, 3 * D, D, e};
    }
    // out1 = in1 + sign * (o Wp^T + bp)
    Gemm proj_map(int blk, const Slot& sl, const float* in1, float* out1, float sign) const {
        Epi e = epi0(); e.kind = EPI_RESIDUAL; e.outf = out1; e.res = in1; e.bias = P(blk, T_BPROJ); e.sign = sign; e.ldo = D;
        return {sl.o, D, P(blk, T_WPROJ), D, D, D, e};
    }
    // the pre-activation of the MLP is kept only where a backward step will read it
    Gemm fc1_map(int blk, const Slot& sl, bool keep_h) const {
        Epi e = epi0(); e.kind = EPI_BIAS_GELU; e.out = keep_h ? sl.h : nullptr; e.out2 = sl.a; e.bias = P(blk, T_BFC1); e.ldo = Dm;
        return {sl.n2, D, P(blk, T_WFC1), D, Dm, D, e};
    }
    // out2 = in2 + sign * (a W2^T + b2)
    Gemm fc2_map(int blk, const Slot& sl, const float* in2, float* out2, float sign) const {
        Epi r = epi0(); r.kind = EPI_RESIDUAL; r.outf = out2; r.res = in2; r.bias = P(blk, T_BFC2); r.sign = sign; r.ldo = D;
        return {sl.a, Dm, P(blk, T_WFC2), Dm, D, Dm, r};
    }
    int run(hipStream_t s, const Ln& l) { return ln_forward<T, T>(s, l.x, l.g, l.b, l.eps, l.y, l.stats, M, D); }
    int run(hipStream_t s, const Gemm& g) { return gemm_nt(s, g.A, g.lda, g.B, g.ldb, M, g.N, g.K, g.epi); }

    // F branch pieces up to the projection input: n1, qkv, o, lse from x2
    int f_pre(hipStream_t s, int blk, const float* x2, const Slot& sl) {
        RC(run(s, ln1(blk, x2, sl)));
        RC(run(s, qkv_map(blk, sl)));
        return attention_forward<T>(s, sl.qkv, sl.o, sl.lse, B, Tn, H, dh, key_len);
    }
    // out2 = in2 + sign * G(y1)
    int g_branch(hipStream_t s, int blk, const float* y1, const Slot& sl, const float* in2, float* out2, float sign,
                 bool keep_h = true) {
        RC(run(s, ln2(blk, y1, sl)));
        RC(run(s, fc1_map(blk, sl, keep_h)));
        return run(s, fc2_map(blk, sl, in2, out2, sign));
    }

    // forward of block blk (0-based): (x1,x2) -> (y1,y2)
    int forward_block(hipStream_t s, int blk, const float* x1, const float* x2, float* y1, float* y2) {
        Slot sl = slot(0);
        RC(f_pre(s, blk, x2, sl));
        RC(run(s, proj_map(blk, sl, x1, y1, 1.f)));
        return g_branch(s, blk, y1, sl, x2, y2, 1.f, false);
    }

    // R_i: (y1,y2) -> (x1,x2) and the slot of block blk
    int recompute(hipStream_t s, int blk, const float* y1, const float* y2, float* x1, float* x2) {
        Slot sl = slot(blk);
        RC(g_branch(s, blk, y1, sl, y2, x2, -1.f));
        RC(f_pre(s, blk, x2, sl));
        return run(s, proj_map(blk, sl, y1, x1, -1.f));
    }

    // dA[M,Kin] = dC[M,Nout] * W[Nout,Kin], the weight read as it is stored; with a map of the block below beside it where there is one
    int dgrad(hipStream_t s, int blk, int wt, const T* dC, int Nout, int Kin, const Epi& e, bool paired, const Gemm& beside) {
        if (paired) return gemm_pair(s, {dC, Nout, P(blk, wt), Kin, Kin, Nout, e}, beside, M);
        if constexpr (kBf16) {
            return gemm_nn_bf16(s, dC, Nout, P(blk, wt), Kin, M, Kin, Nout, e);
        } else {
            return gemm_nn_f32(s, dC, Nout, P(blk, wt), Kin, M, Kin, Nout, e);
        }
    }
    // LayerNorm backward, with the LayerNorm forward of the block below beside it where there is one
    int ln_back(hipStream_t s, const LnBwdCall<T, T>& b, bool paired, const Ln& beside, RedSeg* seg) {
        if (paired) return ln_pair<T, T>(s, b, beside, M, D, seg);
        return ln_backward<T, T>(s, b.dn, b.x, b.stats, b.g, b.r, b.out, b.outb, b.dgb, b.dbias, b.partial, M, D, seg);
    }

    // V_i is issued as two kernel sequences.
    //   grad_d: the input-gradient chain (everything the next block down waits for) plus the cheap
    //           vector/bias gradients that fall out of its kernels;
    //   grad_w: the four weight-gradient GEMMs, which only consume what grad_d and R_i produced.
    // Under PaReprop grad_w rides on the recompute stream, so it overlaps the chain of the same block.
    // y1: first stream of the block's outputs, x2: second stream of its inputs.
    // d1, d2: incoming cotangents (float32); d2b: act-typed copy of d2.
    // o1, o2: outgoing cotangents; o2b: act-typed copy of o2 (nullable).
    // The second stages of the fixed-order sums are left in segs (five at most from grad_d, six from grad_w) for one launch.
    // done_dqkv (nullable): recorded on s when dh, gY1 and dqkv are complete.
    T* gy1_act(int blk, float* o1) const { return kBf16 ? at<T>(L.gy1b[blk & 1]) : reinterpret_cast<T*>(o1); }

    using Item = typename std::conditional<kBf16, WgradItem, WgradF32Item>::type;
    struct Items { Item p[4]; };
    Items w_items(int blk, const T* d2b, float* o1) const {
        Slot sl = slot(blk);
        T* dhb = at<T>(L.dh[blk & 1]);
        T* dqkv = at<T>(L.dqkv[blk & 1]);
        T* gy1b = gy1_act(blk, o1);
        return {{{d2b, D, sl.a, Dm, D, Dm, G(blk, T_WFC2), nullptr}, {dhb, Dm, sl.n2, D, Dm, D, G(blk, T_WFC1), nullptr},
                 {gy1b, D, sl.o, D, D, D, G(blk, T_WPROJ), nullptr},
                 {dqkv, 3 * D, sl.n1, D, 3 * D, D, G(blk, T_WQKV), sums_ride() ? G(blk, T_BQKV) : nullptr}}};
    }
    // QKV's bias gradient (column sums of dqkv) in the launch of the weight gradients, which reads dqkv anyway
    bool sums_ride() const { return kBf16 || M <= COLSUM_ROWS; }
    bool all_ride() const { return blocks_ride(c); }

    // together: grad_w's work is done here too, with the launch that ends the attention branch, and what segs holds by then
    // (with what the block above left there) is summed; the last LayerNorm's sums are left in segs.
    // below (nullable): the recomputation of the block below, whose seven launches have the order and the kinds of D_i's,
    // one launch on, and depend on none of them: each rides in one of D_i's.  Its first LayerNorm is done before; the last launch takes
    // that of the block below it, in the slot of this block, whose grad_w is therefore done before it.
    struct Below { const float *y1, *y2; float *x1, *x2; };
    int grad_d(hipStream_t s, int blk, const float* y1, const float* x2, const float* d1, const float* d2,
               const T* d2b, float* o1, float* o2, T* o2b, hipEvent_t done_dqkv, RedSeg* segs, int* n, bool together, const Below* below) {
        Slot sl = slot(blk), lo = slot(blk + 1);             // (the other one)
        const Below w = below ? *below : Below{};
        const bool pair = below != nullptr;
        const int lb = pair ? blk - 1 : 0;
        T* dhb = at<T>(L.dh[blk & 1]);
        T* dqkv = at<T>(L.dqkv[blk & 1]);
        T* dn = at<T>(L.dn);
        T* dO = at<T>(L.dO);
        float* pcol0 = at<float>(L.part_col[0]);
        T* gy1b = gy1_act(blk, o1);
        int& nseg = *n;

        // ---- G branch: dh = (dY2 W2) * gelu'(h); the bias gradient of fc1 (column sums of dh) rides
        // in the epilogue
        Epi e = epi0(); e.kind = EPI_GELU_BWD; e.out = dhb; e.aux = sl.h; e.ldo = Dm;
        e.colsum = pcol0;
        RC(dgrad(s, blk, T_WFC2, d2b, D, Dm, e, pair, fc1_map(lb, lo, true)));
        segs[nseg++] = {pcol0, G(blk, T_BFC1), nullptr, (int64_t)Dm, (int64_t)Dm, (int64_t)Dm,
                        kBf16 ? gemm_colsum_strips(M, Dm, D) : gemm_f32_colsum_strips(M, Dm)};
        Epi p = epi0(); p.kind = EPI_PLAIN; p.out = dn; p.ldo = D;
        RC(dgrad(s, blk, T_WFC1, dhb, Dm, D, p, pair, fc2_map(lb, lo, w.y2, w.x2, -1.f)));
        // gY1 = dY1 + LN2bwd(dn); its column sums are the bias gradient of the projection
        RC(ln_back(s, {dn, y1, sl.st2, P(blk, T_LN2G), d1, o1, kBf16 ? gy1b : nullptr, G(blk, T_LN2G), G(blk, T_BPROJ), at<float>(L.part_ln[0])},
                   pair, ln1(lb, w.x2, lo), &segs[nseg++]));
        // ---- F branch
        Epi q = epi0(); q.kind = EPI_PLAIN; q.out = dO; q.ldo = D;
        RC(dgrad(s, blk, T_WPROJ, gy1b, D, D, q, pair, qkv_map(lb, lo)));
        const Items wi = w_items(blk, d2b, o1);
        const AttnFwdCall<T> fwd = {lo.qkv, lo.o, lo.lse};
        int begun = 0;                                       // weight gradients whose operands are ready before dqkv
        bool attended = !pair;                               // the block below has had its attention
        if constexpr (kBf16) {
            if (together && attention_takes_wgrad(B, Tn, H, dh)) begun = 3;
            if (begun) RC(attention_backward_wgrad(s, sl.qkv, sl.o, dO, sl.lse, dqkv, B, Tn, H, dh, key_len, wi.p, begun, pair ? &fwd : nullptr));
            attended |= begun > 0;
        } else if (pair) {
            RC(attention_pair_f32(s, sl.qkv, sl.o, dO, sl.lse, dqkv, B, Tn, H, dh, key_len, fwd));
            attended = true;
        }
        if (!begun && (kBf16 || !pair)) RC((attention_backward<T>(s, sl.qkv, sl.o, dO, sl.lse, dqkv, at<float>(L.delta), B, Tn, H, dh, key_len, solo)));
        if (!attended) RC(attention_forward<T>(s, fwd.qkv, fwd.o, fwd.lse, B, Tn, H, dh, key_len));
        if (done_dqkv) REV_HIP(hipEventRecord(done_dqkv, s));
        Epi r = epi0(); r.kind = EPI_PLAIN; r.out = dn; r.ldo = D;
        if (together) {
            const Gemm input = {dqkv, 3 * D, P(blk, T_WQKV), D, D, 3 * D, r}, proj = proj_map(lb, lo, w.y1, w.x1, -1.f), *beside = pair ? &proj : nullptr;
            if constexpr (kBf16) RC(gemm_nn_wgrad_bf16(s, input, M, wi.p + begun, 4 - begun, segs, nseg, beside));
            else RC(gemm_nn_wgrad_f32(s, input, M, wi.p, 4, segs, nseg, beside));
            nseg = 0;
        } else {
            RC(dgrad(s, blk, T_WQKV, dqkv, 3 * D, D, r, pair, proj_map(lb, lo, w.y1, w.x1, -1.f)));
            if constexpr (!kBf16)
                if (!sums_ride()) RC(colsum<T>(s, dqkv, 3 * D, M, 3 * D, G(blk, T_BQKV), at<float>(L.part_col[1]), &segs[nseg++]));
            if (pair) RC(grad_w(s, blk, d2b, o1, segs, n));      // before the last launch overwrites n2 of this slot
        }
        // dX2 = dY2 + LN1bwd(dn); dX2 is the block below's dY2, so its column sums are that block's
        // fc2 bias gradient
        return ln_back(s, {dn, x2, sl.st1, P(blk, T_LN1G), d2, o2, kBf16 ? o2b : nullptr, G(blk, T_LN1G), blk > 0 ? G(blk - 1, T_BFC2) : nullptr,
                           at<float>(L.part_ln[1])}, pair && blk >= 2, pair && blk >= 2 ? ln2(blk - 2, w.x1, sl) : Ln{}, &segs[nseg++]);
    }

    int grad_w(hipStream_t s, int blk, const T* d2b, float* o1, RedSeg* segs, int* nseg) {
        const Items w = w_items(blk, d2b, o1);
        if constexpr (kBf16) {
            // all four in one launch: together their tiles fill the device without cutting the token range (or with
            // fewer cuts), which saves the float32 pieces and most of their reduction
            int n = 0;
            RC(gemm_wgrad_bf16_group(s, w.p, 4, M, at<float>(L.part_wg), L.part_wg_elems, segs + *nseg, &n));
            *nseg += n;
            return REV_OK;
        }
        else return gemm_wgrad_f32_group(s, w.p, 4, M);
    }

    // residual level `lvl` (0..N): stream s1/s2 pointers
    struct Ptrs { const float* in1; const float* in2; float* out1; float* out2; };
    float* res(int lvl, int st, float* x_out1, float* x_out2) const {
        if (lvl == 0 && st == 0 && x_out1) return x_out1;
        if (lvl == 0 && st == 1 && x_out2) return x_out2;
        return at<float>(L.ring[lvl % L.ring_levels][st]);
    }

    // schedule: 0 = Reprop, 1 = PaReprop, 2 = R chain only, 3 = V chain only
    //
    // PaReprop, stream by stream (block indices 1-based, N at the top):
    //   sr:  R_N | R_{N-1}  W_N | R_{N-2}  W_{N-1} | ...      (W_i = grad_w of block i)
    //   sv:  D_N | D_{N-1}      | D_{N-2}          | ...      (D_i = grad_d of block i)
    // Orderings across the streams (three events and three waits per block, in float32 mode four: each costs the host about
    // as much as a launch):
    //   D_i  after R_i                      (activations of block i exist; W_{i+2} precedes R_i on sr, so the dh/dqkv/gY1
    //                                        buffers of the same parity and the dY2 copy of W_{i+2} are free again)
    //   R_i  after D_{i+2}                  (slot i mod 2 and ring level i+2 are free; W_{i+2} precedes R_i on sr)
    //   W_i  after the attention backward of D_i, the last of its kernels that produce an operand of W_i
    // and sv finally waits for W_1, so everything is ordered before later work on sv.  The dY2 copies rotate over three
    // buffers, so that D_i does not have to wait for W_{i+1}, which reads the copy before the last; in float32 mode W reads
    // the two alternating cotangent levels themselves, and D_i does wait.
    int backward(int schedule, const float* Y1, const float* Y2, const float* dY1, const float* dY2,
                 float* dX1, float* dX2, float* X1o, float* X2o, hipStream_t sv, hipStream_t sr) {
        const int N = c.n_blocks;
        const bool doR = schedule != 3, doV = schedule != 2;
        enum { E_R = 0, E_D, E_DQKV, E_W };                       // E_W: float32 mode only
        constexpr int EPB = kBf16 ? 3 : 4;
        EventLease lease;
        std::vector<hipEvent_t>& ev = lease.ev;
        auto E = [&](int i, int k) { return ev[(i - 1) * EPB + k]; };
        const bool two = order == TWO_STREAMS;
        const bool together = !two && all_ride();
        const int per = two ? EPB * N : 0;
        const hipStream_t sv_caller = sv;
        if (schedule == 1) {
            RC(lease.take(per + 2));
            REV_HIP(hipEventRecord(ev[per], sv));                 // fork
            REV_HIP(hipStreamWaitEvent(sr, ev[per], 0));
            // One stream: it is the recompute stream, so that the call keeps its order with the caller's work on both.
            if (!two) sv = sr;
        } else {
            sr = sv;
        }
        const T* top2b = nullptr;
        RedSeg segs[RED_MAX_SEGS];
        int nseg = 0;
        auto reduce = [&](hipStream_t s, RedSeg* which, int* n) -> int {
            const int rc = reduce_multi(s, which, *n);
            *n = 0;
            return rc;
        };
        if (doV) {
            // the incoming dY2 in the activation type, and the fc2 bias gradient of the top block: its column sums (lower
            // blocks get theirs from the LayerNorm-backward kernel that produces their dY2).  The partial sums are added with
            // those of D_N; until then they lie in the cotangent level that D_{N-1} is the first to write.
            T* b = kBf16 ? at<T>(L.cot2b[N % 3]) : nullptr;
            RC(convert_colsum(sv, dY2, reinterpret_cast<bf16*>(b), M, D, G(N - 1, T_BFC2), at<float>(L.cot[N & 1][0]), &segs[nseg++]));
            top2b = kBf16 ? b : reinterpret_cast<const T*>(dY2);
        }
        auto run_R = [&](int i) -> int {   // i = N..1 (1-based block index)
            const float* y1 = (i == N) ? Y1 : res(i, 0, X1o, X2o);
            const float* y2 = (i == N) ? Y2 : res(i, 1, X1o, X2o);
            return recompute(sr, i - 1, y1, y2, res(i - 1, 0, X1o, X2o), res(i - 1, 1, X1o, X2o));
        };
        auto d2b_of = [&](int i) -> const T* {
            if constexpr (kBf16) return (i == N) ? top2b : at<T>(L.cot2b[i % 3]);
            else return reinterpret_cast<const T*>((i == N) ? dY2 : at<float>(L.cot[i & 1][1]));
        };
        auto o1_of = [&](int i) -> float* { return (i == 1) ? dX1 : at<float>(L.cot[(i - 1) & 1][0]); };
        auto run_D = [&](int i, hipEvent_t done_dqkv, const Below* below = nullptr) -> int {
            const float* y1 = (i == N) ? Y1 : res(i, 0, X1o, X2o);
            const float* x2 = res(i - 1, 1, X1o, X2o);
            const float* d1 = (i == N) ? dY1 : at<float>(L.cot[i & 1][0]);
            const float* d2 = (i == N) ? dY2 : at<float>(L.cot[i & 1][1]);
            float* o2 = (i == 1) ? dX2 : at<float>(L.cot[(i - 1) & 1][1]);
            T* o2b = nullptr;
            if constexpr (kBf16) o2b = (i == 1) ? nullptr : at<T>(L.cot2b[(i - 1) % 3]);
            return grad_d(sv, i - 1, y1, x2, d1, d2, d2b_of(i), o1_of(i), o2, o2b, done_dqkv, segs, &nseg, together, below);
        };
        if (two) {
            // nothing runs beside R_N, and its launches take the tiles of one stream (one block, D = 800, 1284 rows: 240 -> 236 us)
            solo = true;
            RC(run_R(N));
            solo = false;
            REV_HIP(hipEventRecord(E(N, E_R), sr));
            for (int i = N; i >= 1; --i) {
                // ---- D_i on the gradient stream
                REV_HIP(hipStreamWaitEvent(sv, E(i, E_R), 0));
                if (!kBf16 && i + 1 <= N) REV_HIP(hipStreamWaitEvent(sv, E(i + 1, E_W), 0));
                RC(run_D(i, E(i, E_DQKV)));
                RC(reduce(sv, segs, &nseg));
                if (i > 2) REV_HIP(hipEventRecord(E(i, E_D), sv));
                // ---- R_{i-1}, then W_i, on the recompute stream
                if (i - 1 >= 1) {
                    if (i + 1 <= N) REV_HIP(hipStreamWaitEvent(sr, E(i + 1, E_D), 0));
                    RC(run_R(i - 1));
                    REV_HIP(hipEventRecord(E(i - 1, E_R), sr));
                }
                REV_HIP(hipStreamWaitEvent(sr, E(i, E_DQKV), 0));
                RedSeg wsegs[RED_MAX_SEGS];
                int nw = 0;
                RC(grad_w(sr, i - 1, d2b_of(i), o1_of(i), wsegs, &nw));
                RC(reduce(sr, wsegs, &nw));
                if (!kBf16 && i > 1) REV_HIP(hipEventRecord(E(i, E_W), sr));
            }
        } else if (order == SIDE_BY_SIDE) {
            RC(run_R(N));
            RC(run(sv, ln2(N - 2, res(N - 1, 0, X1o, X2o), slot(N - 2))));
            for (int i = N; i >= 1; --i) {
                const Below below = {res(i - 1, 0, X1o, X2o), res(i - 1, 1, X1o, X2o), i > 1 ? res(i - 2, 0, X1o, X2o) : nullptr,
                                     i > 1 ? res(i - 2, 1, X1o, X2o) : nullptr};
                RC(run_D(i, nullptr, i > 1 ? &below : nullptr));
                if (together) continue;
                if (i == 1) RC(grad_w(sv, 0, d2b_of(1), o1_of(1), segs, &nseg));
                RC(reduce(sv, segs, &nseg));
            }
            RC(reduce(sv, segs, &nseg));
        } else {
            for (int i = N; i >= 1; --i) {
                if (doR) RC(run_R(i));
                if (doV) {
                    RC(run_D(i, nullptr));
                    if (together) continue;
                    RC(grad_w(sv, i - 1, d2b_of(i), o1_of(i), segs, &nseg));
                    RC(reduce(sv, segs, &nseg));
                }
            }
            RC(reduce(sv, segs, &nseg));
        }
        if (schedule == 1) {
            REV_HIP(hipEventRecord(ev[per + 1], sr));             // join
            REV_HIP(hipStreamWaitEvent(sv_caller, ev[per + 1], 0));
        }
        return REV_OK;
    }

    int forward(const float* X1, const float* X2, float* Y1, float* Y2, hipStream_t s) {
        const int N = c.n_blocks;
        for (int i = 1; i <= N; ++i) {
            const float* x1 = (i == 1) ? X1 : at<float>(L.ring[(i - 1) % L.ring_levels][0]);
            const float* x2 = (i == 1) ? X2 : at<float>(L.ring[(i - 1) % L.ring_levels][1]);
            float* y1 = (i == N) ? Y1 : at<float>(L.ring[i % L.ring_levels][0]);
            float* y2 = (i == N) ? Y2 : at<float>(L.ring[i % L.ring_levels][1]);
            RC(forward_block(s, i - 1, x1, x2, y1, y2));
        }
        return REV_OK;
    }
};

static int check_common(const rev_cfg* cfg, const void* ws, int64_t ws_bytes, bool compact) {
    RC(check_cfg(cfg));
    if (!ws) { set_error("workspace is null"); return REV_EINVAL; }
    if (((uintptr_t)ws & 255) != 0) { set_error("workspace must be 256-byte aligned"); return REV_EINVAL; }
    Layout L = make_layout(*cfg, compact);
    if (ws_bytes < L.total) {
        set_error("workspace too small: need " + std::to_string(L.total) + " bytes, got " + std::to_string(ws_bytes));
        return REV_EWORKSPACE;
    }
    return REV_OK;
}

static bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

static int backward_entry(int schedule, const rev_cfg* cfg, const void* params, const float* Y1, const float* Y2,
                          const float* dY1, const float* dY2, float* dX1, float* dX2, float* X1o, float* X2o,
                          float* dparams, void* ws, int64_t ws_bytes, void* sv, void* sr,
                          const int32_t* key_len = nullptr) {
    const bool compact = schedule == 0;          // the sequential schedule runs in the smaller layout
    RC(check_common(cfg, ws, ws_bytes, compact));
    if (!params || !Y1 || !Y2 || !dY1 || !dY2 || !dX1 || !dX2 || !dparams) {
        set_error("a required pointer is null"); return REV_EINVAL;
    }
    if (!aligned16(params) || !aligned16(Y1) || !aligned16(Y2) || !aligned16(dY1) || !aligned16(dY2) || !aligned16(dX1) ||
        !aligned16(dX2) || !aligned16(dparams) || !aligned16(X1o) || !aligned16(X2o)) {
        set_error("every buffer must be 16-byte aligned"); return REV_EINVAL;
    }
    if (schedule == 1 && sv == sr) { set_error("PaReprop needs two different streams"); return REV_EINVAL; }
    if (((uintptr_t)key_len & 3) != 0) { set_error("key_len must be 4-byte aligned"); return REV_EINVAL; }
    const Order order = issue_order(*cfg, schedule, ws_bytes);
    const bool one_slot = compact && order == IN_TURN;
    if (cfg->mode == REV_MODE_BF16) {
        Runner<bf16> r(*cfg, params, dparams, ws, one_slot, compact, order);
        r.key_len = key_len;
        return r.backward(schedule, Y1, Y2, dY1, dY2, dX1, dX2, X1o, X2o, (hipStream_t)sv, (hipStream_t)sr);
    }
    Runner<float> r(*cfg, params, dparams, ws, one_slot, compact, order);
    r.key_len = key_len;
    return r.backward(schedule, Y1, Y2, dY1, dY2, dX1, dX2, X1o, X2o, (hipStream_t)sv, (hipStream_t)sr);
}

// ---------------------------------------------------------------------------------
// file-scope scratch of the allocation-free entry point
// ---------------------------------------------------------------------------------
// The workspace of rev_stack_backward_reprop_static: every GPU the library runs on holds its own copy of this
// array from the moment the code object is loaded until the process ends.  In host code the name `scratch` is only
// a stand-in for the symbol: the device address is looked up once per device and that pointer is what the kernels get.
static __device__ __align__(256) unsigned char scratch[REV_STATIC_WORKSPACE_BYTES];

static std::mutex g_scratch_mu;
static std::vector<void*> g_scratch_ptr;     // indexed by device ordinal; nullptr = not looked up yet

// device address of `scratch` on the current device
static int scratch_address(void** out) {
    int dev = 0;
    REV_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if ((int)g_scratch_ptr.size() <= dev) g_scratch_ptr.resize(dev + 1, nullptr);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        REV_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || ((uintptr_t)p & 255) != 0) { set_error("static workspace: bad symbol address"); return REV_EHIP; }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return REV_OK;
}

}  // namespace rev

using namespace rev;

extern "C" {

int rev_stack_check_cfg(const rev_cfg* cfg) { return check_cfg(cfg); }

int64_t rev_stack_param_count(const rev_cfg* cfg) {
    int rc = check_cfg(cfg);
    if (rc) return rc;
    return block_params(*cfg) * cfg->n_blocks;
}

int64_t rev_stack_param_offset(const rev_cfg* cfg, int32_t block, int32_t tensor, int64_t* count) {
    int rc = check_cfg(cfg);
    if (rc) return rc;
    if (block < 0 || block >= cfg->n_blocks || tensor < 0 || tensor >= T_COUNT) {
        set_error("param_offset: block or tensor index out of range"); return REV_EINVAL;
    }
    if (count) *count = tensor_count(*cfg, tensor);
    return block_params(*cfg) * block + tensor_offset(*cfg, tensor);
}

int64_t rev_stack_workspace_bytes(const rev_cfg* cfg) {
    int rc = check_cfg(cfg);
    if (rc) return rc;
    return make_layout(*cfg, false).total;
}

int64_t rev_stack_workspace_bytes_reprop(const rev_cfg* cfg) {
    int rc = check_cfg(cfg);
    if (rc) return rc;
    return make_layout(*cfg, true).total;
}

int64_t rev_stack_slot_bytes(const rev_cfg* cfg) {
    int rc = check_cfg(cfg);
    if (rc) return rc;
    return make_layout(*cfg, true).slot_bytes;
}

int rev_stack_backward_order(const rev_cfg* cfg, int32_t pareprop, int64_t ws_bytes) {
    RC(check_cfg(cfg));
    if (ws_bytes < make_layout(*cfg, !pareprop).total) { set_error("backward_order: workspace too small"); return REV_EWORKSPACE; }
    return issue_order(*cfg, pareprop ? 1 : 0, ws_bytes);
}

static int forward_entry(const rev_cfg* cfg, const void* params, const float* X1, const float* X2, float* Y1, float* Y2,
                         void* ws, int64_t ws_bytes, void* stream, const int32_t* key_len) {
    RC(check_common(cfg, ws, ws_bytes, true));
    if (!params || !X1 || !X2 || !Y1 || !Y2) { set_error("a required pointer is null"); return REV_EINVAL; }
    if (!aligned16(params) || !aligned16(X1) || !aligned16(X2) || !aligned16(Y1) || !aligned16(Y2)) {
        set_error("every buffer must be 16-byte aligned"); return REV_EINVAL;
    }
    if (((uintptr_t)key_len & 3) != 0) { set_error("key_len must be 4-byte aligned"); return REV_EINVAL; }
    if (cfg->mode == REV_MODE_BF16) {
        Runner<bf16> r(*cfg, params, nullptr, ws, true, true, IN_TURN);
        r.key_len = key_len;
        return r.forward(X1, X2, Y1, Y2, (hipStream_t)stream);
    }
    Runner<float> r(*cfg, params, nullptr, ws, true, true, IN_TURN);
    r.key_len = key_len;
    return r.forward(X1, X2, Y1, Y2, (hipStream_t)stream);
}

int rev_stack_forward(const rev_cfg* cfg, const void* params, const float* X1, const float* X2, float* Y1, float* Y2,
                      void* ws, int64_t ws_bytes, void* stream) {
    return forward_entry(cfg, params, X1, X2, Y1, Y2, ws, ws_bytes, stream, nullptr);
}

int rev_stack_forward_masked(const rev_cfg* cfg, const void* params, const float* X1, const float* X2,
                             const int32_t* key_len, float* Y1, float* Y2, void* ws, int64_t ws_bytes, void* stream) {
    if (!key_len) { set_error("key_len is null"); return REV_EINVAL; }
    return forward_entry(cfg, params, X1, X2, Y1, Y2, ws, ws_bytes, stream, key_len);
}

int rev_stack_backward_reprop(const rev_cfg* cfg, const void* params, const float* Y1, const float* Y2,
                              const float* dY1, const float* dY2, float* dX1, float* dX2, float* X1_out, float* X2_out,
                              float* dparams, void* ws, int64_t ws_bytes, void* stream) {
    return backward_entry(0, cfg, params, Y1, Y2, dY1, dY2, dX1, dX2, X1_out, X2_out, dparams, ws, ws_bytes, stream, stream);
}

int rev_stack_backward_reprop_static(const rev_cfg* cfg, const void* params, const float* Y1, const float* Y2,
                                     const float* dY1, const float* dY2, float* dX1, float* dX2, float* X1_out,
                                     float* X2_out, float* dparams, void* stream) {
    RC(check_cfg(cfg));
    const int64_t need = make_layout(*cfg, true).total;
    if (need > (int64_t)REV_STATIC_WORKSPACE_BYTES) {
        set_error("static workspace too small for this shape: the sequential schedule needs " + std::to_string(need) +
                  " bytes, the built-in buffer holds " + std::to_string((int64_t)REV_STATIC_WORKSPACE_BYTES) +
                  "; use rev_stack_backward_reprop with a caller-provided workspace");
        return REV_EWORKSPACE;
    }
    void* ws = nullptr;
    RC(scratch_address(&ws));
    return backward_entry(0, cfg, params, Y1, Y2, dY1, dY2, dX1, dX2, X1_out, X2_out, dparams, ws,
                          (int64_t)REV_STATIC_WORKSPACE_BYTES, stream, stream);
}

int rev_stack_backward_pareprop(const rev_cfg* cfg, const void* params, const float* Y1, const float* Y2,
                                const float* dY1, const float* dY2, float* dX1, float* dX2, float* X1_out, float* X2_out,
                                float* dparams, void* ws, int64_t ws_bytes, void* stream_grad, void* stream_recompute) {
    return backward_entry(1, cfg, params, Y1, Y2, dY1, dY2, dX1, dX2, X1_out, X2_out, dparams, ws, ws_bytes,
                          stream_grad, stream_recompute);
}

int rev_stack_backward_reprop_masked(const rev_cfg* cfg, const void* params, const float* Y1, const float* Y2,
                                     const int32_t* key_len, const float* dY1, const float* dY2, float* dX1, float* dX2,
                                     float* X1_out, float* X2_out, float* dparams, void* ws, int64_t ws_bytes,
                                     void* stream) {
    if (!key_len) { set_error("key_len is null"); return REV_EINVAL; }
    return backward_entry(0, cfg, params, Y1, Y2, dY1, dY2, dX1, dX2, X1_out, X2_out, dparams, ws, ws_bytes, stream, stream,
                          key_len);
}

int rev_stack_backward_pareprop_masked(const rev_cfg* cfg, const void* params, const float* Y1, const float* Y2,
                                       const int32_t* key_len, const float* dY1, const float* dY2, float* dX1, float* dX2,
                                       float* X1_out, float* X2_out, float* dparams, void* ws, int64_t ws_bytes,
                                       void* stream_grad, void* stream_recompute) {
    if (!key_len) { set_error("key_len is null"); return REV_EINVAL; }
    return backward_entry(1, cfg, params, Y1, Y2, dY1, dY2, dX1, dX2, X1_out, X2_out, dparams, ws, ws_bytes,
                          stream_grad, stream_recompute, key_len);
}

int rev_stack_backward_chain(const rev_cfg* cfg, const void* params, const float* Y1, const float* Y2,
                             const float* dY1, const float* dY2, float* dX1, float* dX2, float* X1_out, float* X2_out,
                             float* dparams, void* ws, int64_t ws_bytes, void* stream, int32_t chain) {
    if (chain != 0 && chain != 1) { set_error("chain must be 0 or 1"); return REV_EINVAL; }
    return backward_entry(chain == 0 ? 2 : 3, cfg, params, Y1, Y2, dY1, dY2, dX1, dX2, X1_out, X2_out, dparams, ws,
                          ws_bytes, stream, stream);
}

int rev_sgd_step(int64_t n, float* master, void* params_bf16, const float* grad, float lr, void* stream) {
    if (n <= 0) { set_error("sgd: n must be positive"); return REV_EINVAL; }
    if (!master || !grad) { set_error("sgd: a required pointer is null"); return REV_EINVAL; }
    if (!(lr >= 0.f)) { set_error("sgd: need lr >= 0"); return REV_EINVAL; }
    if (!aligned16(master) || !aligned16(grad) || ((uintptr_t)params_bf16 & 7) != 0) {
        set_error("sgd: float32 buffers must be 16-byte aligned, the bf16 copy 8-byte aligned"); return REV_EINVAL;
    }
    return sgd_step((hipStream_t)stream, n, master, params_bf16, grad, lr);
}

int rev_adamw_step(int64_t n, float* master, void* params_bf16, const float* grad, float* m, float* v,
                   int32_t step, float lr, float beta1, float beta2, float eps, float weight_decay, void* stream) {
    if (n <= 0) { set_error("adamw: n must be positive"); return REV_EINVAL; }
    if (!master || !grad || !m || !v) { set_error("adamw: a required pointer is null"); return REV_EINVAL; }
    if (step < 1) { set_error("adamw: the step counter starts at 1"); return REV_EINVAL; }
    if (!(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps >= 0.f) || !(lr >= 0.f) ||
        !(weight_decay >= 0.f)) {
        set_error("adamw: need 0 <= beta < 1, eps >= 0, lr >= 0, weight_decay >= 0"); return REV_EINVAL;
    }
    if (!aligned16(master) || !aligned16(grad) || !aligned16(m) || !aligned16(v) || ((uintptr_t)params_bf16 & 7) != 0) {
        set_error("adamw: float32 buffers must be 16-byte aligned, the bf16 copy 8-byte aligned"); return REV_EINVAL;
    }
    return adamw_step((hipStream_t)stream, n, master, params_bf16, grad, m, v, step, lr, beta1, beta2, eps, weight_decay);
}

int rev_profile_begin(void) {
    for (auto& r : g_prof_recs) { (void)hipEventDestroy(r.e0); (void)hipEventDestroy(r.e1); }
    g_prof_recs.clear();
    for (int k = 0; k < K_COUNT; ++k) { g_prof_ms[k] = 0; g_prof_n[k] = 0; g_prof_work[k] = 0; }
    g_prof_on = true;
    return REV_OK;
}

int rev_profile_end(void) {
    g_prof_on = false;
    REV_HIP(hipDeviceSynchronize());
    for (auto& r : g_prof_recs) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, r.e0, r.e1) == hipSuccess) { g_prof_ms[r.kind] += ms; g_prof_n[r.kind] += 1; }
        (void)hipEventDestroy(r.e0);
        (void)hipEventDestroy(r.e1);
    }
    g_prof_recs.clear();
    return REV_OK;
}

int rev_profile_kinds(void) { return K_COUNT; }
const char* rev_profile_name(int kind) { return (kind >= 0 && kind < K_COUNT) ? g_kind_names[kind] : ""; }
int rev_profile_is_flops(int kind) { return (kind >= 0 && kind < K_COUNT) ? g_kind_flops[kind] : 0; }
int rev_profile_get(int kind, double* total_ms, int64_t* launches, double* work) {
    if (kind < 0 || kind >= K_COUNT) { set_error("profile_get: bad kind"); return REV_EINVAL; }
    if (total_ms) *total_ms = g_prof_ms[kind];
    if (launches) *launches = g_prof_n[kind];
    if (work) *work = g_prof_work[kind];
    return REV_OK;
}

const char* rev_last_error(void) { return g_err.c_str(); }

}  // extern "C"
