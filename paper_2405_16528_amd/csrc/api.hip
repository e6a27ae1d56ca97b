// C ABI of libloqt: argument checking, workspace layout, launch sequences, timing.
#include <math.h>
#include <string.h>

#include <algorithm>

#include "loqt_internal.h"

namespace loqt {

// ---------------------------------------------------------------------------------------
// per-kernel timing (diagnostics): events recorded around every launch while enabled
// ---------------------------------------------------------------------------------------
namespace {
struct TimingState {
    bool on = false;
    int n = 0;
    hipEvent_t* begin = nullptr;
    hipEvent_t* end = nullptr;
    int* slot = nullptr;
    int created = 0;
} g_timing;
const char* kSlotNames[SLOT_COUNT] = {"nf4_quantize", "nf4_dequantize", "gemm_u",   "gemm_y",      "gemm_z",
                                      "gemm_dx",      "gemm_db",        "reduce_db", "merge_requant", "prepass", "fold_weight",
                                      "init_requant", "init_solve_b", "merge_dense", "adam_step"};
}  // namespace

TimedLaunch::TimedLaunch(int slot_, hipStream_t s) : stream(s), slot(slot_), idx(-1) {
    if (slot_ < 0 || !g_timing.on || g_timing.n >= LOQT_TIMING_MAX_EVENTS) return;
    idx = g_timing.n++;
    if (idx >= g_timing.created) {
        (void)hipEventCreate(&g_timing.begin[idx]);
        (void)hipEventCreate(&g_timing.end[idx]);
        g_timing.created = idx + 1;
    }
    g_timing.slot[idx] = slot;
    (void)hipEventRecord(g_timing.begin[idx], stream);
}
TimedLaunch::~TimedLaunch() {
    if (idx >= 0) (void)hipEventRecord(g_timing.end[idx], stream);
}

namespace {

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

constexpr int64_t kMaxDim = (int64_t)1 << 30;  // index arithmetic inside the kernels is 32-bit per axis

loqt_status check_nf4(const loqt_nf4_mat* m) {
    if (!m || !m->codes || !m->absmax) return LOQT_INVALID_ARG;
    if (m->rows < 0 || m->cols < 0 || m->ld < 0) return LOQT_INVALID_ARG;
    if (m->rows == 0 || m->cols == 0 || m->rows > kMaxDim || m->cols > kMaxDim) return LOQT_BAD_SHAPE;
    if (m->ld % 64 != 0 || m->ld < m->cols) return LOQT_BAD_SHAPE;
    if (!aligned(m->codes, 16) || !aligned(m->absmax, 4)) return LOQT_MISALIGNED;
    return LOQT_OK;
}

loqt_status check_bf16(const void* p, int64_t rows, int64_t cols, int64_t ld) {
    if (!p) return LOQT_INVALID_ARG;
    if (rows < 0 || cols < 0 || ld < 0) return LOQT_INVALID_ARG;
    if (rows == 0 || cols == 0 || rows > kMaxDim || cols > kMaxDim) return LOQT_BAD_SHAPE;
    if (ld % 8 != 0 || ld < cols) return LOQT_BAD_SHAPE;
    if (!aligned(p, 16)) return LOQT_MISALIGNED;
    return LOQT_OK;
}

#define LOQT_TRY(expr)                     \
    do {                                   \
        loqt_status st__ = (expr);         \
        if (st__ != LOQT_OK) return st__;  \
    } while (0)
#define LOQT_HIP(expr)                                    \
    do {                                                  \
        if ((expr) != hipSuccess) return LOQT_LAUNCH_FAILED; \
    } while (0)

// shapes of the layer: W out x in, P out x r
loqt_status check_layer(const loqt_nf4_mat* Wq, const loqt_nf4_mat* Pq, const void* B, int64_t ld_B) {
    LOQT_TRY(check_nf4(Wq));
    LOQT_TRY(check_nf4(Pq));
    if (Pq->rows != Wq->rows) return LOQT_BAD_SHAPE;
    LOQT_TRY(check_bf16(B, Pq->cols, Wq->cols, ld_B));
    return LOQT_OK;
}

// ---------------------------------------------------------------------------------------
// Two implementations of every call: "fused" (NF4 expanded inside the GEMM's operand staging,
// no pre-pass; best when few tokens share a weight tile) and "prepass" (NF4 expanded to bf16
// once per call, then plain NT GEMMs; best from about a thousand tokens up).
// ---------------------------------------------------------------------------------------
int g_path = LOQT_PATH_AUTO;

// Forward and backward: measured on 768^2 ... 11008x4096 weights, the pre-pass family is ahead of the fused
// form at every token count from 16 up (the fused GEMM pays the NF4 expansion once per 256-token tile row
// and its main loop is slower), so AUTO never picks the fused form there; it stays selectable.
bool use_prepass(int64_t /*tokens*/) {
    return g_path != LOQT_PATH_FUSED;
}
// Forward with a handful of tokens: the codes are streamed once and expanded in registers (few.hip), no copy of the weight.
bool use_few_tokens(int64_t tokens) { return g_path == LOQT_PATH_AUTO && tokens <= FEW_TOKENS_MAX; }
// Merge: a weight of 1024 columns or more always takes the pre-pass form (and so has to come with a workspace); a narrower
// one takes it if the caller brought the workspace (narrow_merge_prepass).
bool use_prepass_merge(int64_t in) {
    if (g_path == LOQT_PATH_FUSED) return false;
    if (g_path != LOQT_PATH_AUTO) return true;
    return in >= 1024;
}

// Within the pre-pass family: carry the rank-r term through every token as a second K segment
// (2 T r (in + out) flop per pass) or fold it into the bf16 copy of the weight once per call
// (W_eff = deq(W) + s deq(P) B, 2 out in r flop).  Folding wins from T = out in / (in + out) up.
bool use_folded(int64_t T, int64_t out, int64_t in) {
    if (g_path == LOQT_PATH_FOLDED) return true;
    if (g_path != LOQT_PATH_AUTO) return false;
    return T * (in + out) >= out * in;  // measured: still ahead at the break-even of the flop counts
}

// Backward pass: Z = s dy deq(P) exists anyway (dB needs it), so carrying the rank-r term as a second K segment of
// the dx product costs only 2 T r in flop at the rate of the large products, against 2 out in r flop at the rate of
// the fold (about half of that: short contraction, heavy epilogue) -- cheaper when the weight has many more rows
// than the step has tokens.  Measured rates put the break-even near out = 0.73 T (7B gate / up at 8192 tokens and
// every projection of the 13B block at 4096 tokens take the second-segment form, the square 7B projections fold).
bool use_folded_bwd(int64_t T, int64_t out, int64_t in) {
    if (!use_folded(T, out, in)) return false;
    if (g_path != LOQT_PATH_AUTO) return true;
    return (double)out <= 0.73 * (double)T;
}

// A few hundred tokens that do not fold: the codes are expanded inside the products (nf4_tile.hip) and no copy of the
// weight is made.  That pays for a weight whose copy costs more than the slower loop, the more so the more tokens there are, and
// where the contraction (in; backward out) is long enough for the prologues of a k-tile's pipeline not to count.  In the backward
// pass the copies win more often: they go out beside nothing else, the products of dx fill the chip (the more the wider the weight)
// and the gradient shares their launch.  Time of the backward call with the codes against with copies, means over random weights
// (2700 calls of 0.4 to 80 million elements, ranks 32 to 1024), by out (lines) and in:
//   up to 32 tokens  512   1024  2048  4096  8192    33..64     512   1024  2048  4096  8192
//   724..1023        1.37  1.30  1.25  1.17  1.09               1.43  1.38  1.28  1.24  1.18
//   1024..1447       1.19  1.15  0.95  0.96  1.09               1.19  1.10  1.09  1.10  1.17
//   1448..2047       1.02  1.01  0.95  0.86  1.01               1.00  0.97  0.96  1.01  1.12
//   2048..2895       1.08  0.94  0.89  0.81  1.02               0.98  0.96  0.91  0.90  1.06
//   4096..5791       0.93  0.85  0.80  0.82  0.84               0.87  0.92  0.86  0.83  0.87
//   65..128                                          129..256
//   2048..2895       1.12  1.07  0.99  1.11  1.10               1.27  1.25  1.33  1.30  1.26
//   2896..4095       1.06  1.02  0.99  1.03  1.03               1.21  1.21  1.18  1.17  1.16
//   4096..5791       1.01  1.00  0.96  0.91  0.92               1.28  1.18  1.13  1.14  1.04
//   5792..8191       1.02  1.02  0.95  0.86  0.86               1.27  1.20  1.06  0.94  1.06
//   8192..11584      1.07  0.96  0.89  0.82                     1.22  1.16  1.00  0.93  1.00
// Forward (2170 calls, 33 tokens and more) it is the size of the weight, in / out counting for little.  A copy of P is made or not
// with that of W, so a high rank counts towards the codes.  65 tokens take tiles of 128.  The lines below leave calls 0.21 % (forward) and
// 0.31 % (backward) above the better of the two on the mean, 1.4 % and 2.4 % of them by more than 5 %; lines by steps of T and of one side,
// which they replace, 0.35 % and 0.49 %, 2.5 % and 3.9 % (forward, 50 tokens, 6080 x 1024, rank 882, 22.2 us with the codes, 25.5 with
// copies; backward, 10 tokens, 1280 x 4864, rank 807, 27.4 and 32.3).
bool use_nf4_tile(int64_t T, int64_t out, int64_t in, int64_t r, bool backward) {
    if (T > 256) return false;
    if (g_path == LOQT_PATH_CODES) return true;
    if (g_path != LOQT_PATH_AUTO || use_folded(T, out, in)) return false;
    if (!backward)
        return (double)out * ((double)in + 0.5 * (double)r) >= (double)(2000000 + 50000 * T) * pow((double)out / (double)in, 0.1);
    const int64_t least = T <= 64 ? 1250 + 7 * T : std::min<int64_t>(5500, 2600 + 40 * (T - 64));
    return 2 * out + r >= 2 * least && out * in >= std::max<int64_t>(1500000, 200000 * T - 10000000) &&
           64 * in <= std::max<int64_t>(256, 416 - 3 * T) * out;
}

inline size_t bf16_bytes(int64_t rows, int64_t cols) {
    return round_up((size_t)rows * (size_t)round_up(cols, 8) * 2, 256);
}
size_t bwd_z_bytes(int64_t T, int64_t r) { return bf16_bytes(T, r); }

// Workspace layouts of the pre-pass family.  Products take their operands in whichever orientation
// they are stored (rows x K or K x rows), so nothing is ever transposed: the only pre-passes are NF4
// expansions, one per NF4 operand and call.
// A product that leaves compute units idle runs in fp32 slices of its contraction (plan_nt in gemm_nt.hip), and the
// slices live in the workspace.  loqt_workspace_bytes counts room for the best plan; a call accepts less, down to
// `least`, and then plans with the slices it has room for.  `least` holds the slices of dB (M x N outputs, contraction
// K) that this older estimate asks for, in k-tile steps.
int least_splits(int64_t M, int64_t N, int64_t K) {
    auto cdiv = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    const bool wide = M >= 512;
    const int64_t tiles = wide ? cdiv(M, 256) * cdiv(N, 128) : cdiv(M, 128) * cdiv(N, 128);
    const int64_t slots = wide ? 256 : 512;
    const int64_t nkt = cdiv(K, 64);
    const double per_slice = (double)M * (double)N * 8.0 / 12.0e6;
    int best = 1;
    double best_cost = 0.0;
    for (int s = 1; s <= 16; ++s) {
        if (s > 1 && nkt / s < 8) break;
        const double cost = (double)cdiv(tiles * s, slots) * ((double)cdiv(nkt, s) + 6.0) + per_slice * s;
        if (s == 1 || cost < best_cost) best = s, best_cost = cost;
    }
    return best;
}
// ... and, for Z = s dy deq(P) (T x r outputs, contraction over `out`), two slices where its 256x128 tiles number
// 64 to 128
int least_z_splits(int64_t T, int64_t out, int64_t r) {
    if (T < 512 || out < 2048) return 1;
    const int64_t tiles = ((T + 255) / 256) * ((r + 127) / 128);
    return (tiles >= 64 && tiles <= 128) ? 2 : 1;
}
// slices of an M x N sum over K of which `room` bytes hold the fp32 values (pitch ldp)
int planned_splits(int64_t M, int64_t N, int64_t K, int64_t ldp, size_t room) {
    const int64_t fit = (int64_t)(room / ((size_t)M * (size_t)ldp * 4));
    return plan_nt(M, N, (K + 63) / 64, true, 1, (int)std::min<int64_t>(std::max<int64_t>(fit, 1), NT_MAX_SPLITS)).splits;
}
size_t slices_bytes(int64_t splits, int64_t M, int64_t ldp) { return round_up((size_t)splits * (size_t)M * (size_t)ldp * 4, 256); }

// The layouts below take the size of the workspace at hand; ALL: the size that loqt_workspace_bytes asks for.
constexpr size_t ALL = ~(size_t)0;

// Pitch of the bf16 copy of the weight: rows that start on a cache line (128 bytes) where the workspace has room for it.
// (x of 5461 columns at a pitch of 5464 makes every 128-byte piece of a row span two lines; the weight need not as well.)
struct Region {
    size_t at, end;
    int64_t ld;
};
Region weight_region(size_t at, int64_t rows, int64_t cols, size_t rest, size_t ws_bytes) {
    const int64_t wide = (int64_t)round_up(cols, 64), ld = at + bf16_bytes(rows, wide) + rest <= ws_bytes ? wide : (int64_t)round_up(cols, 8);
    return Region{at, at + bf16_bytes(rows, ld), ld};
}

// `saved`: the caller keeps W_eff in a buffer of its own (loqt_linear_fwd_save / loqt_linear_bwd_saved), so the
// workspace holds no copy of the weight (and the forward pass, always folded then, no U)
struct FwdWs {
    size_t U, Wb, Pb, split, least, total;  // U = s x B^T; Wb = deq(W) or W_eff; Pb = deq(P); slices of U, then of y
    int64_t ldw;
    FwdWs(int64_t T, int64_t out, int64_t in, int64_t r, bool saved, size_t ws_bytes) {
        U = 0;
        Wb = U + (saved ? 0 : bf16_bytes(T, r));
        const size_t rest = bf16_bytes(out, r), remainder = round_up((size_t)remainder_split_floats(T, out) * 4, 256);
        const Region w = weight_region(Wb, out, in, rest + remainder, ws_bytes);
        ldw = w.ld;
        Pb = saved ? Wb : w.end;
        split = Pb + rest;
        least = Wb + (saved ? 0 : bf16_bytes(out, in)) + rest + remainder;
        total = least;
        if (ws_bytes == ALL) {
            // (whichever form runs: the size does not depend on the path option)
            int64_t most = product_split_floats(T, out, in, 0);
            if (!saved) most = std::max({most, product_split_floats(T, r, in, 0), product_split_floats(T, out, in, r)});
            total = std::max(split + remainder, split + round_up((size_t)most * 4, 256));
        }
    }
};
struct BwdWs {
    size_t Z, Wb, Pb, partials, least, total;  // Z = s dy deq(P); Wb = deq(W) or W_eff; Pb = deq(P); fp32 slices
    int64_t ldw, ldp;
    BwdWs(int64_t T, int64_t out, int64_t in, int64_t r, bool saved, size_t ws_bytes) {
        Z = 0;
        Wb = Z + bf16_bytes(T, r);
        ldp = (int64_t)round_up(in, 4);
        const int64_t ldzp = (int64_t)round_up(r, 4);
        // the slices of Z are summed into Z before those of dx are written, and both before the dB product writes
        // its own: one region serves all three
        const int least_z = least_z_splits(T, out, r);
        const size_t rest = bf16_bytes(out, r);
        const size_t least_slices = std::max({slices_bytes(least_splits(r, in, T), r, ldp),
                                              least_z > 1 ? slices_bytes(least_z, T, ldzp) : (size_t)0,
                                              round_up((size_t)remainder_split_floats(T, in) * 4, 256)});
        const Region w = weight_region(Wb, out, in, rest + least_slices, ws_bytes);
        ldw = w.ld;
        Pb = saved ? Wb : w.end;
        partials = Pb + rest;
        least = Wb + (saved ? 0 : bf16_bytes(out, in)) + rest + least_slices;
        total = least;
        if (ws_bytes == ALL) {
            const int64_t most = std::max({product_split_floats(T, in, out, 0), product_split_floats(T, in, out, r),
                                           product_split_floats(T, r, out, 0)});
            total = partials + std::max({least_slices, slices_bytes(planned_splits(r, in, T, ldp, ALL), r, ldp),
                                         round_up((size_t)most * 4, 256)});
        }
    }
};
struct MergeWs {
    size_t Pb, total;
    MergeWs(int64_t out, int64_t in, int64_t r) {
        (void)in;
        Pb = 0;
        total = Pb + bf16_bytes(out, r);
    }
};

// compensation loop: Pb = bf16(P) (out x r), E = W - deq(Q_c) (out x round_up(in, 64), bf16),
// fp32 slices of B = P^T E over the contraction along `out`
struct InitWs {
    size_t Pb, E, partials, least, total;
    int64_t ldp, lde, ldr;
    InitWs(int64_t out, int64_t in, int64_t r) {
        ldr = (int64_t)round_up(r, 8);
        lde = (int64_t)round_up(in, 64);
        ldp = (int64_t)round_up(in, 4);
        Pb = 0;
        E = Pb + round_up((size_t)out * (size_t)ldr * 2, 256);
        partials = E + round_up((size_t)out * (size_t)lde * 2, 256);
        least = partials + slices_bytes(least_splits(r, in, out), r, ldp);
        total = std::max(least, partials + slices_bytes(planned_splits(r, in, out, ldp, ALL), r, ldp));
    }
};

// LoQT-nq: U or Z (T x r) first, then the dB slices (backward), then room for the folded weight W_eff (out x in, bf16),
// whether or not the path option makes this call fold, then the slices of U or Z and of y or dx
struct NqWs {
    size_t partials, We, split, least, total;  // least: for a call that folds
    int64_t ldw, ldp;
    NqWs(bool bwd, int64_t T, int64_t out, int64_t in, int64_t r, size_t ws_bytes) {
        partials = bf16_bytes(T, r);
        ldp = (int64_t)round_up(in, 4);
        // the region of the dB slices is as large as loqt_linear_bwd's least workspace makes it
        size_t slices = 0;
        if (bwd) {
            const BwdWs L(T, out, in, r, true, 0);
            slices = L.least - L.partials;
        }
        We = partials + slices;
        const Region w = weight_region(We, out, in, 0, ws_bytes);
        ldw = w.ld;
        split = w.end;
        least = We + bf16_bytes(out, in);
        total = least;
        if (ws_bytes == ALL) {
            int64_t most;
            if (bwd) most = std::max({product_split_floats(T, r, out, 0), product_split_floats(T, in, out, 0),
                                      product_split_floats(T, in, out, r), planned_splits(r, in, T, ldp, ALL) * r * ldp});
            else most = std::max({product_split_floats(T, r, in, 0), product_split_floats(T, out, in, 0),
                                  product_split_floats(T, out, in, r)});
            total = split + round_up((size_t)most * 4, 256);
        }
    }
};

// right-side variant (W + s Bp Q^T): Qb = deq(Q) (in x r), We = folded weight (out x in), V = s x Qb
// (T x r), fp32 slices of dBp = dy^T V over the contraction along T
struct RightWs {
    size_t Qb, We, V, partials, least, total;  // partials: slices of V, of y or dx, of dBp, one after the other
    int64_t ldr, ldw, ldp;
    RightWs(int op, int64_t T, int64_t out, int64_t in, int64_t r, size_t ws_bytes) {
        ldr = (int64_t)round_up(r, 8);
        ldp = (int64_t)round_up(r, 4);
        Qb = 0;
        We = Qb + bf16_bytes(in, r);
        const bool weight = op != LOQT_OP_MERGE_RIGHT, bwd = op == LOQT_OP_BWD_RIGHT;
        const size_t v = bwd ? bf16_bytes(T, r) : 0, least_slices = bwd ? slices_bytes(least_splits(out, r, T), out, ldp) : 0;
        const Region w = weight_region(We, out, in, v + least_slices, ws_bytes);
        ldw = w.ld;
        V = weight ? w.end : We;
        partials = V + v;
        least = We + (weight ? bf16_bytes(out, in) : 0) + v + least_slices;
        total = least;
        if (ws_bytes == ALL && weight) {
            int64_t most = bwd ? std::max(product_split_floats(T, r, in, 0), product_split_floats(T, in, out, 0))
                               : product_split_floats(T, out, in, 0);
            total = partials + std::max({least_slices, round_up((size_t)most * 4, 256),
                                         bwd ? slices_bytes(planned_splits(out, r, T, ldp, ALL), out, ldp) : (size_t)0});
        }
    }
};

// shapes of the right-side layer: W out x in, Q in x r, Bp out x r
loqt_status check_layer_right(const loqt_nf4_mat* Wq, const loqt_nf4_mat* Qq, const void* Bp, int64_t ld_Bp) {
    LOQT_TRY(check_nf4(Wq));
    LOQT_TRY(check_nf4(Qq));
    if (Qq->rows != Wq->cols) return LOQT_BAD_SHAPE;
    LOQT_TRY(check_bf16(Bp, Wq->rows, Qq->cols, ld_Bp));
    return LOQT_OK;
}

Operand nf4_operand(const loqt_nf4_mat* m, int rows, int K) {
    Operand o;
    o.ptr = m->codes;
    o.absmax = m->absmax;
    o.ld = m->ld;
    o.rows = rows;
    o.K = K;
    return o;
}
Operand bf16_operand(const void* p, int64_t ld, int rows, int K) {
    Operand o;
    o.ptr = p;
    o.absmax = nullptr;
    o.ld = ld;
    o.rows = rows;
    o.K = K;
    return o;
}
Operand no_operand() {
    Operand o;
    memset(&o, 0, sizeof(o));
    return o;
}

// whether the n bytes at p and the nq at q have none in common
bool apart(const void* p, size_t n, const void* q, size_t nq) {
    return (uintptr_t)p + n <= (uintptr_t)q || (uintptr_t)q + nq <= (uintptr_t)p;
}
size_t span_bytes(int64_t rows, int64_t cols, int64_t ld, size_t size) { return (size_t)((rows - 1) * ld + cols) * size; }
// ... the n bytes at p and a bf16 operand (rc: stored K x rows)
bool apart_from(const void* p, size_t n, const Operand& o, bool rc) {
    return o.K == 0 || apart(p, n, o.ptr, rc ? span_bytes(o.K, o.rows, o.ld, 2) : span_bytes(o.rows, o.K, o.ld, 2));
}
// A fold or merge that reads P as its codes reads them while others of its work-groups store: none of the n bytes it writes may
// be P's.
bool apart_from(const void* p, size_t n, const loqt_nf4_mat* Pq) {
    return apart(p, n, Pq->codes, (size_t)Pq->rows * (Pq->ld / 2)) && apart(p, n, Pq->absmax, (size_t)Pq->rows * (Pq->ld / 64) * 4);
}

// W_eff[out x in] (bf16, pitch ldw) = deq(Wq) + s * deq(Pq) B; Pb receives deq(Pq) in bf16
// (dequant_p; else it is there).  z: a product that goes out with the fold, reading Pb too, or null
loqt_status fold_weight(const loqt_nf4_mat* Wq, const loqt_nf4_mat* Pq, const loqt_bf16* B, int64_t ld_B, float s,
                        uint16_t* Pb, uint16_t* We, int64_t ldw, bool dequant_p, const GemmParams* z, hipStream_t st) {
    const int64_t out = Wq->rows, in = Wq->cols, r = Pq->cols;
    const int64_t ldr = (int64_t)round_up(r, 8);
    const bool from_codes = dequant_p && g_path == LOQT_PATH_AUTO && weight_takes_codes(out, in, r) &&
                            apart_from(We, (size_t)out * ldw * 2, Pq);
    if (dequant_p && !from_codes)
        LOQT_HIP(launch_dequantize(Pq->codes, Pq->absmax, out, r, Pq->ld, Pb, LOQT_BF16, ldr, st, SLOT_PREPASS));
    GemmParams p;
    memset(&p, 0, sizeof(p));
    p.A[0] = from_codes ? nf4_operand(Pq, (int)out, (int)r) : bf16_operand(Pb, ldr, (int)out, (int)r);  // out x r, K contiguous
    p.B[0] = bf16_operand(B, ld_B, (int)in, (int)r);    // r x in: K x rows
    p.M = (int)out;
    p.N = (int)in;
    p.alpha = s;
    p.C = We;
    p.ldc = ldw;
    p.w_codes = Wq->codes;
    p.w_absmax = Wq->absmax;
    p.w_ld = Wq->ld;
    p.w_cols = (int)in;
    if (z) LOQT_HIP(launch_z_fold(SLOT_GEMM_Z, *z, SLOT_FOLD, EPI_FOLD, true, p, st));
    else LOQT_HIP(launch_gemm_nt(SLOT_FOLD, EPI_FOLD, false, true, p, st));
    return LOQT_OK;
}

// bf16 copies of the weight and of P in one launch (two cost a launch more and leave P, a small one, alone on the chip; whole
// forward calls with 300 tokens, us, two / one: 512 x 512, rank 128, 17.2 / 16.7; 4096 x 4096, rank 1024, 64.1 / 60.2;
// 13824 x 5120, rank 1024, 131.5 / 129.3)
// u: U = s x B^T, which goes out with them, or null.
hipError_t expand_weight(const loqt_nf4_mat* Wq, uint16_t* Wb, int64_t ldw, const loqt_nf4_mat* Pq, uint16_t* Pb, int64_t ldp,
                         const GemmParams* u, hipStream_t st) {
    const DequantGroupItem both[2] = {{Wq->codes, Wq->absmax, Wb, Wq->rows, Wq->ld, ldw, (int)Wq->cols},
                                      {Pq->codes, Pq->absmax, Pb, Pq->rows, Pq->ld, ldp, (int)Pq->cols}};
    return u ? launch_u_copies(SLOT_GEMM_U, *u, both, st) : launch_dequantize_grouped(both, 2, st, SLOT_PREPASS);
}

// U = s x B^T for a handful of tokens, where it has a launch of its own.  Its r rows make few work-groups (64 at rank 1024), each reading all of x, so a
// long contraction goes out in slices instead, which find room where a copy of the weight would be.  Both forms timed in whole
// calls of both layers (1024 and 4096 rows, rank 64 to 1024, contractions of 1024 to 13824): slices are ahead from 5500 (1
// token), 4600 (8) and 3500 (16) on, with the second token tile from 2800 (17) and 2050 (32).  At 4096 and 16 tokens they save
// 0.9 us of 24, at 8192 and 32 tokens 12.7 us.  A contraction that ends inside a k-tile costs them 2 to 4 us more (rows that
// start off cache lines; 5461: -1.7 us at 4 tokens, -0.4 at 16, 2.6 at 32), which is 2000 of contraction.
hipError_t launch_u_few(GemmParams& p, float* split_ws, size_t split_bytes, hipStream_t st) {
    const int line = (p.M <= 16 ? 5632 - 128 * p.M : 3584 - 48 * p.M) + (p.A[0].K % 64 ? 2000 : 0);
    const bool room = split_bytes >= (size_t)8 * p.M * round_up(p.N, 4) * 4;  // (one slice alone would be slower still)
    if ((p.A[0].K <= line || !room) && p.N <= FEW_ROWS_MAX_BF16) return launch_few_tokens(SLOT_GEMM_U, false, p, st);
    p.split_ws = split_ws;
    p.split_ws_floats = (int64_t)(split_bytes / 4);
    return launch_gemm_nt(SLOT_GEMM_U, EPI_BF16, false, false, p, st);
}

// dB[M x N] (fp32 or bf16, pitch ld_dB) = sum of the planned slices of Z^T x and its relatives (both operands K x rows), or,
// accumulating, that much more.  One slice that need not be added to anything goes straight to dB (rank 1024, 5120
// columns, 256 tokens: a launch of 7 us less).  dx: the product of dx, which goes out with it, or null.  The caller's dB may lie
// over an input: it is written in a launch that reads it as well only where they have no byte in common.
hipError_t gradient_product(int slot, GemmParams p, float* part, size_t part_bytes, int64_t ldp, void* dB, int dB_dtype,
                            int64_t ld_dB, int accumulate, const GemmParams* dx, hipStream_t st) {
    auto go = [&](int epi) {
        return dx ? launch_dx_gradient(SLOT_GEMM_DX, *dx, slot, epi, p, st) : launch_gemm_nt(slot, epi, true, true, p, st);
    };
    p.splits = planned_splits(p.M, p.N, p.A[0].K, ldp, part_bytes);
    const bool bf16 = dB_dtype == LOQT_BF16;
    const size_t n = span_bytes(p.M, p.N, ld_dB, bf16 ? 2 : 4);
    if (p.splits == 1 && !accumulate && g_nt_tile_override == 0 && ld_dB % (bf16 ? 8 : 4) == 0 && aligned(dB, 16) &&
        apart_from(dB, n, p.A[0], true) && apart_from(dB, n, p.B[0], true)) {
        if (dx && !(apart_from(dB, n, dx->A[0], false) && apart_from(dB, n, dx->A[1], false) && apart_from(dB, n, dx->B[0], true) &&
                    apart_from(dB, n, dx->B[1], true) && apart(dB, n, dx->C, span_bytes(dx->M, dx->N, dx->ldc, 2)))) {
            hipError_t e = launch_gemm_nt(SLOT_GEMM_DX, EPI_BF16, false, true, *dx, st);
            if (e != hipSuccess) return e;
            dx = nullptr;
        }
        p.C = dB;
        p.ldc = ld_dB;
        return go(bf16 ? EPI_BF16 : EPI_F32_SPLITK);
    }
    p.C = part;
    p.ldc = ldp;
    hipError_t e = go(EPI_F32_SPLITK);
    if (e != hipSuccess) return e;
    return launch_reduce_db(part, p.splits, p.M, p.N, ldp, dB, dB_dtype, ld_dB, accumulate, st);
}

// Slices that fit: fp32 M x N at a pitch that is a multiple of 4
int64_t slices_that_fit(int64_t M, int64_t N, size_t bytes) { return (int64_t)(bytes / ((size_t)M * round_up(N, 4) * 4)); }

// C[M x N] (bf16) = alpha * the product that launch_nf4_tile makes of p, in slices at `ws`
loqt_status nf4_product(int slot, bool b_rc, GemmParams p, uint16_t* C, int64_t ldc, float* ws, size_t ws_bytes,
                        hipStream_t st) {
    const int64_t nkt = (p.A[0].K + 63) / 64 + (b_rc ? 0 : (p.A[1].K + 63) / 64), ld = (int64_t)round_up(p.N, 4);
    const int extra = b_rc && p.A[1].K > 0 ? 1 : 0;
    p.splits = nf4_tile_splits(p.M, p.N, nkt, extra, slices_that_fit(p.M, p.N, ws_bytes) - extra);
    p.C = ws;
    p.ldc = ld;
    TimedLaunch tl(slot, st);  // the product and the sum of its slices
    LOQT_HIP(launch_nf4_tile(b_rc, p, st));
    LOQT_HIP(launch_reduce_db(ws, p.splits + extra, p.M, p.N, ld, C, LOQT_BF16, ldc, 0, st, false));
    return LOQT_OK;
}

loqt_status merge_fused(const loqt_nf4_mat* Wq, uint8_t* codes_out, float* absmax_out,
                        const loqt_nf4_mat* Pq, const loqt_bf16* B, int64_t ld_B, float s, hipStream_t st) {
    const int out = (int)Wq->rows, in = (int)Wq->cols, r = (int)Pq->cols;
    GemmParams p;
    memset(&p, 0, sizeof(p));
    // transposed product: rows of the tile run along `in`; the grid reaches the padding
    // columns cols..ld-1 as well (operand rows past `in` read as zero)
    p.A[0] = bf16_operand(B, ld_B, in, r);  // B is r x in: K x rows
    p.B[0] = nf4_operand(Pq, out, r);       // P is out x r: rows x K
    p.M = (int)Wq->ld;
    p.N = out;
    p.alpha = s;
    p.w_codes = Wq->codes;
    p.w_absmax = Wq->absmax;
    p.out_codes = codes_out;
    p.out_absmax = absmax_out;
    p.w_ld = Wq->ld;
    p.w_cols = in;
    LOQT_HIP(launch_gemm(GEMM_MERGE, p, st));
    return LOQT_OK;
}

bool outputs_apart(const uint8_t* codes_out, const float* absmax_out, const loqt_nf4_mat* Wq, const loqt_nf4_mat* Pq) {
    return apart_from(codes_out, (size_t)Wq->rows * (Wq->ld / 2), Pq) && apart_from(absmax_out, (size_t)Wq->rows * (Wq->ld / 64) * 4, Pq);
}

loqt_status merge_prepass(const loqt_nf4_mat* Wq, uint8_t* codes_out, float* absmax_out,
                          const loqt_nf4_mat* Pq, const loqt_bf16* B, int64_t ld_B, float s, void* ws,
                          hipStream_t st) {
    const int64_t out = Wq->rows, in = Wq->cols, r = Pq->cols;
    const MergeWs L(out, in, r);
    uint16_t* Pb = reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(ws) + L.Pb);
    const int64_t ldr = (int64_t)round_up(r, 8);
    const bool from_codes = g_path == LOQT_PATH_AUTO && weight_takes_codes(out, Wq->ld, r) && outputs_apart(codes_out, absmax_out, Wq, Pq);
    if (!from_codes)
        LOQT_HIP(launch_dequantize(Pq->codes, Pq->absmax, out, r, Pq->ld, Pb, LOQT_BF16, ldr, st, SLOT_PREPASS));
    GemmParams p;
    memset(&p, 0, sizeof(p));
    p.A[0] = from_codes ? nf4_operand(Pq, (int)out, (int)r) : bf16_operand(Pb, ldr, (int)out, (int)r);  // rows of the tile are rows of W
    p.B[0] = bf16_operand(B, ld_B, (int)in, (int)r);   // r x in: K x rows, columns run along `in`
    p.M = (int)out;
    p.N = (int)Wq->ld;  // reach the padding columns (operand columns past `in` are never used)
    p.alpha = s;
    p.w_codes = Wq->codes;
    p.w_absmax = Wq->absmax;
    p.out_codes = codes_out;
    p.out_absmax = absmax_out;
    p.w_ld = Wq->ld;
    p.w_cols = (int)in;
    LOQT_HIP(launch_gemm_nt(SLOT_MERGE, EPI_MERGE, false, true, p, st));
    return LOQT_OK;
}

size_t merge_ws_bytes(int64_t out, int64_t in, int64_t r) { return MergeWs(out, in, r).total; }

// A narrow weight may come without a workspace (the fused form needs none); with one it takes the pre-pass form as well
// (same bits; 2048 x 768, rank 256: 15.4 -> 11.8 us)
bool narrow_merge_prepass(const loqt_nf4_mat* Wq, const loqt_nf4_mat* Pq, const void* ws, size_t ws_bytes) {
    return g_path == LOQT_PATH_AUTO && ws && aligned(ws, 256) && ws_bytes >= merge_ws_bytes(Wq->rows, Wq->cols, Pq->cols);
}

loqt_status merge_checked(const loqt_nf4_mat* Wq, uint8_t* codes_out, float* absmax_out,
                          const loqt_nf4_mat* Pq, const loqt_bf16* B, int64_t ld_B, float s, void* ws, size_t ws_bytes,
                          hipStream_t st) {
    if (use_prepass_merge(Wq->cols) || narrow_merge_prepass(Wq, Pq, ws, ws_bytes))
        return merge_prepass(Wq, codes_out, absmax_out, Pq, B, ld_B, s, ws, st);
    return merge_fused(Wq, codes_out, absmax_out, Pq, B, ld_B, s, st);
}

loqt_status check_merge_ws(const loqt_nf4_mat* Wq, const loqt_nf4_mat* Pq, void* ws, size_t ws_bytes) {
    if (!use_prepass_merge(Wq->cols)) return LOQT_OK;
    if (!ws) return LOQT_INVALID_ARG;
    if (!aligned(ws, 256)) return LOQT_MISALIGNED;
    if (ws_bytes < merge_ws_bytes(Wq->rows, Wq->cols, Pq->cols)) return LOQT_WORKSPACE_TOO_SMALL;
    return LOQT_OK;
}

// full aliasing of the merge output with its input is allowed, partial overlap is not
loqt_status check_out_alias(const loqt_nf4_mat* Wq, const uint8_t* codes_out, const float* absmax_out) {
    const size_t cb = (size_t)Wq->rows * (size_t)(Wq->ld / 2), ab = (size_t)Wq->rows * (size_t)(Wq->ld / 64) * 4;
    const uint8_t* ci = Wq->codes;
    const uint8_t* ai = reinterpret_cast<const uint8_t*>(Wq->absmax);
    const uint8_t* ao = reinterpret_cast<const uint8_t*>(absmax_out);
    if (codes_out != ci && codes_out < ci + cb && ci < codes_out + cb) return LOQT_INVALID_ARG;
    if (ao != ai && ao < ai + ab && ai < ao + ab) return LOQT_INVALID_ARG;
    return LOQT_OK;
}

loqt_status check_merge(const loqt_nf4_mat* Wq, uint8_t* codes_out, float* absmax_out,
                        const loqt_nf4_mat* Pq, const loqt_bf16* B, int64_t ld_B) {
    if (!codes_out || !absmax_out) return LOQT_INVALID_ARG;
    LOQT_TRY(check_layer(Wq, Pq, B, ld_B));
    if (!aligned(codes_out, 16) || !aligned(absmax_out, 4)) return LOQT_MISALIGNED;
    return check_out_alias(Wq, codes_out, absmax_out);
}

}  // namespace
}  // namespace loqt

using namespace loqt;

extern "C" {

const char* loqt_status_string(loqt_status st) {
    switch (st) {
        case LOQT_OK: return "LOQT_OK";
        case LOQT_INVALID_ARG: return "LOQT_INVALID_ARG";
        case LOQT_BAD_SHAPE: return "LOQT_BAD_SHAPE";
        case LOQT_MISALIGNED: return "LOQT_MISALIGNED";
        case LOQT_WORKSPACE_TOO_SMALL: return "LOQT_WORKSPACE_TOO_SMALL";
        case LOQT_LAUNCH_FAILED: return "LOQT_LAUNCH_FAILED";
        case LOQT_STATIC_SCRATCH_TOO_SMALL: return "LOQT_STATIC_SCRATCH_TOO_SMALL";
    }
    return "LOQT_UNKNOWN_STATUS";
}

loqt_status nf4_quantize(const float* w, int64_t rows, int64_t cols, int64_t ld_w, uint8_t* codes,
                         float* absmax, int64_t ld_q, void* hip_stream) {
    if (!w || !codes || !absmax) return LOQT_INVALID_ARG;
    if (rows < 0 || cols < 0 || ld_w < 0 || ld_q < 0) return LOQT_INVALID_ARG;
    if (rows == 0 || cols == 0 || rows > kMaxDim || cols > kMaxDim) return LOQT_BAD_SHAPE;
    if (ld_w % 4 != 0 || ld_w < cols || ld_q % 64 != 0 || ld_q < cols) return LOQT_BAD_SHAPE;
    if (!aligned(w, 16) || !aligned(codes, 16) || !aligned(absmax, 4)) return LOQT_MISALIGNED;
    LOQT_HIP(launch_quantize(w, rows, cols, ld_w, codes, absmax, ld_q, (hipStream_t)hip_stream));
    return LOQT_OK;
}

loqt_status nf4_dequantize(const uint8_t* codes, const float* absmax, int64_t rows, int64_t cols,
                           int64_t ld_q, void* out, int out_dtype, int64_t ld_out, void* hip_stream) {
    if (!codes || !absmax || !out) return LOQT_INVALID_ARG;
    if (out_dtype != LOQT_F32 && out_dtype != LOQT_BF16) return LOQT_INVALID_ARG;
    if (rows < 0 || cols < 0 || ld_q < 0 || ld_out < 0) return LOQT_INVALID_ARG;
    if (rows == 0 || cols == 0 || rows > kMaxDim || cols > kMaxDim) return LOQT_BAD_SHAPE;
    if (ld_q % 64 != 0 || ld_q < cols || ld_out < cols) return LOQT_BAD_SHAPE;
    if (ld_out % (out_dtype == LOQT_BF16 ? 8 : 4) != 0) return LOQT_BAD_SHAPE;
    if (!aligned(codes, 16) || !aligned(absmax, 4) || !aligned(out, 16)) return LOQT_MISALIGNED;
    LOQT_HIP(launch_dequantize(codes, absmax, rows, cols, ld_q, out, out_dtype, ld_out,
                               (hipStream_t)hip_stream));
    return LOQT_OK;
}

size_t loqt_workspace_bytes(int op, int64_t T, int64_t out, int64_t in, int64_t r) {
    if (out <= 0 || in <= 0 || r <= 0) return 0;
    // enough for either implementation, so that the size does not depend on the path option
    switch (op) {
        case LOQT_OP_FWD: {
            if (T <= 0) return 0;
            return FwdWs(T, out, in, r, false, ALL).total;  // the fused path needs only its first part (U)
        }
        case LOQT_OP_BWD: {
            if (T <= 0) return 0;
            const size_t fused = bwd_z_bytes(T, r) + round_up((size_t)gemm_db_splits(T, r, in) * (size_t)r * (size_t)in * 4, 256);
            const size_t pre = BwdWs(T, out, in, r, false, ALL).total;
            return fused > pre ? fused : pre;
        }
        case LOQT_OP_FWD_SAVE: return T <= 0 ? 0 : FwdWs(T, out, in, r, true, ALL).total;
        case LOQT_OP_BWD_SAVED: return T <= 0 ? 0 : BwdWs(T, out, in, r, true, ALL).total;
        case LOQT_OP_MERGE: return merge_ws_bytes(out, in, r);
        case LOQT_OP_INIT: return InitWs(out, in, r).total;
        case LOQT_OP_FWD_RIGHT:
        case LOQT_OP_BWD_RIGHT:
            if (T <= 0) return 0;
            return RightWs(op, T, out, in, r, ALL).total;
        case LOQT_OP_MERGE_RIGHT: return RightWs(op, 0, out, in, r, ALL).total;
        case LOQT_OP_FWD_NQ: return T <= 0 ? 0 : NqWs(false, T, out, in, r, ALL).total;
        case LOQT_OP_BWD_NQ: return T <= 0 ? 0 : NqWs(true, T, out, in, r, ALL).total;
        default: return 0;
    }
}

// save_weff != NULL: the folded form is used whatever the path option says and W_eff goes to the caller's
// buffer (pitch ld_save) instead of the workspace
static loqt_status fwd_impl(const loqt_bf16* x, int64_t ld_x, int64_t T, const loqt_nf4_mat* Wq,
                            const loqt_nf4_mat* Pq, const loqt_bf16* B, int64_t ld_B, float s, loqt_bf16* y,
                            int64_t ld_y, loqt_bf16* save_weff, int64_t ld_save, void* ws, size_t ws_bytes,
                            void* hip_stream) {
    LOQT_TRY(check_layer(Wq, Pq, B, ld_B));
    const int64_t out = Wq->rows, in = Wq->cols, r = Pq->cols;
    LOQT_TRY(check_bf16(x, T, in, ld_x));
    LOQT_TRY(check_bf16(y, T, out, ld_y));
    if (!ws) return LOQT_INVALID_ARG;
    if (!aligned(ws, 256)) return LOQT_MISALIGNED;
    const FwdWs L(T, out, in, r, save_weff != nullptr, ws_bytes);
    if (ws_bytes < L.least) return LOQT_WORKSPACE_TOO_SMALL;
    hipStream_t st = (hipStream_t)hip_stream;
    const int64_t ld_u = (int64_t)round_up(r, 8);
    loqt_bf16* U = reinterpret_cast<loqt_bf16*>(ws);
    GemmParams p;

    if (save_weff) LOQT_TRY(check_bf16(save_weff, out, in, ld_save));
    if (!save_weff && use_few_tokens(T)) {
        memset(&p, 0, sizeof(p));  // U = s x B^T
        p.A[0] = bf16_operand(x, ld_x, (int)T, (int)in);
        p.B[0] = bf16_operand(B, ld_B, (int)r, (int)in);
        p.M = (int)T;
        p.N = (int)r;
        p.alpha = s;
        p.C = U;
        p.ldc = ld_u;
        float* const room = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + L.Wb);
        if (few_layer_fits((int)T, (int)out, (int)in, (int)r, ws_bytes - L.Wb)) {
            GemmParams w, q;
            memset(&w, 0, sizeof(w));
            w.A[0] = bf16_operand(x, ld_x, (int)T, (int)in);
            w.B[0] = nf4_operand(Wq, (int)out, (int)in);
            w.M = (int)T;
            w.N = (int)out;
            w.split_ws = room;
            q = w;
            q.A[0] = bf16_operand(U, ld_u, (int)T, (int)r);
            q.B[0] = nf4_operand(Pq, (int)out, (int)r);
            q.alpha = 1.0f;
            q.C = y;
            q.ldc = ld_y;
            LOQT_HIP(launch_few_layer(p, w, q, st));
            return LOQT_OK;
        }
        LOQT_HIP(launch_u_few(p, room, ws_bytes - L.Wb, st));
        memset(&p, 0, sizeof(p));  // y = x deq(W)^T + U deq(P)^T
        p.A[0] = bf16_operand(x, ld_x, (int)T, (int)in);
        p.B[0] = nf4_operand(Wq, (int)out, (int)in);
        p.A[1] = bf16_operand(U, ld_u, (int)T, (int)r);
        p.B[1] = nf4_operand(Pq, (int)out, (int)r);
        p.M = (int)T;
        p.N = (int)out;
        p.alpha = 1.0f;
        p.C = y;
        p.ldc = ld_y;
        LOQT_HIP(launch_few_tokens(SLOT_GEMM_Y, true, p, st));
        return LOQT_OK;
    }
    // (the slices go where the copy of the weight would be)
    char* const slices = reinterpret_cast<char*>(ws) + L.Wb;
    const size_t slices_room = ws_bytes - L.Wb;
    if (!save_weff && use_nf4_tile(T, out, in, r, false) && slices_that_fit(T, out, slices_room) >= 1) {
        memset(&p, 0, sizeof(p));  // U = s x B^T
        p.A[0] = bf16_operand(x, ld_x, (int)T, (int)in);
        p.B[0] = bf16_operand(B, ld_B, (int)r, (int)in);
        p.M = (int)T;
        p.N = (int)r;
        p.alpha = s;
        p.C = U;
        p.ldc = ld_u;
        p.split_ws = reinterpret_cast<float*>(slices);
        p.split_ws_floats = (int64_t)(slices_room / 4);
        LOQT_HIP(launch_gemm_nt(SLOT_GEMM_U, EPI_BF16, false, false, p, st));
        memset(&p, 0, sizeof(p));  // y = x deq(W)^T + U deq(P)^T
        p.A[0] = bf16_operand(x, ld_x, (int)T, (int)in);
        p.B[0] = nf4_operand(Wq, (int)out, (int)in);
        p.A[1] = bf16_operand(U, ld_u, (int)T, (int)r);
        p.B[1] = nf4_operand(Pq, (int)out, (int)r);
        p.M = (int)T;
        p.N = (int)out;
        p.alpha = 1.0f;
        return nf4_product(SLOT_GEMM_Y, false, p, y, ld_y, reinterpret_cast<float*>(slices), slices_room, st);
    }
    if (save_weff || use_prepass(T)) {
        char* base = reinterpret_cast<char*>(ws);
        uint16_t* Wb = save_weff ? save_weff : reinterpret_cast<uint16_t*>(base + L.Wb);
        uint16_t* Pb = reinterpret_cast<uint16_t*>(base + L.Pb);
        const int64_t ldw = save_weff ? ld_save : L.ldw;
        const bool folded = save_weff || use_folded(T, out, in);
        if (folded) {
            // y = x W_eff^T with W_eff = deq(W) + s deq(P) B folded once per call
            LOQT_TRY(fold_weight(Wq, Pq, B, ld_B, s, Pb, Wb, ldw, true, nullptr, st));
        } else {
            // U = s x B^T
            memset(&p, 0, sizeof(p));
            p.A[0] = bf16_operand(x, ld_x, (int)T, (int)in);
            p.B[0] = bf16_operand(B, ld_B, (int)r, (int)in);
            p.M = (int)T;
            p.N = (int)r;
            p.alpha = s;
            p.C = U;
            p.ldc = ld_u;
            p.split_ws = reinterpret_cast<float*>(base + L.split);
            p.split_ws_floats = (int64_t)((ws_bytes - L.split) / 4);
            LOQT_HIP(expand_weight(Wq, Wb, ldw, Pq, Pb, ld_u, &p, st));
        }
        // y = x Wb^T (+ U deq(P)^T when the rank-r term is not folded into Wb)
        memset(&p, 0, sizeof(p));
        p.A[0] = bf16_operand(x, ld_x, (int)T, (int)in);
        p.B[0] = bf16_operand(Wb, ldw, (int)out, (int)in);
        if (!folded) {
            p.A[1] = bf16_operand(U, ld_u, (int)T, (int)r);
            p.B[1] = bf16_operand(Pb, ld_u, (int)out, (int)r);
        }
        p.M = (int)T;
        p.N = (int)out;
        p.alpha = 1.0f;
        p.C = y;
        p.ldc = ld_y;
        p.split_ws = reinterpret_cast<float*>(base + L.split);
        p.split_ws_floats = (int64_t)((ws_bytes - L.split) / 4);
        LOQT_HIP(launch_gemm_nt(SLOT_GEMM_Y, EPI_BF16, false, false, p, st));
        return LOQT_OK;
    }

    memset(&p, 0, sizeof(p));
    // U = s x B^T
    p.A[0] = bf16_operand(x, ld_x, (int)T, (int)in);
    p.B[0] = bf16_operand(B, ld_B, (int)r, (int)in);
    p.M = (int)T;
    p.N = (int)r;
    p.alpha = s;
    p.C = U;
    p.ldc = ld_u;
    LOQT_HIP(launch_gemm(GEMM_U, p, st));
    // y = x deq(W)^T + U deq(P)^T
    memset(&p, 0, sizeof(p));
    p.A[0] = bf16_operand(x, ld_x, (int)T, (int)in);
    p.B[0] = nf4_operand(Wq, (int)out, (int)in);
    p.A[1] = bf16_operand(U, ld_u, (int)T, (int)r);
    p.B[1] = nf4_operand(Pq, (int)out, (int)r);
    p.M = (int)T;
    p.N = (int)out;
    p.alpha = 1.0f;
    p.C = y;
    p.ldc = ld_y;
    LOQT_HIP(launch_gemm(GEMM_Y, p, st));
    return LOQT_OK;
}

loqt_status loqt_linear_fwd(const loqt_bf16* x, int64_t ld_x, int64_t T, const loqt_nf4_mat* Wq,
                            const loqt_nf4_mat* Pq, const loqt_bf16* B, int64_t ld_B, float s,
                            loqt_bf16* y, int64_t ld_y, void* ws, size_t ws_bytes, void* hip_stream) {
    return fwd_impl(x, ld_x, T, Wq, Pq, B, ld_B, s, y, ld_y, nullptr, 0, ws, ws_bytes, hip_stream);
}

loqt_status loqt_linear_fwd_save(const loqt_bf16* x, int64_t ld_x, int64_t T, const loqt_nf4_mat* Wq,
                                 const loqt_nf4_mat* Pq, const loqt_bf16* B, int64_t ld_B, float s, loqt_bf16* y,
                                 int64_t ld_y, loqt_bf16* w_eff, int64_t ld_weff, void* ws, size_t ws_bytes,
                                 void* hip_stream) {
    if (!w_eff) return LOQT_INVALID_ARG;
    return fwd_impl(x, ld_x, T, Wq, Pq, B, ld_B, s, y, ld_y, w_eff, ld_weff, ws, ws_bytes, hip_stream);
}

// saved != NULL: W_eff (out x in_saved, bf16, pitch ld_saved) was produced by loqt_linear_fwd_save with the same
// W_q, P_q, B and s; it replaces the fold, and Wq / B are not looked at
static loqt_status bwd_impl(const loqt_bf16* dy, int64_t ld_dy, const loqt_bf16* x, int64_t ld_x, int64_t T,
                            const loqt_nf4_mat* Wq, const loqt_nf4_mat* Pq, const loqt_bf16* B, int64_t ld_B,
                            float s, loqt_bf16* dx, int64_t ld_dx, void* dB, int dB_dtype, int64_t ld_dB,
                            int accumulate, const loqt_bf16* saved, int64_t ld_saved, int64_t in_saved, void* ws,
                            size_t ws_bytes, void* hip_stream) {
    if (saved) {
        LOQT_TRY(check_nf4(Pq));
        if (in_saved < 0) return LOQT_INVALID_ARG;
        LOQT_TRY(check_bf16(saved, Pq->rows, in_saved, ld_saved));
    } else {
        LOQT_TRY(check_layer(Wq, Pq, B, ld_B));
    }
    const int64_t out = Pq->rows, in = saved ? in_saved : Wq->cols, r = Pq->cols;
    LOQT_TRY(check_bf16(dy, T, out, ld_dy));
    LOQT_TRY(check_bf16(x, T, in, ld_x));
    if (dx) LOQT_TRY(check_bf16(dx, T, in, ld_dx));
    if (!dB) return LOQT_INVALID_ARG;
    if (dB_dtype != LOQT_F32 && dB_dtype != LOQT_BF16) return LOQT_INVALID_ARG;
    if (ld_dB < in) return LOQT_BAD_SHAPE;
    if (!aligned(dB, dB_dtype == LOQT_BF16 ? 2 : 4)) return LOQT_MISALIGNED;
    if (!ws) return LOQT_INVALID_ARG;
    if (!aligned(ws, 256)) return LOQT_MISALIGNED;
    const BwdWs L(T, out, in, r, saved != nullptr, ws_bytes);
    // (the fused form sums as many slices as it likes, in a workspace laid out Z, slices)
    const size_t fused = bwd_z_bytes(T, r) + round_up((size_t)gemm_db_splits(T, r, in) * (size_t)r * (size_t)in * 4, 256);
    if (ws_bytes < (saved ? L.least : std::max(L.least, fused))) return LOQT_WORKSPACE_TOO_SMALL;
    hipStream_t st = (hipStream_t)hip_stream;
    const int64_t ld_z = (int64_t)round_up(r, 8);
    loqt_bf16* Z = reinterpret_cast<loqt_bf16*>(ws);
    float* partials = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + bwd_z_bytes(T, r));

    GemmParams p, pz, pdx;  // pz, pdx: products that go out together with a later one
    bool dx_later = false;
    if (saved || use_prepass(T)) {
        char* base = reinterpret_cast<char*>(ws);
        const uint16_t* Wb = saved ? saved : reinterpret_cast<const uint16_t*>(base + L.Wb);
        uint16_t* Pb = reinterpret_cast<uint16_t*>(base + L.Pb);
        float* part = reinterpret_cast<float*>(base + L.partials);
        const int64_t part_floats = (int64_t)((ws_bytes - L.partials) / 4);
        const int64_t ldw = saved ? ld_saved : L.ldw;
        // a few hundred tokens: Z and dx straight from the codes, their slices where the copies of W and P would be
        const size_t room = ws_bytes - L.Wb;
        const bool tile = !saved && use_nf4_tile(T, out, in, r, true) && slices_that_fit(T, r, room) >= 1 &&
                          slices_that_fit(T, in, room) >= 2;
        if (tile) {
            memset(&p, 0, sizeof(p));
            p.A[0] = bf16_operand(dy, ld_dy, (int)T, (int)out);
            p.B[0] = nf4_operand(Pq, (int)r, (int)out);
            p.M = (int)T;
            p.N = (int)r;
            p.alpha = s;
            float* const sl = reinterpret_cast<float*>(base + L.Wb);
            LOQT_TRY(nf4_product(SLOT_GEMM_Z, true, p, Z, ld_z, sl, room, st));
            if (dx) {
                p.B[0] = nf4_operand(Wq, (int)in, (int)out);
                p.N = (int)in;
                p.alpha = 1.0f;
                p.A[1] = bf16_operand(Z, ld_z, (int)T, (int)r);
                p.B[1] = bf16_operand(B, ld_B, (int)in, (int)r);
                LOQT_TRY(nf4_product(SLOT_GEMM_DX, true, p, dx, ld_dx, sl, room, st));
            }
        } else {
        const bool folded = dx && (saved || use_folded_bwd(T, out, in));
        if (dx && !folded) LOQT_HIP(expand_weight(Wq, reinterpret_cast<uint16_t*>(base + L.Wb), ldw, Pq, Pb, ld_z, nullptr, st));
        else LOQT_HIP(launch_dequantize(Pq->codes, Pq->absmax, out, r, Pq->ld, Pb, LOQT_BF16, ld_z, st, SLOT_PREPASS));
        // Z rides along with dx (one product [dx | Z] over the shared operand dy) when that is estimated to
        // take less time than the two launches: its tiles then fill a partly empty round of the dx product
        bool z_with_dx = false;
        if (folded) {
            const int64_t tm = (T + 255) / 256;
            const int64_t t_dx = tm * ((in + 255) / 256), t_z = tm * ((r + 255) / 256);
            const int64_t kt = (out + 63) / 64;
            const NtPlan z = plan_nt(T, r, kt, false, 1, NT_MAX_SPLITS);
            if (out >= 2048) {
                // in rounds of 256x256 tiles (a k-tile of such a round: 1.56 us); Z alone on those when they fill the chip,
                // else by plan_nt
                const double z_alone = t_z >= 224 ? plan_bf16_product(T, r, 0).cost : z.cost / (1.56 * (double)kt + 8.0);
                z_with_dx = t_dx >= 224 && plan_bf16_product(T, in, r).cost < plan_bf16_product(T, in, 0).cost + z_alone;
            } else {
                // contractions too short for those tiles: where dx runs on 128x128, a Z that needs no further round of them
                // costs nothing beside it (saved backward, us, Z alone / beside dx: 3021 tokens, 81 x 6892, rank 21, 49.9 /
                // 45.4; 1539 tokens, 128 x 8640, rank 128, 39.4 / 35.4; but 1605 tokens, 2029 x 10791, rank 8, whose dx is
                // better off on 256x128, 123 / 128)
                const NtPlan d = plan_nt(T, in, kt, false, 1, NT_MAX_SPLITS);
                z_with_dx = t_dx >= 224 && d.tile == NT_128x128 && d.splits == 1 && joint_cost_128(T, in, r, kt) < d.cost + z.cost;
            }
        }
        if (!z_with_dx) {
            // Z = s dy deq(P): deq(P) is out x r, i.e. K x rows
            memset(&p, 0, sizeof(p));
            p.A[0] = bf16_operand(dy, ld_dy, (int)T, (int)out);
            p.B[0] = bf16_operand(Pb, ld_z, (int)r, (int)out);
            p.M = (int)T;
            p.N = (int)r;
            p.alpha = s;
            p.C = Z;
            p.ldc = ld_z;
            p.split_ws = part;
            p.split_ws_floats = part_floats;
            pz = p;
            if (!folded || saved) LOQT_HIP(launch_gemm_nt(SLOT_GEMM_Z, EPI_BF16, false, true, p, st));
        }
        if (dx) {
            // dx = dy Wb (+ Z B when the rank-r term is not folded into Wb); Wb is out x in: K x rows
            uint16_t* Wws = reinterpret_cast<uint16_t*>(base + L.Wb);
            if (folded && !saved) LOQT_TRY(fold_weight(Wq, Pq, B, ld_B, s, Pb, Wws, ldw, false, z_with_dx ? nullptr : &pz, st));
            memset(&p, 0, sizeof(p));
            p.A[0] = bf16_operand(dy, ld_dy, (int)T, (int)out);
            p.B[0] = bf16_operand(Wb, ldw, (int)in, (int)out);
            if (!folded) {
                p.A[1] = bf16_operand(Z, ld_z, (int)T, (int)r);
                p.B[1] = bf16_operand(B, ld_B, (int)in, (int)r);  // r x in: K x rows
            }
            p.M = (int)T;
            p.N = (int)in;
            p.alpha = 1.0f;
            p.C = dx;
            p.ldc = ld_dx;
            if (z_with_dx) {  // [dx | Z] = dy [W_eff | s deq(P)]
                p.Bx = bf16_operand(Pb, ld_z, (int)r, (int)out);
                p.Nx = (int)r;
                p.alphax = s;
                p.Cx = Z;
                p.ldcx = ld_z;
            }
            p.split_ws = part;  // (the slices of Z, if any, have been summed by now; those of dB come later)
            p.split_ws_floats = part_floats;
            if (z_with_dx) LOQT_HIP(launch_gemm_nt(SLOT_GEMM_DX, EPI_BF16, false, true, p, st));
            else pdx = p, dx_later = true;
        }
        }
        // dB = Z^T x: Z is T x r and x is T x in, both K x rows; contraction over T in slices
        memset(&p, 0, sizeof(p));
        p.A[0] = bf16_operand(Z, ld_z, (int)r, (int)T);
        p.B[0] = bf16_operand(x, ld_x, (int)in, (int)T);
        p.M = (int)r;
        p.N = (int)in;
        p.alpha = 1.0f;
        LOQT_HIP(gradient_product(SLOT_GEMM_DB, p, part, ws_bytes - L.partials, L.ldp, dB, dB_dtype, ld_dB, accumulate,
                                  dx_later ? &pdx : nullptr, st));
        return LOQT_OK;
    }
    memset(&p, 0, sizeof(p));
    // Z = s dy deq(P)
    p.A[0] = bf16_operand(dy, ld_dy, (int)T, (int)out);
    p.B[0] = nf4_operand(Pq, (int)r, (int)out);  // P is out x r: K x rows
    p.M = (int)T;
    p.N = (int)r;
    p.alpha = s;
    p.C = Z;
    p.ldc = ld_z;
    LOQT_HIP(launch_gemm(GEMM_Z, p, st));
    if (dx) {
        // dx = dy deq(W) + Z B
        memset(&p, 0, sizeof(p));
        p.A[0] = bf16_operand(dy, ld_dy, (int)T, (int)out);
        p.B[0] = nf4_operand(Wq, (int)in, (int)out);  // W is out x in: K x rows
        p.A[1] = bf16_operand(Z, ld_z, (int)T, (int)r);
        p.B[1] = bf16_operand(B, ld_B, (int)in, (int)r);  // B is r x in: K x rows
        p.M = (int)T;
        p.N = (int)in;
        p.alpha = 1.0f;
        p.C = dx;
        p.ldc = ld_dx;
        LOQT_HIP(launch_gemm(GEMM_DX, p, st));
    }
    // dB = Z^T x, contraction over T split into a fixed number of slices
    memset(&p, 0, sizeof(p));
    p.A[0] = bf16_operand(Z, ld_z, (int)r, (int)T);   // Z is T x r: K x rows
    p.B[0] = bf16_operand(x, ld_x, (int)in, (int)T);  // x is T x in: K x rows
    p.M = (int)r;
    p.N = (int)in;
    p.alpha = 1.0f;
    p.C = partials;
    p.splits = gemm_db_splits(T, r, in);
    LOQT_HIP(launch_gemm(GEMM_DB, p, st));
    LOQT_HIP(launch_reduce_db(partials, p.splits, r, in, in, dB, dB_dtype, ld_dB, accumulate, st));
    return LOQT_OK;
}

loqt_status loqt_linear_bwd(const loqt_bf16* dy, int64_t ld_dy, const loqt_bf16* x, int64_t ld_x, int64_t T,
                            const loqt_nf4_mat* Wq, const loqt_nf4_mat* Pq, const loqt_bf16* B, int64_t ld_B,
                            float s, loqt_bf16* dx, int64_t ld_dx, void* dB, int dB_dtype, int64_t ld_dB,
                            int accumulate, void* ws, size_t ws_bytes, void* hip_stream) {
    return bwd_impl(dy, ld_dy, x, ld_x, T, Wq, Pq, B, ld_B, s, dx, ld_dx, dB, dB_dtype, ld_dB, accumulate, nullptr,
                    0, 0, ws, ws_bytes, hip_stream);
}

loqt_status loqt_linear_bwd_saved(const loqt_bf16* dy, int64_t ld_dy, const loqt_bf16* x, int64_t ld_x, int64_t T,
                                  const loqt_nf4_mat* Pq, int64_t in, float s, const loqt_bf16* w_eff,
                                  int64_t ld_weff, loqt_bf16* dx, int64_t ld_dx, void* dB, int dB_dtype,
                                  int64_t ld_dB, int accumulate, void* ws, size_t ws_bytes, void* hip_stream) {
    if (!w_eff) return LOQT_INVALID_ARG;
    return bwd_impl(dy, ld_dy, x, ld_x, T, nullptr, Pq, nullptr, 0, s, dx, ld_dx, dB, dB_dtype, ld_dB, accumulate,
                    w_eff, ld_weff, in, ws, ws_bytes, hip_stream);
}

loqt_status loqt_merge_requant(const loqt_nf4_mat* Wq, uint8_t* codes_out, float* absmax_out,
                               const loqt_nf4_mat* Pq, const loqt_bf16* B, int64_t ld_B, float s, void* ws,
                               size_t ws_bytes, void* hip_stream) {
    LOQT_TRY(check_merge(Wq, codes_out, absmax_out, Pq, B, ld_B));
    LOQT_TRY(check_merge_ws(Wq, Pq, ws, ws_bytes));
    return merge_checked(Wq, codes_out, absmax_out, Pq, B, ld_B, s, ws, ws_bytes, (hipStream_t)hip_stream);
}

loqt_status loqt_merge_requant_batched(int n_layers, const loqt_merge_desc* descs, void* ws, size_t ws_bytes,
                                       void* hip_stream) {
    if (n_layers < 0 || (n_layers > 0 && !descs)) return LOQT_INVALID_ARG;
    for (int i = 0; i < n_layers; ++i) {
        LOQT_TRY(check_merge(&descs[i].Wq, descs[i].codes_out, descs[i].absmax_out, &descs[i].Pq, descs[i].B,
                             descs[i].ld_B));
        LOQT_TRY(check_merge_ws(&descs[i].Wq, &descs[i].Pq, ws, ws_bytes));
    }
    // Layers that take the pre-pass form go out in groups: one launch expands the P_q of the group into the
    // workspace, one launch runs the merge tiles of all its layers.  A group holds as many consecutive layers as
    // the workspace has room for (at most MERGE_GROUP_MAX); with the minimum workspace that is one layer at a
    // time, the same kernels, the same bits.  Layers on the fused form (narrow weights that come without room for
    // their P_q) run one by one.
    hipStream_t st = (hipStream_t)hip_stream;
    int i = 0;
    while (i < n_layers) {
        auto prepass = [&](const loqt_merge_desc& d) {
            return use_prepass_merge(d.Wq.cols) || narrow_merge_prepass(&d.Wq, &d.Pq, ws, ws_bytes);
        };
        if (!prepass(descs[i])) {
            LOQT_TRY(merge_checked(&descs[i].Wq, descs[i].codes_out, descs[i].absmax_out, &descs[i].Pq, descs[i].B,
                                   descs[i].ld_B, descs[i].s, ws, ws_bytes, st));
            ++i;
            continue;
        }
        MergeGroupLayer layers[MERGE_GROUP_MAX];
        DequantGroupItem deq[MERGE_GROUP_MAX];
        int n = 0;
        size_t used = 0;
        int64_t most_r = 0, tiles = 0;
        bool apart = true;
        while (i + n < n_layers && n < MERGE_GROUP_MAX && prepass(descs[i + n])) {
            const loqt_merge_desc& d = descs[i + n];
            const int64_t out = d.Wq.rows, in = d.Wq.cols, r = d.Pq.cols;
            const size_t need = merge_ws_bytes(out, in, r);
            if (n > 0 && used + need > ws_bytes) break;
            uint16_t* Pb = reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(ws) + used);
            const int64_t ldr = (int64_t)round_up(r, 8);
            deq[n] = DequantGroupItem{d.Pq.codes, d.Pq.absmax, Pb, out, d.Pq.ld, ldr, (int)r};
            layers[n] = MergeGroupLayer{Pb, nullptr, d.B, ldr, d.ld_B, d.Wq.codes, d.Wq.absmax, d.codes_out, d.absmax_out,
                                        d.Wq.ld, (int)out, (int)in, (int)r, d.s};
            used += need;
            most_r = std::max(most_r, r);
            tiles += codes_tiles(out, d.Wq.ld);
            ++n;
        }
        for (int a = 0; a < n; ++a)
            for (int b = 0; b < n; ++b)
                apart = apart && outputs_apart(descs[i + a].codes_out, descs[i + a].absmax_out, &descs[i + a].Wq, &descs[i + b].Pq);
        if (apart && g_path == LOQT_PATH_AUTO && group_takes_codes(most_r, tiles)) {
            for (int k = 0; k < n; ++k)
                layers[k].A = deq[k].codes, layers[k].A_absmax = deq[k].absmax, layers[k].lda = deq[k].ld_q;
        } else {
            LOQT_HIP(launch_dequantize_grouped(deq, n, st, SLOT_PREPASS));
        }
        LOQT_HIP(launch_merge_grouped(SLOT_MERGE, layers, n, st));
        i += n;
    }
    return LOQT_OK;
}

size_t loqt_merge_batched_workspace_bytes(int n_layers, const loqt_merge_desc* descs) {
    if (n_layers <= 0 || !descs) return 0;
    // the largest sum over MERGE_GROUP_MAX consecutive layers: with that much every group is full
    size_t best = 0;
    for (int i = 0; i < n_layers; ++i) {
        size_t sum = 0;
        for (int k = i; k < n_layers && k < i + MERGE_GROUP_MAX; ++k)
            sum += merge_ws_bytes(descs[k].Wq.rows, descs[k].Wq.cols, descs[k].Pq.cols);
        best = std::max(best, sum);
    }
    return best;
}

int loqt_resolved_path(int op, int64_t T, int64_t out, int64_t in) {
    if (op == LOQT_OP_MERGE) return use_prepass_merge(in) ? LOQT_PATH_PREPASS : LOQT_PATH_FUSED;
    if (!use_prepass(T) || (op == LOQT_OP_FWD && use_few_tokens(T))) return LOQT_PATH_FUSED;
    if (op == LOQT_OP_BWD) return use_folded_bwd(T, out, in) ? LOQT_PATH_FOLDED : LOQT_PATH_PREPASS;
    return use_folded(T, out, in) ? LOQT_PATH_FOLDED : LOQT_PATH_PREPASS;
}

int loqt_expands_codes(int op, int64_t T, int64_t out, int64_t in, int64_t r) {
    if (T <= 0 || out <= 0 || in <= 0 || r <= 0) return 0;
    if (op == LOQT_OP_FWD) return !use_few_tokens(T) && use_nf4_tile(T, out, in, r, false);
    return op == LOQT_OP_BWD && use_nf4_tile(T, out, in, r, true);
}

loqt_status loqt_init_compensate(const float* W, int64_t ld_w, const float* P, int64_t ld_p, int64_t out,
                                 int64_t in, int64_t r, float s, int iters, int warm_start, uint8_t* codes_out,
                                 float* absmax_out, int64_t ld_q, loqt_bf16* B, int64_t ld_B, void* ws,
                                 size_t ws_bytes, void* hip_stream) {
    if (!W || !P || !codes_out || !absmax_out) return LOQT_INVALID_ARG;
    if (out < 0 || in < 0 || r < 0 || ld_w < 0 || ld_p < 0 || ld_q < 0) return LOQT_INVALID_ARG;
    if (iters < 1 || (warm_start != 0 && warm_start != 1)) return LOQT_INVALID_ARG;
    if (!(s > 0.f) || !(s <= 3.0e38f)) return LOQT_INVALID_ARG;  // also rejects NaN
    if (out == 0 || in == 0 || r == 0 || out > kMaxDim || in > kMaxDim || r > kMaxDim) return LOQT_BAD_SHAPE;
    if (ld_w % 4 != 0 || ld_w < in || ld_p % 4 != 0 || ld_p < r) return LOQT_BAD_SHAPE;
    if (ld_q % 64 != 0 || ld_q < in) return LOQT_BAD_SHAPE;
    LOQT_TRY(check_bf16(B, r, in, ld_B));
    if (!aligned(W, 16) || !aligned(P, 16) || !aligned(codes_out, 16) || !aligned(absmax_out, 4))
        return LOQT_MISALIGNED;
    if (!ws) return LOQT_INVALID_ARG;
    if (!aligned(ws, 256)) return LOQT_MISALIGNED;
    const InitWs L(out, in, r);
    if (ws_bytes < L.least) return LOQT_WORKSPACE_TOO_SMALL;
    const int splits = planned_splits(r, in, out, L.ldp, ws_bytes - L.partials);
    hipStream_t st = (hipStream_t)hip_stream;
    char* base = reinterpret_cast<char*>(ws);
    uint16_t* Pb = reinterpret_cast<uint16_t*>(base + L.Pb);
    uint16_t* E = reinterpret_cast<uint16_t*>(base + L.E);
    float* part = reinterpret_cast<float*>(base + L.partials);

    LOQT_HIP(launch_f32_to_bf16(P, out, r, ld_p, Pb, L.ldr, st));
    GemmParams p;
    for (int c = 0; c < iters; ++c) {
        // Q_c = q_NF4(W - s P B) and E = W - deq(Q_c); the first step of a cold start has B = 0
        const bool with_product = c > 0 || warm_start;
        memset(&p, 0, sizeof(p));
        p.A[0] = bf16_operand(Pb, L.ldr, (int)out, with_product ? (int)r : 0);  // out x r, K contiguous
        p.B[0] = bf16_operand(B, ld_B, (int)in, with_product ? (int)r : 0);     // r x in: K x rows
        p.M = (int)out;
        p.N = (int)ld_q;  // reach the padding columns of the code matrix
        p.alpha = -s;
        p.out_codes = codes_out;
        p.out_absmax = absmax_out;
        p.w_ld = ld_q;
        p.w_cols = (int)in;
        p.w_f32 = W;
        p.w_f32_ld = ld_w;
        p.e_out = E;
        p.e_ld = L.lde;
        LOQT_HIP(launch_gemm_nt(SLOT_INIT_Q, EPI_COMP, false, true, p, st));
        // B = P^T E / s: P is out x r and E is out x in, both K x rows; contraction over `out` in slices
        memset(&p, 0, sizeof(p));
        p.A[0] = bf16_operand(Pb, L.ldr, (int)r, (int)out);
        p.B[0] = bf16_operand(E, L.lde, (int)in, (int)out);
        p.M = (int)r;
        p.N = (int)in;
        p.alpha = 1.0f / s;
        p.C = part;
        p.ldc = L.ldp;
        p.splits = splits;
        LOQT_HIP(launch_gemm_nt(SLOT_INIT_B, EPI_F32_SPLITK, true, true, p, st));
        LOQT_HIP(launch_reduce_db(part, splits, r, in, L.ldp, B, LOQT_BF16, ld_B, 0, st));
    }
    return LOQT_OK;
}

// ---------------------------------------------------------------------------------------
// right-side projection variant: W_eff = deq(W_q) + s Bp deq(Q_q)^T
// ---------------------------------------------------------------------------------------
namespace {
// Qb = deq(Qq) (bf16, in x r) and We = deq(Wq) + s Bp Qb^T (bf16, out x in, pitch ldw)
loqt_status fold_weight_right(const loqt_nf4_mat* Wq, const loqt_nf4_mat* Qq, const loqt_bf16* Bp, int64_t ld_Bp,
                              float s, uint16_t* Qb, int64_t ldr, uint16_t* We, int64_t ldw, const GemmParams* v, hipStream_t st) {
    const int64_t out = Wq->rows, in = Wq->cols, r = Qq->cols;
    GemmParams p;
    memset(&p, 0, sizeof(p));
    p.A[0] = bf16_operand(Bp, ld_Bp, (int)out, (int)r);  // out x r, K contiguous
    p.B[0] = bf16_operand(Qb, ldr, (int)in, (int)r);     // in x r: rows x K, K contiguous
    p.M = (int)out;
    p.N = (int)in;
    p.alpha = s;
    p.C = We;
    p.ldc = ldw;
    p.w_codes = Wq->codes;
    p.w_absmax = Wq->absmax;
    p.w_ld = Wq->ld;
    p.w_cols = (int)in;
    if (v) LOQT_HIP(launch_z_fold(SLOT_GEMM_U, *v, SLOT_FOLD, EPI_FOLD, false, p, st));
    else LOQT_HIP(launch_gemm_nt(SLOT_FOLD, EPI_FOLD, false, false, p, st));
    return LOQT_OK;
}
loqt_status check_ws(void* ws, size_t ws_bytes, size_t need) {
    if (!ws) return LOQT_INVALID_ARG;
    if (!aligned(ws, 256)) return LOQT_MISALIGNED;
    if (ws_bytes < need) return LOQT_WORKSPACE_TOO_SMALL;
    return LOQT_OK;
}
}  // namespace

loqt_status loqt_linear_fwd_right(const loqt_bf16* x, int64_t ld_x, int64_t T, const loqt_nf4_mat* Wq,
                                  const loqt_nf4_mat* Qq, const loqt_bf16* Bp, int64_t ld_Bp, float s,
                                  loqt_bf16* y, int64_t ld_y, void* ws, size_t ws_bytes, void* hip_stream) {
    LOQT_TRY(check_layer_right(Wq, Qq, Bp, ld_Bp));
    const int64_t out = Wq->rows, in = Wq->cols, r = Qq->cols;
    LOQT_TRY(check_bf16(x, T, in, ld_x));
    LOQT_TRY(check_bf16(y, T, out, ld_y));
    const RightWs L(LOQT_OP_FWD_RIGHT, T, out, in, r, ws_bytes);
    LOQT_TRY(check_ws(ws, ws_bytes, L.least));
    hipStream_t st = (hipStream_t)hip_stream;
    char* base = reinterpret_cast<char*>(ws);
    uint16_t* Qb = reinterpret_cast<uint16_t*>(base + L.Qb);
    uint16_t* We = reinterpret_cast<uint16_t*>(base + L.We);
    LOQT_HIP(launch_dequantize(Qq->codes, Qq->absmax, in, r, Qq->ld, Qb, LOQT_BF16, L.ldr, st, SLOT_PREPASS));
    LOQT_TRY(fold_weight_right(Wq, Qq, Bp, ld_Bp, s, Qb, L.ldr, We, L.ldw, nullptr, st));
    GemmParams p;
    memset(&p, 0, sizeof(p));
    p.A[0] = bf16_operand(x, ld_x, (int)T, (int)in);
    p.B[0] = bf16_operand(We, L.ldw, (int)out, (int)in);
    p.M = (int)T;
    p.N = (int)out;
    p.alpha = 1.0f;
    p.C = y;
    p.ldc = ld_y;
    p.split_ws = reinterpret_cast<float*>(base + L.partials);
    p.split_ws_floats = (int64_t)((ws_bytes - L.partials) / 4);
    LOQT_HIP(launch_gemm_nt(SLOT_GEMM_Y, EPI_BF16, false, false, p, st));
    return LOQT_OK;
}

loqt_status loqt_linear_bwd_right(const loqt_bf16* dy, int64_t ld_dy, const loqt_bf16* x, int64_t ld_x, int64_t T,
                                  const loqt_nf4_mat* Wq, const loqt_nf4_mat* Qq, const loqt_bf16* Bp,
                                  int64_t ld_Bp, float s, loqt_bf16* dx, int64_t ld_dx, void* dBp, int dBp_dtype,
                                  int64_t ld_dBp, int accumulate, void* ws, size_t ws_bytes, void* hip_stream) {
    LOQT_TRY(check_layer_right(Wq, Qq, Bp, ld_Bp));
    const int64_t out = Wq->rows, in = Wq->cols, r = Qq->cols;
    LOQT_TRY(check_bf16(dy, T, out, ld_dy));
    LOQT_TRY(check_bf16(x, T, in, ld_x));
    if (dx) LOQT_TRY(check_bf16(dx, T, in, ld_dx));
    if (!dBp) return LOQT_INVALID_ARG;
    if (dBp_dtype != LOQT_F32 && dBp_dtype != LOQT_BF16) return LOQT_INVALID_ARG;
    if (ld_dBp < r) return LOQT_BAD_SHAPE;
    if (!aligned(dBp, dBp_dtype == LOQT_BF16 ? 2 : 4)) return LOQT_MISALIGNED;
    const RightWs L(LOQT_OP_BWD_RIGHT, T, out, in, r, ws_bytes);
    LOQT_TRY(check_ws(ws, ws_bytes, L.least));
    const int64_t part_floats = (int64_t)((ws_bytes - L.partials) / 4);
    hipStream_t st = (hipStream_t)hip_stream;
    char* base = reinterpret_cast<char*>(ws);
    uint16_t* Qb = reinterpret_cast<uint16_t*>(base + L.Qb);
    uint16_t* We = reinterpret_cast<uint16_t*>(base + L.We);
    uint16_t* V = reinterpret_cast<uint16_t*>(base + L.V);
    float* part = reinterpret_cast<float*>(base + L.partials);
    LOQT_HIP(launch_dequantize(Qq->codes, Qq->absmax, in, r, Qq->ld, Qb, LOQT_BF16, L.ldr, st, SLOT_PREPASS));
    GemmParams p;
    // V = s x deq(Q): deq(Q) is in x r, i.e. K x rows
    memset(&p, 0, sizeof(p));
    p.A[0] = bf16_operand(x, ld_x, (int)T, (int)in);
    p.B[0] = bf16_operand(Qb, L.ldr, (int)r, (int)in);
    p.M = (int)T;
    p.N = (int)r;
    p.alpha = s;
    p.C = V;
    p.ldc = L.ldr;
    p.split_ws = part;
    p.split_ws_floats = part_floats;
    GemmParams pdx;
    if (!dx) {
        LOQT_HIP(launch_gemm_nt(SLOT_GEMM_U, EPI_BF16, false, true, p, st));
    } else {
        // dx = dy W_eff, W_eff out x in: K x rows
        LOQT_TRY(fold_weight_right(Wq, Qq, Bp, ld_Bp, s, Qb, L.ldr, We, L.ldw, &p, st));
        memset(&p, 0, sizeof(p));
        p.A[0] = bf16_operand(dy, ld_dy, (int)T, (int)out);
        p.B[0] = bf16_operand(We, L.ldw, (int)in, (int)out);
        p.M = (int)T;
        p.N = (int)in;
        p.alpha = 1.0f;
        p.C = dx;
        p.ldc = ld_dx;
        p.split_ws = part;
        p.split_ws_floats = part_floats;
        pdx = p;
    }
    // dBp = dy^T V: dy is T x out and V is T x r, both K x rows; contraction over T in slices
    memset(&p, 0, sizeof(p));
    p.A[0] = bf16_operand(dy, ld_dy, (int)out, (int)T);
    p.B[0] = bf16_operand(V, L.ldr, (int)r, (int)T);
    p.M = (int)out;
    p.N = (int)r;
    p.alpha = 1.0f;
    LOQT_HIP(gradient_product(SLOT_GEMM_DB, p, part, ws_bytes - L.partials, L.ldp, dBp, dBp_dtype, ld_dBp, accumulate,
                              dx ? &pdx : nullptr, st));
    return LOQT_OK;
}

loqt_status loqt_merge_requant_right(const loqt_nf4_mat* Wq, uint8_t* codes_out, float* absmax_out,
                                     const loqt_nf4_mat* Qq, const loqt_bf16* Bp, int64_t ld_Bp, float s, void* ws,
                                     size_t ws_bytes, void* hip_stream) {
    if (!codes_out || !absmax_out) return LOQT_INVALID_ARG;
    LOQT_TRY(check_layer_right(Wq, Qq, Bp, ld_Bp));
    if (!aligned(codes_out, 16) || !aligned(absmax_out, 4)) return LOQT_MISALIGNED;
    LOQT_TRY(check_out_alias(Wq, codes_out, absmax_out));
    const int64_t out = Wq->rows, in = Wq->cols, r = Qq->cols;
    const RightWs L(LOQT_OP_MERGE_RIGHT, 0, out, in, r, ws_bytes);
    LOQT_TRY(check_ws(ws, ws_bytes, L.total));
    hipStream_t st = (hipStream_t)hip_stream;
    uint16_t* Qb = reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(ws) + L.Qb);
    LOQT_HIP(launch_dequantize(Qq->codes, Qq->absmax, in, r, Qq->ld, Qb, LOQT_BF16, L.ldr, st, SLOT_PREPASS));
    GemmParams p;
    memset(&p, 0, sizeof(p));
    p.A[0] = bf16_operand(Bp, ld_Bp, (int)out, (int)r);  // rows of the tile are rows of W
    p.B[0] = bf16_operand(Qb, L.ldr, (int)in, (int)r);   // in x r: columns of the tile run along `in`
    p.M = (int)out;
    p.N = (int)Wq->ld;  // reach the padding columns (operand rows past `in` are never used)
    p.alpha = s;
    p.w_codes = Wq->codes;
    p.w_absmax = Wq->absmax;
    p.out_codes = codes_out;
    p.out_absmax = absmax_out;
    p.w_ld = Wq->ld;
    p.w_cols = (int)in;
    LOQT_HIP(launch_gemm_nt(SLOT_MERGE, EPI_MERGE, false, false, p, st));
    return LOQT_OK;
}

loqt_status loqt_merge_dense(const loqt_nf4_mat* Wq, const loqt_nf4_mat* Pq, const loqt_bf16* B, int64_t ld_B,
                             float s, float* W_out, int64_t ld_out, void* ws, size_t ws_bytes, void* hip_stream) {
    if (!W_out) return LOQT_INVALID_ARG;
    LOQT_TRY(check_layer(Wq, Pq, B, ld_B));
    const int64_t out = Wq->rows, in = Wq->cols, r = Pq->cols;
    if (ld_out < 0) return LOQT_INVALID_ARG;
    if (ld_out % 4 != 0 || ld_out < in) return LOQT_BAD_SHAPE;
    if (!aligned(W_out, 16)) return LOQT_MISALIGNED;
    const MergeWs L(out, in, r);
    if (!ws) return LOQT_INVALID_ARG;
    if (!aligned(ws, 256)) return LOQT_MISALIGNED;
    if (ws_bytes < L.total) return LOQT_WORKSPACE_TOO_SMALL;
    hipStream_t st = (hipStream_t)hip_stream;
    uint16_t* Pb = reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(ws) + L.Pb);
    const int64_t ldr = (int64_t)round_up(r, 8);
    LOQT_HIP(launch_dequantize(Pq->codes, Pq->absmax, out, r, Pq->ld, Pb, LOQT_BF16, ldr, st, SLOT_PREPASS));
    GemmParams p;
    memset(&p, 0, sizeof(p));
    p.A[0] = bf16_operand(Pb, ldr, (int)out, (int)r);
    p.B[0] = bf16_operand(B, ld_B, (int)in, (int)r);  // r x in: K x rows
    p.M = (int)out;
    p.N = (int)in;
    p.alpha = s;
    p.C = W_out;
    p.ldc = ld_out;
    p.splits = 1;
    p.w_codes = Wq->codes;
    p.w_absmax = Wq->absmax;
    p.w_ld = Wq->ld;
    p.w_cols = (int)in;
    LOQT_HIP(launch_gemm_nt(SLOT_MERGE_DENSE, EPI_FOLD_F32, false, true, p, st));
    return LOQT_OK;
}

loqt_status loqt_adam_step(loqt_bf16* B, int64_t ld_B, int64_t rows, int64_t cols, const void* grad, int grad_dtype,
                           int64_t ld_grad, float* m, float* v, int64_t ld_mv, float lr, float beta1, float beta2,
                           float eps, int64_t step, void* hip_stream) {
    if (!grad || !m || !v) return LOQT_INVALID_ARG;
    if (grad_dtype != LOQT_F32 && grad_dtype != LOQT_BF16) return LOQT_INVALID_ARG;
    if (step < 1 || !(lr >= 0.f) || !(eps >= 0.f) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f))
        return LOQT_INVALID_ARG;
    LOQT_TRY(check_bf16(B, rows, cols, ld_B));
    if (ld_grad < cols || ld_mv < cols) return LOQT_BAD_SHAPE;
    if (!aligned(grad, grad_dtype == LOQT_BF16 ? 2 : 4) || !aligned(m, 4) || !aligned(v, 4)) return LOQT_MISALIGNED;
    // bias corrections in double on the host
    const double bc1 = 1.0 / (1.0 - pow((double)beta1, (double)step));
    const double bc2 = 1.0 / (1.0 - pow((double)beta2, (double)step));
    LOQT_HIP(launch_adam(B, ld_B, grad, grad_dtype, ld_grad, m, v, ld_mv, rows, cols, lr, beta1, beta2, eps,
                         (float)bc1, (float)bc2, (hipStream_t)hip_stream));
    return LOQT_OK;
}

loqt_status loqt_merge_schedule(double tau, double psi, int64_t cap, int n, int64_t* steps_out) {
    if (!steps_out || n < 0) return LOQT_INVALID_ARG;
    if (!(tau >= 1.0) || !(psi >= 1.0) || cap < 1) return LOQT_INVALID_ARG;
    int64_t t = 0;
    for (int i = 0; i < n; ++i) {
        const double gap = floor(tau + pow(psi, (double)i));  // +inf once psi^i overflows: capped below
        t += gap >= (double)cap ? cap : (int64_t)gap;
        steps_out[i] = t;
    }
    return LOQT_OK;
}

// ---------------------------------------------------------------------------------------
// LoQT-nq: W and P in bf16, no quantisation anywhere
// ---------------------------------------------------------------------------------------
namespace {
loqt_status check_layer_nq(const loqt_bf16* W, int64_t ld_W, const loqt_bf16* P, int64_t ld_P, const loqt_bf16* B,
                           int64_t ld_B, int64_t out, int64_t in, int64_t r) {
    LOQT_TRY(check_bf16(W, out, in, ld_W));
    LOQT_TRY(check_bf16(P, out, r, ld_P));
    LOQT_TRY(check_bf16(B, r, in, ld_B));
    return LOQT_OK;
}
}  // namespace

// W_eff = bf16(W + s P B) for the unquantised layer (the product of loqt_merge_nq, written to `We`, pitch ld_we,
// instead of over W)
static hipError_t fold_nq(const loqt_bf16* W, int64_t ld_W, const loqt_bf16* P, int64_t ld_P, const loqt_bf16* B,
                          int64_t ld_B, int64_t out, int64_t in, int64_t r, float s, uint16_t* We, int64_t ld_we,
                          const GemmParams* z, hipStream_t st) {
    GemmParams p;
    memset(&p, 0, sizeof(p));
    p.A[0] = bf16_operand(P, ld_P, (int)out, (int)r);
    p.B[0] = bf16_operand(B, ld_B, (int)in, (int)r);  // r x in: K x rows
    p.M = (int)out;
    p.N = (int)in;
    p.alpha = s;
    p.C = We;
    p.ldc = ld_we;
    p.w_bf16 = W;
    p.w_bf16_ld = ld_W;
    if (z) return launch_z_fold(SLOT_GEMM_Z, *z, SLOT_FOLD, EPI_ACC_BF16, true, p, st);
    return launch_gemm_nt(SLOT_FOLD, EPI_ACC_BF16, false, true, p, st);
}

loqt_status loqt_linear_fwd_nq(const loqt_bf16* x, int64_t ld_x, int64_t T, const loqt_bf16* W, int64_t ld_W,
                               const loqt_bf16* P, int64_t ld_P, const loqt_bf16* B, int64_t ld_B, int64_t out,
                               int64_t in, int64_t r, float s, loqt_bf16* y, int64_t ld_y, void* ws,
                               size_t ws_bytes, void* hip_stream) {
    LOQT_TRY(check_layer_nq(W, ld_W, P, ld_P, B, ld_B, out, in, r));
    LOQT_TRY(check_bf16(x, T, in, ld_x));
    LOQT_TRY(check_bf16(y, T, out, ld_y));
    const bool few = use_few_tokens(T) && out <= FEW_ROWS_MAX_BF16, folded = use_folded(T, out, in);
    const NqWs L(false, T, out, in, r, ws_bytes);
    LOQT_TRY(check_ws(ws, ws_bytes, folded ? L.least : L.We));
    hipStream_t st = (hipStream_t)hip_stream;
    // slices of U and y: past the folded weight, or in its place when this call does not fold
    const size_t split_off = folded ? L.split : L.We;
    float* split = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + split_off);
    const int64_t split_floats = (int64_t)((ws_bytes - split_off) / 4);
    uint16_t* U = reinterpret_cast<uint16_t*>(ws);
    const int64_t ld_u = (int64_t)round_up(r, 8);
    GemmParams p;
    if (folded && !few) {  // y = x W_eff^T with the rank-r term folded into a transient copy of the weight
        uint16_t* We = reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(ws) + L.We);
        const int64_t ld_we = L.ldw;
        LOQT_HIP(fold_nq(W, ld_W, P, ld_P, B, ld_B, out, in, r, s, We, ld_we, nullptr, st));
        memset(&p, 0, sizeof(p));
        p.A[0] = bf16_operand(x, ld_x, (int)T, (int)in);
        p.B[0] = bf16_operand(We, ld_we, (int)out, (int)in);
        p.M = (int)T;
        p.N = (int)out;
        p.alpha = 1.0f;
        p.C = y;
        p.ldc = ld_y;
        p.split_ws = split;
        p.split_ws_floats = split_floats;
        LOQT_HIP(launch_gemm_nt(SLOT_GEMM_Y, EPI_BF16, false, false, p, st));
        return LOQT_OK;
    }
    memset(&p, 0, sizeof(p));  // U = s x B^T
    p.A[0] = bf16_operand(x, ld_x, (int)T, (int)in);
    p.B[0] = bf16_operand(B, ld_B, (int)r, (int)in);
    p.M = (int)T;
    p.N = (int)r;
    p.alpha = s;
    p.C = U;
    p.ldc = ld_u;
    p.split_ws = split;
    p.split_ws_floats = split_floats;
    LOQT_HIP(few ? launch_u_few(p, split, (size_t)split_floats * 4, st) : launch_gemm_nt(SLOT_GEMM_U, EPI_BF16, false, false, p, st));
    memset(&p, 0, sizeof(p));  // y = [x | U] [W | P]^T
    p.A[0] = bf16_operand(x, ld_x, (int)T, (int)in);
    p.B[0] = bf16_operand(W, ld_W, (int)out, (int)in);
    p.A[1] = bf16_operand(U, ld_u, (int)T, (int)r);
    p.B[1] = bf16_operand(P, ld_P, (int)out, (int)r);
    p.M = (int)T;
    p.N = (int)out;
    p.alpha = 1.0f;
    p.C = y;
    p.ldc = ld_y;
    p.split_ws = split;
    p.split_ws_floats = split_floats;
    LOQT_HIP(few ? launch_few_tokens(SLOT_GEMM_Y, false, p, st) : launch_gemm_nt(SLOT_GEMM_Y, EPI_BF16, false, false, p, st));
    return LOQT_OK;
}

loqt_status loqt_linear_bwd_nq(const loqt_bf16* dy, int64_t ld_dy, const loqt_bf16* x, int64_t ld_x, int64_t T,
                               const loqt_bf16* W, int64_t ld_W, const loqt_bf16* P, int64_t ld_P,
                               const loqt_bf16* B, int64_t ld_B, int64_t out, int64_t in, int64_t r, float s,
                               loqt_bf16* dx, int64_t ld_dx, void* dB, int dB_dtype, int64_t ld_dB, int accumulate,
                               void* ws, size_t ws_bytes, void* hip_stream) {
    LOQT_TRY(check_layer_nq(W, ld_W, P, ld_P, B, ld_B, out, in, r));
    LOQT_TRY(check_bf16(dy, T, out, ld_dy));
    LOQT_TRY(check_bf16(x, T, in, ld_x));
    if (dx) LOQT_TRY(check_bf16(dx, T, in, ld_dx));
    if (!dB) return LOQT_INVALID_ARG;
    if (dB_dtype != LOQT_F32 && dB_dtype != LOQT_BF16) return LOQT_INVALID_ARG;
    if (ld_dB < in) return LOQT_BAD_SHAPE;
    if (!aligned(dB, dB_dtype == LOQT_BF16 ? 2 : 4)) return LOQT_MISALIGNED;
    const NqWs L(true, T, out, in, r, ws_bytes);
    const size_t z_bytes = bf16_bytes(T, r);
    const bool folded = dx && use_folded(T, out, in);
    // slices of Z, dx and dB, one after the other: in the region of the dB slices, or past the folded weight (or in its
    // place) where there is more room
    LOQT_TRY(check_ws(ws, ws_bytes, folded ? L.least : L.We));
    hipStream_t st = (hipStream_t)hip_stream;
    uint16_t* Z = reinterpret_cast<uint16_t*>(ws);
    uint16_t* We = reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(ws) + L.We);
    const bool at_end = folded && ws_bytes - L.split > L.We - L.partials;
    float* part = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + (at_end ? L.split : z_bytes));
    const size_t part_bytes = at_end ? ws_bytes - L.split : folded ? L.We - L.partials : ws_bytes - L.partials;
    const int64_t ld_we = L.ldw;
    const int64_t ld_z = (int64_t)round_up(r, 8);
    GemmParams p;
    memset(&p, 0, sizeof(p));  // Z = s dy P: P is out x r, i.e. K x rows
    p.A[0] = bf16_operand(dy, ld_dy, (int)T, (int)out);
    p.B[0] = bf16_operand(P, ld_P, (int)r, (int)out);
    p.M = (int)T;
    p.N = (int)r;
    p.alpha = s;
    p.C = Z;
    p.ldc = ld_z;
    p.split_ws = part;
    p.split_ws_floats = (int64_t)(part_bytes / 4);
    if (folded) LOQT_HIP(fold_nq(W, ld_W, P, ld_P, B, ld_B, out, in, r, s, We, ld_we, &p, st));
    else LOQT_HIP(launch_gemm_nt(SLOT_GEMM_Z, EPI_BF16, false, true, p, st));
    GemmParams pdx;
    if (dx) {  // dx = [dy | Z] [W ; B]: W is out x in and B is r x in, both K x rows; folded: dx = dy W_eff
        memset(&p, 0, sizeof(p));
        p.A[0] = bf16_operand(dy, ld_dy, (int)T, (int)out);
        p.B[0] = folded ? bf16_operand(We, ld_we, (int)in, (int)out) : bf16_operand(W, ld_W, (int)in, (int)out);
        if (!folded) {
            p.A[1] = bf16_operand(Z, ld_z, (int)T, (int)r);
            p.B[1] = bf16_operand(B, ld_B, (int)in, (int)r);
        }
        p.M = (int)T;
        p.N = (int)in;
        p.alpha = 1.0f;
        p.C = dx;
        p.ldc = ld_dx;
        p.split_ws = part;
        p.split_ws_floats = (int64_t)(part_bytes / 4);
        pdx = p;
    }
    memset(&p, 0, sizeof(p));  // dB = Z^T x over slices of T
    p.A[0] = bf16_operand(Z, ld_z, (int)r, (int)T);
    p.B[0] = bf16_operand(x, ld_x, (int)in, (int)T);
    p.M = (int)r;
    p.N = (int)in;
    p.alpha = 1.0f;
    LOQT_HIP(gradient_product(SLOT_GEMM_DB, p, part, part_bytes, L.ldp, dB, dB_dtype, ld_dB, accumulate, dx ? &pdx : nullptr, st));
    return LOQT_OK;
}

loqt_status loqt_merge_nq(loqt_bf16* W, int64_t ld_W, const loqt_bf16* P, int64_t ld_P, const loqt_bf16* B,
                          int64_t ld_B, int64_t out, int64_t in, int64_t r, float s, void* hip_stream) {
    LOQT_TRY(check_layer_nq(W, ld_W, P, ld_P, B, ld_B, out, in, r));
    GemmParams p;
    memset(&p, 0, sizeof(p));  // W <- bf16(W + s P B), in place
    p.A[0] = bf16_operand(P, ld_P, (int)out, (int)r);
    p.B[0] = bf16_operand(B, ld_B, (int)in, (int)r);  // r x in: K x rows
    p.M = (int)out;
    p.N = (int)in;
    p.alpha = s;
    p.C = W;
    p.ldc = ld_W;
    p.w_bf16 = W;
    p.w_bf16_ld = ld_W;
    LOQT_HIP(launch_gemm_nt(SLOT_MERGE, EPI_ACC_BF16, false, true, p, (hipStream_t)hip_stream));
    return LOQT_OK;
}

size_t loqt_absmax_dq_workspace_bytes(int64_t n) {
    return n <= 0 ? 0 : round_up((size_t)dq_partials(n) * sizeof(double), 256);
}

loqt_status loqt_absmax_dq_compress(const float* absmax, int64_t n, uint8_t* codes8, float* c1, float* mean, void* ws,
                                    size_t ws_bytes, void* hip_stream) {
    if (!absmax || !codes8 || !c1 || !mean) return LOQT_INVALID_ARG;
    if (n <= 0 || n > ((int64_t)1 << 40)) return LOQT_BAD_SHAPE;
    if (!aligned(absmax, 4) || !aligned(c1, 4) || !aligned(mean, 4)) return LOQT_MISALIGNED;
    LOQT_TRY(check_ws(ws, ws_bytes, loqt_absmax_dq_workspace_bytes(n)));
    if (!aligned(ws, 8)) return LOQT_MISALIGNED;
    LOQT_HIP(launch_dq_compress(absmax, n, codes8, c1, mean, reinterpret_cast<double*>(ws), (hipStream_t)hip_stream));
    return LOQT_OK;
}

int64_t loqt_absmax_dq_static_max_n(void) { return dq_static_max_n(); }

loqt_status loqt_absmax_dq_compress_static(const float* absmax, int64_t n, uint8_t* codes8, float* c1, float* mean,
                                           void* hip_stream) {
    if (!absmax || !codes8 || !c1 || !mean) return LOQT_INVALID_ARG;
    if (n <= 0) return LOQT_BAD_SHAPE;
    if (n > dq_static_max_n()) return LOQT_STATIC_SCRATCH_TOO_SMALL;
    if (!aligned(absmax, 4) || !aligned(c1, 4) || !aligned(mean, 4)) return LOQT_MISALIGNED;
    LOQT_HIP(launch_dq_compress_static(absmax, n, codes8, c1, mean, (hipStream_t)hip_stream));
    return LOQT_OK;
}

loqt_status loqt_absmax_dq_expand(const uint8_t* codes8, const float* c1, const float* mean, int64_t n, float* absmax_out,
                                  void* hip_stream) {
    if (!codes8 || !c1 || !mean || !absmax_out) return LOQT_INVALID_ARG;
    if (n <= 0 || n > ((int64_t)1 << 40)) return LOQT_BAD_SHAPE;
    if (!aligned(c1, 4) || !aligned(mean, 4) || !aligned(absmax_out, 4)) return LOQT_MISALIGNED;
    LOQT_HIP(launch_dq_expand(codes8, c1, mean, n, absmax_out, (hipStream_t)hip_stream));
    return LOQT_OK;
}

loqt_status loqt_prepare(void) {
    LOQT_HIP(prepare_nt_kernels());
    LOQT_HIP(prepare_fused_kernels());
    LOQT_HIP(prepare_nf4_tile_kernels());
    void* scratch_ptr = nullptr;
    LOQT_HIP(dq_static_scratch(&scratch_ptr));
    return LOQT_OK;
}

loqt_status loqt_set_path(int path) {
    if (path < LOQT_PATH_AUTO || path > LOQT_PATH_CODES) return LOQT_INVALID_ARG;
    g_path = path;
    return LOQT_OK;
}

loqt_status loqt_set_tile(int tile) {
    if (tile < LOQT_TILE_AUTO || tile > LOQT_TILE_128x128) return LOQT_INVALID_ARG;
    g_nt_tile_override = tile;
    return LOQT_OK;
}

loqt_status loqt_plan_product(int64_t M, int64_t N, int64_t Nx, int64_t* n_large, double* rounds) {
    if (M <= 0 || N <= 0 || Nx < 0 || M > ((int64_t)1 << 30) || N > ((int64_t)1 << 30) || Nx > ((int64_t)1 << 30))
        return LOQT_BAD_SHAPE;
    const BF16Plan plan = plan_bf16_product(M, N, Nx);
    if (n_large) *n_large = plan.n1;
    if (rounds) *rounds = plan.cost;
    return LOQT_OK;
}

loqt_status loqt_plan_tiles(int64_t M, int64_t N, int64_t K, int sliced, int max_splits, int* tile, int* splits) {
    if (M <= 0 || N <= 0 || K <= 0 || max_splits < 1 || M > ((int64_t)1 << 30) || N > ((int64_t)1 << 30) ||
        K > ((int64_t)1 << 30))
        return LOQT_BAD_SHAPE;
    const NtPlan plan = plan_nt(M, N, (K + 63) / 64, sliced != 0, 1, max_splits);
    if (tile) *tile = plan.tile;
    if (splits) *splits = plan.splits;
    return LOQT_OK;
}

int loqt_plan_weight(int op, int64_t out, int64_t in, int64_t r) {
    constexpr int64_t LIMIT = (int64_t)1 << 30;
    if (out <= 0 || in <= 0 || r <= 0 || out > LIMIT || in > LIMIT || r > LIMIT) return 0;
    const bool merge = op == LOQT_OP_MERGE || op == LOQT_OP_MERGE_RIGHT, right = op == LOQT_OP_FWD_RIGHT || op == LOQT_OP_MERGE_RIGHT;
    if (!merge && !right && op != LOQT_OP_FWD && op != LOQT_OP_FWD_NQ) return 0;
    GemmParams p;
    memset(&p, 0, sizeof(p));
    p.M = (int)out;
    p.N = (int)(merge ? round_up(in, 64) : in);
    p.A[0].K = (int)r;
    return weight_tile(merge ? EPI_MERGE : op == LOQT_OP_FWD_NQ ? EPI_ACC_BF16 : EPI_FOLD, !right, p);
}

int loqt_plan_merge_group(int n, const int64_t* out, const int64_t* in, const int64_t* r) {
    if (n < 1 || n > MERGE_GROUP_MAX || !out || !in || !r) return 0;
    MergeGroupLayer layers[MERGE_GROUP_MAX];
    memset(layers, 0, sizeof(layers));
    for (int i = 0; i < n; ++i) {
        constexpr int64_t LIMIT = (int64_t)1 << 30;
        if (out[i] <= 0 || in[i] <= 0 || r[i] <= 0 || out[i] > LIMIT || in[i] > LIMIT || r[i] > LIMIT) return 0;
        layers[i].out = (int)out[i], layers[i].in = (int)in[i], layers[i].r = (int)r[i], layers[i].w_ld = (int64_t)round_up(in[i], 64);
    }
    return merge_group_tile(layers, n);
}

int loqt_plan_codes(int64_t T, int64_t N, int64_t K, int extra, int max_slices) {
    if (T <= 0 || N <= 0 || K <= 0 || max_slices < 1 || T > ((int64_t)1 << 30) || N > ((int64_t)1 << 30) || K > ((int64_t)1 << 30)) return 0;
    return nf4_tile_splits(T, N, (K + 63) / 64, extra != 0, max_slices);
}

void loqt_timing_enable(int on) {
    if (on) {
        if (!g_timing.begin) {
            g_timing.begin = new hipEvent_t[LOQT_TIMING_MAX_EVENTS];
            g_timing.end = new hipEvent_t[LOQT_TIMING_MAX_EVENTS];
            g_timing.slot = new int[LOQT_TIMING_MAX_EVENTS];
        }
        g_timing.n = 0;
        g_timing.on = true;
    } else {
        g_timing.on = false;
    }
}

int loqt_timing_slots(void) { return SLOT_COUNT; }

loqt_status loqt_timing_read(int slot, const char** name, int64_t* launches, double* total_ms) {
    if (slot < 0 || slot >= SLOT_COUNT || !name || !launches || !total_ms) return LOQT_INVALID_ARG;
    *name = kSlotNames[slot];
    *launches = 0;
    *total_ms = 0.0;
    for (int i = 0; i < g_timing.n; ++i) {
        if (g_timing.slot[i] != slot) continue;
        if (hipEventSynchronize(g_timing.end[i]) != hipSuccess) return LOQT_LAUNCH_FAILED;
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, g_timing.begin[i], g_timing.end[i]) != hipSuccess) return LOQT_LAUNCH_FAILED;
        *launches += 1;
        *total_ms += ms;
    }
    return LOQT_OK;
}

}  // extern "C"
