// Launches of the plain products (bf16 outputs and fp32 slices of the contraction): tile shape and number of slices from the
// sizes.  The kernel itself is in nt_tile.h; the products whose epilogue walks the weight are in gemm_weight.hip.
#include <string.h>

#include <algorithm>

#include "nt_tile.h"

namespace loqt {

// Plan of a bf16-output product of M rows and N (+ Nx extra) columns in units of one round of 256x256 tiles
// (256 tiles, one per compute unit).  A round of 128x128 tiles (512, two per compute unit) takes 0.68 of that,
// measured, whether it is full or half full.  n1 > 0: the first n1 columns as 256x256 tiles in whole rounds, the
// rest and the extra columns as 128x128 tiles.
BF16Plan plan_bf16_product(int64_t M, int64_t N, int64_t Nx) {
    auto cdiv = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    const int64_t tm = cdiv(M, 256), tn = cdiv(N, 256), tnx = cdiv(Nx, 256);
    BF16Plan plan;
    plan.n1 = 0;
    plan.cost = (double)cdiv(tm * (tn + tnx), 256);
    const int64_t whole = tm * tn / 256;
    const int64_t c1 = whole * 256 / tm;  // tile columns of the first launch
    if (whole >= 1 && c1 > 0 && c1 < tn && whole * 256 - c1 * tm < 32) {
        const int64_t n1 = c1 * 256;
        const int64_t tiles_b = cdiv(M, 128) * (cdiv(N - n1, 128) + cdiv(Nx, 128));
        const double cost = (double)whole + 0.68 * (double)cdiv(tiles_b, 512);
        if (cost < plan.cost) plan.cost = cost, plan.n1 = (int)n1;
    }
    return plan;
}

// Products that do not fill the chip with 256x256 tiles over a long contraction (few tokens, narrow outputs, short
// contractions) and the fp32 slices of dB and its relatives: tile shape and number of slices of the contraction from
// an estimate in microseconds.  Per shape: work-groups per compute unit, the time of one k-tile when a few work-groups
// have memory to themselves (a serial chain of barrier, fragment reads and matrix instructions), when every compute unit runs
// one and when it runs two (shared LDS, L2, fabric and power), and the rest of a tile (first loads, epilogue).
// Over 6000 random products (y, dx and Z, gradients; every tile, 1 to 32 slices, timed by themselves) the plan takes 1.023 of the time of the
// best choice, 1.033 over those of 9 us and more, one in eight of which is more than 10 % off (1.025, 1.037 and one in seven with 128x128 at
// the price of the two-stage loop everywhere).  Constants fitted to products by themselves (1.016) don't hold in whole calls, so two
// come from 33700 products of forward and backward calls of random sizes (timed with loops in which every wave loaded).  A tile of
// 256x128 costs 5.0 beside its loop: with 4.0 they were taken, often in two or three slices, where 256x256 or 128x128 in one are ahead (y of 7817 x 13467 x 1856 350 us
// against 308).  And `cold`: operands of more than 128 MB do not stay in the Infinity Cache, and the smaller the tile the more often they
// are read (y of 4417 x 2135 x 12381 329 us on 256x128 in three slices and 216 on 256x256, of 7621 x 1465 x 9856 234 in two and 177).
// With both, 122 of those products make their call 1.05 times as fast or more, 15 as slow.  The 64-row tiles have rings of
// three and four stages (256 x 128 x 4096 on 64x64, us: 17.8 with three, 18.0 with four, 21.6 with eight; 1024 x 1024 x 4096
// 21.1, 18.8 and 23.3).  128x128 tiles have two, which lets a compute unit hold two of them; where it gets one at most they have three and
// waves of their own for the loads, and a price of their own (kLone128).
struct TileSpec {
    int id, bm, bn, per_cu;
    double alone, full, both, fix, cold;
};
constexpr TileSpec kTiles[] = {
    {NT_64x64, 64, 64, 2, 0.22, 0.24, 0.48, 1.99, 1.15},
    {NT_64x128, 64, 128, 2, 0.27, 0.34, 0.79, 2.24, 1.1},
    {NT_128x128, 128, 128, 2, 0.47, 0.61, 1.08, 3.0, 1.1},
    {NT_256x128, 256, 128, 1, 0.60, 0.78, 0.78, 5.0, 1.25},
    {NT_256x256, 256, 256, 1, 1.20, 1.49, 1.49, 7.95, 1.0},
};
// 128x128 tiles in a launch that gives a compute unit one of them at most (one_to_a_unit).  At the price of the two-stage loop (0.47 to
// 0.61) they lost to 64x128 and to slices of 256x128 that are slower (forward + backward of 746 tokens, 3234 x 3234, rank 64, unquantised,
// 106.7 -> 85.9 us; 640, 3970 x 3970, rank 32, 126.8 -> 111.5).  Of 1444 random calls of more than 256 tokens 157 change, to 0.970 of
// the time on the mean, two by more than 4 % for the worse.  By themselves these products take 0.35 to 0.51 us per k-tile, but at 0.57
// they also take one slice where 256x128 in two is ahead in the call (y of 7808 x 384 x 7296, 161.6 -> 171.1): 274 change then, eight
// for the worse.  (Another 919 calls of 45 us and more: 0.994 over all, 47 of them 4 % faster or more, one slower, 1152 x 5760, rank 69,
// 2176 tokens, 113.5 -> 119.3.)  Not for gradients: on 64-row tiles they share the launch of dx (451 tokens, 1792 x 3035, rank 768, 77 us; 86 with
// the gradient on 128x128).
constexpr TileSpec kLone128{NT_128x128, 128, 128, 1, 0.27, 0.62, 0.62, 2.8, 1.1};

// `tiles` of the output in `splits` slices of at most `per` k-tiles: the time of the fullest compute unit.  Each XCD takes an
// eighth of the tiles, rounded up, of every slice: 84 tiles in three slices are 33 work-groups for each of seven XCDs with 32
// compute units, two rounds, although they number 252 (256x128 tiles of 5209 x 480 x 6160, us: one slice 82, two 57, three 81).
// And the first unit with a second work-group holds up the launch, though less than when all have two and share what is beyond
// the unit: of the way from `full` to `both`, 0.3 at once (1024 x 5120 x 13824: 320 tiles of 128x128 231, 160 of 256x128 165;
// 437 x 5062 x 5384: 280 of 64x128 82, 80 of 256x128 in three slices 48).
// lone: 128x128 may take the price of kLone128.
double tile_cost(const TileSpec& shape, int64_t tiles, int per, int splits, bool cold, bool lone) {
    const int64_t wgs = (tiles + 7) / 8 * splits;  // of the fullest XCD
    const TileSpec& t = lone && shape.id == NT_128x128 && wgs <= 32 ? kLone128 : shape;
    const int log2_round = t.per_cu == 2 ? 6 : 5;  // ... and in one round of its 32 compute units
    const int64_t rounds = wgs >> log2_round, rest = wgs & ((1 << log2_round) - 1);
    const double kt = (double)per * (cold ? t.cold : 1.0);
    auto one = [&](int64_t w) {
        const double u = (double)w / 32.0;
        if (u <= 1.0) return kt * (t.alone + (t.full - t.alone) * u) + t.fix;
        return kt * (t.full + (t.both - t.full) * (0.3 + 0.7 * (u - 1.0))) + t.fix;
    };
    return (rounds ? (double)rounds * one((int64_t)1 << log2_round) : 0.0) + (rest ? one(rest) : 0.0);
}

// `rows` of both operands together
bool cold_operands(int64_t rows, int64_t nkt) { return rows * nkt > (int64_t)1000000; }  // 128 bytes to a k-tile

// slices > 1 (or `sliced`: the result is summed from fp32 slices in any case) cost their own traffic and the
// reduction's: written at about 6 TB/s, read back at 7, and a launch
double slices_cost(int64_t M, int64_t N, int splits) {
    const double bytes = (double)M * (double)N * 4.0 * splits;
    return bytes / 6.0e6 + 4.0 + (bytes + (double)M * (double)N * 2.0) / 7.0e6;
}

// Runs once per product and call, so it is kept to about a microsecond (5.5 without the bound on the slices and with 64-bit
// divisions in the loop, as much as a launch).
NtPlan plan_nt(int64_t M, int64_t N, int64_t nkt, bool sliced, int min_splits, int max_splits) {
    auto cdiv = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    const int kts = (int)nkt;  // dimensions are at most 2^30
    const bool cold = cold_operands(M + N, nkt);
    NtPlan best{0, 1, 0.0};
    for (const TileSpec& t : kTiles) {
        if (sliced && t.id == NT_256x256) continue;  // no such kernel: its slices were slower than those of 256x128
        // dB and its relatives from rank 512 up: operands come from HBM, and shorter tiles read the longer one more often
        // (512 x 5461 x 8192, us: 66 on 256x128, 80 on 128x128; 5461 x 512 x 4096 36 and 43; 1024 x 5120 x 256 14 and 21).
        // The estimate does not see that: with 128x128 in it, 60 random products of 512 to 1024 rows take 1.01 of the time,
        // single ones 0.94 to 1.16.  One work-group to a unit at most is another matter (8141 x 384 x 1774 23 us on 128x128 in one
        // slice, 27 and a sum of 9 on 256x128 in two; 896 x 4480 x 3337 35 and 47 in one slice of either).
        const int64_t tiles = cdiv(M, t.bm) * cdiv(N, t.bn);
        const bool crowds = sliced && M >= 512 && t.id == NT_128x128;
        for (int splits = min_splits; splits <= max_splits; ++splits) {
            const int per = (int)((unsigned)(kts + splits - 1) / (unsigned)splits);
            if (min_splits < max_splits && splits > min_splits) {
                if (per < 4 || t.id == NT_256x256) break;
                if ((int)((unsigned)(kts + per - 1) / (unsigned)per) != splits) continue;  // the last slices would be empty
            }
            if (crowds && (tiles + 7) / 8 * splits > 32) break;
            const double extra = sliced || splits > 1 ? slices_cost(M, N, splits) : 0.0;
            if (best.tile != 0 && extra >= best.cost) break;  // and more slices cost more still
            const double cost = tile_cost(t, tiles, per, splits, cold, !sliced) + extra;
            if (best.tile == 0 || cost < best.cost) best = NtPlan{t.id, splits, cost};
        }
    }
    return best;
}

// a product of M rows and N columns with Nx extra columns beside them, on 128x128 tiles
double joint_cost_128(int64_t M, int64_t N, int64_t Nx, int64_t nkt) {
    auto cdiv = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    for (const TileSpec& t : kTiles)
        if (t.id == NT_128x128) return tile_cost(t, cdiv(M, 128) * (cdiv(N, 128) + cdiv(Nx, 128)), (int)nkt, 1, cold_operands(M + N + Nx, nkt), true);
    return 0.0;
}

// whether a bf16-output product of M rows, N (+ Nx) columns and contraction K runs on 256x256 tiles by the plan above
static bool large_product(int64_t M, int64_t N, int64_t Nx, int64_t K) {
    auto cdiv = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    return K >= 2048 && cdiv(M, 256) * (cdiv(N, 256) + cdiv(Nx, 256)) >= 224;
}

int64_t product_split_floats(int64_t M, int64_t N, int64_t K0, int64_t K1) {
    if (large_product(M, N, 0, K0 + K1)) return remainder_split_floats(M, N);
    const NtPlan plan = plan_nt(M, N, (K0 + BK - 1) / BK + (K1 + BK - 1) / BK, false, 1, NT_MAX_SPLITS);
    return plan.splits > 1 ? plan.splits * M * ((N + 3) / 4 * 4) : 0;
}

// Scratch (floats) for the column remainder of a bf16-output product of M rows and N columns in two fp32 slices
// of the contraction: when the plan has a remainder and its 256x128 tiles number 64 to 128 (see launch_nt_sized).
int64_t remainder_split_floats(int64_t M, int64_t N) {
    if (M < 512 || M * 2 > (int64_t)1 << 30) return 0;
    if (((M + 255) / 256) * ((N + 255) / 256) < 224) return 0;  // such a product takes no 256x256 tiles at all
    const BF16Plan plan = plan_bf16_product(M, N, 0);
    if (plan.n1 <= 0) return 0;
    const int64_t nb = N - plan.n1;
    const int64_t tiles = ((M + 255) / 256) * ((nb + 127) / 128);
    if (tiles < 64 || tiles > 128) return 0;
    return 2 * M * ((nb + 3) / 4 * 4);
}

namespace {

// one launch on the given tile shape
template <int EPI, bool ARC, bool BRC>
hipError_t launch_nt_tile(int tile, const GemmParams& p, hipStream_t st) {
    switch (tile) {
        case NT_256x256:
            if constexpr (EPI == EPI_BF16 && !ARC) return launch_nt<256, 256, EPI, ARC, BRC>(p, st);
            break;
        case NT_256x128: return launch_nt<256, 128, EPI, ARC, BRC, 3, false, false, true>(p, st);
        case NT_128x128:
            if (one_to_a_unit<EPI>(p)) return launch_nt<128, 128, EPI, ARC, BRC, 3, false, false, true>(p, st);
            return launch_nt<128, 128, EPI, ARC, BRC>(p, st);
        case NT_64x128: return launch_nt<64, 128, EPI, ARC, BRC, 3, false, false, true>(p, st);
        case NT_64x64: return launch_nt<64, 64, EPI, ARC, BRC, 4, false, false, true>(p, st);
    }
    return hipErrorInvalidValue;
}

int ktiles(const GemmParams& p) { return (p.A[0].K + BK - 1) / BK + (p.A[1].K + BK - 1) / BK; }

// the gradient of a factor: fp32 slices at p.C, or bf16
template <int EPI>
hipError_t launch_gradient(const GemmParams& p, hipStream_t st, const NtPlan* planned) {
    const int tile = planned ? planned->tile : gradient_tile(EPI, p);
    if constexpr (EPI == EPI_F32_SPLITK) {
        if (tile == NT_256x256) return launch_nt<256, 256, EPI, true, true>(p, st);  // (forced only)
    }
    return launch_nt_tile<EPI, true, true>(tile, p, st);
}

// C in bf16
template <bool BRC>
hipError_t launch_product(const GemmParams& p, hipStream_t st, const NtPlan* planned) {
    constexpr int EPI = EPI_BF16;
    if (g_nt_tile_override != 0) return launch_nt_tile<EPI, false, BRC>(g_nt_tile_override, p, st);
    // 256x256 tiles (one work-group per compute unit) have the best ratio of MFMA work to LDS and
    // global traffic and win on long contractions.
    if (!large_product(p.M, p.N, p.Nx, p.A[0].K + p.A[1].K)) {
        if (p.Nx != 0) return launch_nt_tile<EPI, false, BRC>(NT_128x128, p, st);
        const NtPlan plan = planned ? *planned : product_plan(p);
        if (plan.splits == 1) return launch_nt_tile<EPI, false, BRC>(plan.tile, p, st);
        const GemmParams c = product_slices(p, plan.splits);
        hipError_t e = launch_nt_tile<EPI_F32_SPLITK, false, BRC>(plan.tile, c, st);
        if (e != hipSuccess) return e;
        return launch_reduce_db(p.split_ws, plan.splits, p.M, p.N, c.ldc, p.C, LOQT_BF16, p.ldc, 0, st, false);
    }
    // 256x256 tiles run in rounds of one tile per compute unit.  When the last round would be mostly
    // empty, the tile columns that fill whole rounds go out as one launch and the remaining columns
    // (with the extra columns Nx, if any) as a second launch of 128x128 tiles.
    const BF16Plan plan = plan_bf16_product(p.M, p.N, p.Nx);
    if (plan.n1 <= 0) return launch_nt<256, 256, EPI, false, BRC>(p, st);
    const int n1 = plan.n1;
    GemmParams a = p, b = p;
    a.N = n1;
    a.Nx = 0;
    for (int seg = 0; seg < 2; ++seg) {
        if (p.A[seg].K == 0) continue;
        a.B[seg].rows = std::min(p.B[seg].rows, n1);
        b.B[seg].rows = p.B[seg].rows - n1;
        b.B[seg].ptr = reinterpret_cast<const uint16_t*>(p.B[seg].ptr) + (BRC ? (int64_t)n1 : (int64_t)n1 * p.B[seg].ld);
    }
    b.N = p.N - n1;
    b.C = reinterpret_cast<uint16_t*>(p.C) + n1;
    hipError_t e = launch_nt<256, 256, EPI, false, BRC>(a, st);
    if (e != hipSuccess) return e;
    // A remainder whose 256x128 tiles would fill no more than half of the compute units (13B block at
    // 4096 tokens: 1024 of 5120 columns, 128 tiles) goes out as two fp32 slices of the contraction,
    // twice the work-groups at half the depth, and the fixed-order sum of the two into bf16 (75 -> 47 us)
    const int64_t need = remainder_split_floats(p.M, p.N);
    if (need > 0 && b.Nx == 0 && p.split_ws != nullptr && p.split_ws_floats >= need) {
        GemmParams c = b;
        c.C = p.split_ws;
        c.ldc = (b.N + 3) / 4 * 4;
        c.splits = 2;
        e = launch_nt_tile<EPI_F32_SPLITK, false, BRC>(NT_256x128, c, st);
        if (e != hipSuccess) return e;
        return launch_reduce_db(p.split_ws, 2, b.M, b.N, c.ldc, b.C, LOQT_BF16, b.ldc, 0, st, false);
    }
    // between 129 and 256 tiles of 256x128 (7B gate / up forward: 768 of 11008 columns; 13B gate / up
    // forward: 1536 of 13824): that shape, one work-group per compute unit
    const int64_t t2 = ((int64_t)(b.M + 255) / 256) * ((b.N + 127) / 128);
    if (b.Nx == 0 && t2 > 128 && t2 <= 256) return launch_nt_tile<EPI, false, BRC>(NT_256x128, b, st);
    return launch_nt_tile<EPI, false, BRC>(NT_128x128, b, st);
}

template <int EPI, bool ARC, bool BRC>
hipError_t prepare_tiles() {
    hipError_t e;
    if constexpr (!ARC && EPI == EPI_BF16) {
        if ((e = ensure_attr<256, 256, EPI, ARC, BRC>()) != hipSuccess) return e;
        if ((e = ensure_attr<256, 256, EPI, ARC, BRC, 2, true>()) != hipSuccess) return e;
    }
    if ((e = ensure_attr<256, 128, EPI, ARC, BRC, 3, false, false, true>()) != hipSuccess) return e;
    if ((e = ensure_attr<256, 128, EPI, ARC, BRC, 3, true, false, true>()) != hipSuccess) return e;
    if ((e = ensure_attr<128, 128, EPI, ARC, BRC>()) != hipSuccess) return e;
    if ((e = ensure_attr<128, 128, EPI, ARC, BRC, 3, false, false, true>()) != hipSuccess) return e;
    if ((e = ensure_attr<64, 128, EPI, ARC, BRC, 3, false, false, true>()) != hipSuccess) return e;
    return ensure_attr<64, 64, EPI, ARC, BRC, 4, false, false, true>();
}

}  // namespace

int g_nt_tile_override = 0;

NtPlan product_plan(const GemmParams& p) {
    if (g_nt_tile_override != 0 || p.Nx != 0 || large_product(p.M, p.N, 0, p.A[0].K + p.A[1].K)) return NtPlan{0, 1, 0.0};
    const int64_t room = p.split_ws ? p.split_ws_floats / (p.M * ((p.N + 3) / 4 * 4)) : 0;
    return plan_nt(p.M, p.N, ktiles(p), false, 1, (int)std::min<int64_t>(std::max<int64_t>(room, 1), NT_MAX_SPLITS));
}

// fp32 slices of the contraction, for a fixed-order sum
GemmParams product_slices(const GemmParams& p, int splits) {
    GemmParams c = p;
    c.C = p.split_ws;
    c.ldc = (p.N + 3) / 4 * 4;
    c.splits = splits;
    return c;
}

// the number of slices was fixed with the workspace (plan_nt); the tile that goes with it
int gradient_tile(int epi, const GemmParams& p) {
    if (g_nt_tile_override != 0) return g_nt_tile_override;
    const int n = epi == EPI_BF16 ? 1 : p.splits;
    return plan_nt(p.M, p.N, ktiles(p), true, n, n).tile;
}

// every kernel configuration launch_gemm_nt / launch_merge_grouped can reach
hipError_t prepare_nt_kernels() {
    hipError_t e;
    if ((e = prepare_tiles<EPI_BF16, false, false>()) != hipSuccess) return e;
    if ((e = prepare_tiles<EPI_BF16, false, true>()) != hipSuccess) return e;
    if ((e = prepare_tiles<EPI_BF16, true, true>()) != hipSuccess) return e;
    if ((e = prepare_tiles<EPI_F32_SPLITK, false, false>()) != hipSuccess) return e;
    if ((e = prepare_tiles<EPI_F32_SPLITK, false, true>()) != hipSuccess) return e;
    if ((e = prepare_tiles<EPI_F32_SPLITK, true, true>()) != hipSuccess) return e;
    if ((e = ensure_attr<256, 256, EPI_F32_SPLITK, true, true>()) != hipSuccess) return e;
    if ((e = prepare_pair_kernels()) != hipSuccess) return e;
    return prepare_weight_kernels();
}

// a_rc / b_rc: the operand is stored K x rows (rows contiguous) instead of rows x K
hipError_t launch_gemm_nt(int slot, int epi, bool a_rc, bool b_rc, const GemmParams& p, hipStream_t st, const NtPlan* plan) {
    TimedLaunch tl(slot, st);
    if (epi != EPI_BF16 && epi != EPI_F32_SPLITK) return a_rc ? hipErrorInvalidValue : launch_weight_product(epi, b_rc, p, st);
    if (!a_rc && epi == EPI_BF16) return b_rc ? launch_product<true>(p, st, plan) : launch_product<false>(p, st, plan);
    if (!a_rc || !b_rc) return hipErrorInvalidValue;
    return epi == EPI_BF16 ? launch_gradient<EPI_BF16>(p, st, plan) : launch_gradient<EPI_F32_SPLITK>(p, st, plan);
}

}  // namespace loqt
