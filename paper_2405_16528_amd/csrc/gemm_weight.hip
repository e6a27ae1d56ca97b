// Products whose epilogue walks the weight (M = out, N = in): the fold of the rank-r term into a bf16 copy of the 4-bit or bf16
// weight, the merge with requantisation, one step of the compensated initialisation, the dense merge.  The kernel is in
// nt_tile.h.
#include <string.h>

#include <algorithm>

#include "nt_tile.h"

namespace loqt {

namespace {

// The merges of several layers (Alg. 1 line 5, one layer after the other) as ONE launch: the tiles of all layers
// form one grid, so the prologue and epilogue of one layer's tiles overlap with the products of the next layer's
// instead of every layer paying its own ramp-up, tail round and launch gap.  The per-layer descriptors travel in
// the kernel argument block itself (no device-side table to fill, nothing to allocate, capture-safe), which
// bounds a group at MERGE_GROUP_MAX layers.  per_xcd_end: running total of the tiles each XCD has walked when it
// is through with this layer.
struct MergeGroupItem {
    const void* A;          // left operand of s * A B: P, out x r, K contiguous, in bf16 or
    const float* A_absmax;  // as its codes
    const void* B;          // right operand: r x in stored K x rows
    int64_t lda, ldb;
    const uint8_t* w_codes;
    const float* w_absmax;
    uint8_t* out_codes;
    float* out_absmax;
    int64_t w_ld;
    int M, N, K, w_cols;
    float alpha;
    int per_xcd_end;
};
struct MergeGroupParams {
    int n;
    MergeGroupItem it[MERGE_GROUP_MAX];
};
static_assert(sizeof(MergeGroupParams) <= 4096, "kernel arguments are limited to 4 KB");

template <int BM>
constexpr int GROUP_BN = BM == 256 ? 256 : 128;
template <int BM, bool ANF4>
using GroupCfg = NtCfg<BM, GROUP_BN<BM>, 2, ANF4, BM == 256 ? 8 : 4>;

template <int BM, bool ANF4>
__global__ __launch_bounds__((GroupCfg<BM, ANF4>::THREADS), (GroupCfg<BM, ANF4>::THREADS / 256 * GroupCfg<BM, ANF4>::PER_CU)) void nt_merge_grouped_kernel(const MergeGroupParams g) {
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    int li = 0;
    while (li + 1 < g.n && j >= g.it[li].per_xcd_end) ++li;  // wave-uniform
    const int start = li ? g.it[li - 1].per_xcd_end : 0;
    const MergeGroupItem& it = g.it[li];
    GemmParams p;
    p.A[0].ptr = it.A, p.A[0].absmax = it.A_absmax, p.A[0].ld = it.lda, p.A[0].rows = it.M, p.A[0].K = it.K;
    p.B[0].ptr = it.B, p.B[0].absmax = nullptr, p.B[0].ld = it.ldb, p.B[0].rows = it.w_cols, p.B[0].K = it.K;
    p.A[1].ptr = nullptr, p.A[1].absmax = nullptr, p.A[1].ld = 0, p.A[1].rows = 0, p.A[1].K = 0;
    p.B[1] = p.A[1];
    p.Bx = p.A[1];
    p.M = it.M, p.N = it.N, p.alpha = it.alpha;
    p.C = nullptr, p.ldc = 0, p.splits = 1;
    p.Cx = nullptr, p.ldcx = 0, p.Nx = 0, p.alphax = 0.f;
    p.w_codes = it.w_codes, p.w_absmax = it.w_absmax, p.out_codes = it.out_codes, p.out_absmax = it.out_absmax;
    p.w_ld = it.w_ld, p.w_cols = it.w_cols;
    p.w_bf16 = nullptr, p.w_bf16_ld = 0, p.w_f32 = nullptr, p.w_f32_ld = 0, p.e_out = nullptr, p.e_ld = 0;
    const int per_xcd = it.per_xcd_end - start;
    nt_gemm_tile<BM, GROUP_BN<BM>, EPI_MERGE, false, true, 2, false, ANF4, false, GroupCfg<BM, ANF4>::THREADS / 64>(p, xcd * per_xcd + (j - start), 0);
}

// g: null only raises the kernel's LDS size
template <int BM, bool ANF4>
hipError_t launch_grouped(MergeGroupParams* g, hipStream_t st) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(nt_merge_grouped_kernel<BM, ANF4>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (GroupCfg<BM, ANF4>::SMEM));
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    if (!g) return hipSuccess;
    int per_xcd_total = 0;
    for (int i = 0; i < g->n; ++i) {
        MergeGroupItem& it = g->it[i];
        const int tiles = ((it.M + BM - 1) / BM) * ((it.N + GROUP_BN<BM> - 1) / GROUP_BN<BM>);
        per_xcd_total += (tiles + 7) / 8;
        it.per_xcd_end = per_xcd_total;
    }
    hipLaunchKernelGGL((nt_merge_grouped_kernel<BM, ANF4>), dim3((unsigned)per_xcd_total * 8u), dim3((GroupCfg<BM, ANF4>::THREADS)), (GroupCfg<BM, ANF4>::SMEM), st, *g);
    return hipGetLastError();
}

// (256x128 tiles were behind wherever they were timed: loqt_set_tile alone selects them.)
template <int EPI, bool BRC>
hipError_t launch_sized(const GemmParams& p, hipStream_t st) {
    constexpr bool HEAVY = EPI == EPI_COMP || EPI == EPI_FOLD_F32;  // small tiles only
    switch (weight_tile(EPI, BRC, p)) {
        case NT_256x256:
            if constexpr (!HEAVY) return launch_nt<256, 256, EPI, false, BRC, 2, false, false, false, 8>(p, st);
            break;
        case NT_256x128:
            if constexpr (!HEAVY) return launch_nt<256, 128, EPI, false, BRC>(p, st);
            break;
        case NT_64x128:
            if constexpr (EPI != EPI_FOLD_F32) return launch_nt<64, 128, EPI, false, BRC>(p, st);
            break;
        default: break;
    }
    return launch_nt<128, 128, EPI, false, BRC>(p, st);
}

template <int EPI, bool BRC>
hipError_t prepare_sized() {
    hipError_t e;
    if constexpr (EPI != EPI_COMP && EPI != EPI_FOLD_F32) {
        if ((e = ensure_attr<256, 256, EPI, false, BRC, 2, false, false, false, 8>()) != hipSuccess) return e;
        if ((e = ensure_attr<256, 256, EPI, false, BRC, 2, true, false, false, 8>()) != hipSuccess) return e;
        if ((e = ensure_attr<256, 128, EPI, false, BRC>()) != hipSuccess) return e;
    }
    if constexpr (EPI != EPI_FOLD_F32)
        if ((e = ensure_attr<64, 128, EPI, false, BRC>()) != hipSuccess) return e;
    return ensure_attr<128, 128, EPI, false, BRC>();
}

}  // namespace

// The tile of a group that has P in bf16
int merge_group_tile(const MergeGroupLayer* layers, int n) {
    int64_t tiles = 0, per_xcd256 = 0, most = 0, least = layers[0].r;  // of 128x128; of 256x256, on an XCD; ranks
    for (int i = 0; i < n; ++i) {
        const MergeGroupLayer& l = layers[i];
        tiles += ((l.out + 127) / 128) * ((l.w_ld + 127) / 128);
        per_xcd256 += (((l.out + 255) / 256) * ((l.w_ld + 255) / 256) + 7) / 8;
        most = std::max<int64_t>(most, l.r), least = std::min<int64_t>(least, l.r);
    }
    if (g_nt_tile_override != 0) return NT_128x128;
    // 64x128 where they take no more rounds, as in weight_tile.  The call for a block of seven weights, us, 128x128 / 64x128 /
    // 64x128 from the codes, by tiles of 128x128 (and of 64x128):
    //         196 (392)           280 (528)             432 (864)             574 (1102)            784 (1552)            1210 (2420)
    //   rank
    //   64    12.8 / 11.7 / 8.4   13.6 / 12.3 / 11.0    14.6 / 15.3 / 12.9    19.0 / 17.1 / 16.4    21.4 / 20.5 / 21.2    26.4 / 26.2 / 28.3
    //   128   13.9 / 12.8 / 9.4   15.5 / 13.8 / 12.5    16.0 / 16.8 / 14.9    20.5 / 18.6 / 18.7    23.0 / 22.2 / 23.9    28.5 / 28.5 / 32.0
    //   256   15.7 / 14.5 / 11.1  17.4 / 15.2 / 15.6    17.9 / 19.1 / 18.3    24.8 / 22.7 / 22.9    28.0 / 27.2 / 30.0    35.1 / 35.1 / 40.3
    //   384   16.6 / 15.2         21.1 / 18.3           21.8 / 23.3           28.0 / 25.9           31.8 / 31.5           40.1 / 40.8
    // Higher ranks, another machine:
    //         196           360           540           616           721           760           784
    //   384   19.6 / 18.2   25.2 / 22.4   31.3 / 28.2   31.8 / 29.1   33.5 / 31.1   34.2 / 31.8   35.4 / 34.7
    //   512   22.5 / 21.1   27.4 / 24.4   34.1 / 31.2   34.5 / 32.0   38.0 / 35.6   37.5 / 35.7   38.8 / 39.1
    //   768   26.0 / 24.0   32.3 / 28.4   41.2 / 37.8   40.9 / 38.4   43.3 / 42.7   43.6 / 42.6   47.1 / 47.4
    //   1024  27.8 / 26.3   36.1 / 32.7   46.6 / 43.5   46.2 / 44.0   49.1 / 49.4   50.2 / 49.7   54.4 / 55.6
    // 768 are two rounds of 64x128, three to a unit; a third one of a few tiles is made up for where the rank is small.
    if (tiles <= 384 || (tiles > 512 && tiles <= (most <= 384 ? 800 : 768))) return NT_64x128;
    // 256x256 where every rank is high and their rounds (tiles of an XCD's 32 units; the last one counts half at least) are hardly
    // more than the group's 128x128 tiles would fill without a gap or a padded edge: up to 1.02 times at rank 640, 1.05 at 1024.
    // The call, 256x256 / 128x128, mean and largest, by that quotient (2400 groups of 7 to 24 weights, hidden sizes of 1536 to 5120):
    //   rank              1.01          1.02          1.03          1.04          1.05          1.06          1.07
    //   640               1.001 1.024   1.006 1.018   1.000 1.012   1.012 1.052   1.007 1.049   1.028 1.054   1.044 1.069
    //   700 to 800        0.979 1.000   0.986 1.014   0.992 1.015   1.008 1.057   1.005 1.078   1.014 1.036   1.035 1.072
    //   800 to 900        0.984 1.001   0.989 1.019   0.988 1.020   1.000 1.047   0.998 1.053   1.005 1.042   1.027 1.059
    //   900 to 1000       0.971 0.978   0.974 0.999   0.981 1.015   0.984 1.041   0.993 1.046   1.000 1.036   1.017 1.041
    //   1024              0.970 1.005   0.976 1.010   0.978 1.008   0.985 1.038   0.987 1.056   0.997 1.024   1.015 1.053
    // (A line by the fill of the last round alone, from rank 512 on, took 256x256 for 14 weights of 1792 x 5016, rank 512, 133 -> 157 us,
    // and for 21 of 1664 x 3584, whose tiles are padded, rank 635, 181 -> 213: 1.030 of the time on the mean.)
    const double rounds = std::min((double)((per_xcd256 + 31) / 32), (double)per_xcd256 / 32.0 + 0.5);
    if (least >= 640 && rounds * 1024.0 <= (0.97 + (double)std::min<int64_t>(least, 1024) / 12800.0) * (double)tiles) return NT_256x256;
    return NT_128x128;
}

hipError_t launch_merge_grouped(int slot, const MergeGroupLayer* layers, int n, hipStream_t st) {
    if (n < 1 || n > MERGE_GROUP_MAX) return hipErrorInvalidValue;
    TimedLaunch tl(slot, st);
    MergeGroupParams g;
    memset(&g, 0, sizeof(g));
    g.n = n;
    for (int i = 0; i < n; ++i) {
        const MergeGroupLayer& l = layers[i];
        MergeGroupItem& it = g.it[i];
        it.A = l.A, it.A_absmax = l.A_absmax, it.lda = l.lda, it.B = l.B, it.ldb = l.ldb;
        it.w_codes = l.w_codes, it.w_absmax = l.w_absmax, it.out_codes = l.out_codes, it.out_absmax = l.out_absmax;
        it.w_ld = l.w_ld, it.M = l.out, it.N = (int)l.w_ld, it.K = l.r, it.w_cols = l.in, it.alpha = l.s;
        if (l.A_absmax && (l.r > A_CODES_TILES * BK || !layers[0].A_absmax)) return hipErrorInvalidValue;
        if (!l.A_absmax && layers[0].A_absmax) return hipErrorInvalidValue;
    }
    if (layers[0].A_absmax) return launch_grouped<64, true>(&g, st);
    switch (merge_group_tile(layers, n)) {
        case NT_256x256: return launch_grouped<256, false>(&g, st);
        case NT_64x128: return launch_grouped<64, false>(&g, st);
        default: return launch_grouped<128, false>(&g, st);
    }
}

hipError_t prepare_weight_kernels() {
    hipError_t e;
    if ((e = prepare_sized<EPI_MERGE, false>()) != hipSuccess) return e;
    if ((e = prepare_sized<EPI_MERGE, true>()) != hipSuccess) return e;
    if ((e = prepare_sized<EPI_FOLD, false>()) != hipSuccess) return e;
    if ((e = prepare_sized<EPI_FOLD, true>()) != hipSuccess) return e;
    if ((e = prepare_sized<EPI_ACC_BF16, true>()) != hipSuccess) return e;
    if ((e = prepare_sized<EPI_COMP, true>()) != hipSuccess) return e;
    if ((e = prepare_sized<EPI_FOLD_F32, true>()) != hipSuccess) return e;
    if ((e = ensure_attr<64, 128, EPI_MERGE, false, true, 2, false, true>()) != hipSuccess) return e;
    if ((e = ensure_attr<64, 128, EPI_FOLD, false, true, 2, false, true>()) != hipSuccess) return e;
    if ((e = launch_grouped<64, true>(nullptr, nullptr)) != hipSuccess) return e;
    if ((e = launch_grouped<64, false>(nullptr, nullptr)) != hipSuccess) return e;
    if ((e = launch_grouped<256, false>(nullptr, nullptr)) != hipSuccess) return e;
    return launch_grouped<128, false>(nullptr, nullptr);
}

// Rounds of an XCD's 32 compute units, each with one 256x256 tile or two of 128x128; the last one by its fill
static double rounds_of_256x256(int64_t tiles) {
    const int64_t x = (tiles + 7) / 8, rest = x & 31;
    return (double)(x >> 5) + (rest ? 0.7 + 0.3 * (double)rest / 32.0 : 0.0);
}
static double rounds_of_128x128(int64_t tiles) {
    const int64_t x = (tiles + 7) / 8, rest = x & 63;
    return (double)(x >> 6) + (rest == 0 ? 0.0 : rest <= 32 ? 0.5 + 0.15 * (double)rest / 32.0 : 0.85 + 0.15 * (double)(rest - 32) / 32.0);
}

int weight_tile(int epi, bool b_rc, const GemmParams& p) {
    auto tiles = [&](int bm, int bn) { return (int64_t)((p.M + bm - 1) / bm) * ((p.N + bn - 1) / bn); };
    if (g_nt_tile_override != 0) return g_nt_tile_override;
    // One 256x256 tile per compute unit, eight waves, moves the least data per product, but has nothing to hide its first loads and its
    // last stores behind, which two resident 128x128 work-groups have, and its rounds of 256 tiles are coarser and padded more.  So
    // the rounds of either are counted, and one of 256x256 takes 1 / `per` of one of 128x128 (two to a unit), a little less the longer
    // the contraction.  Time of the launch, 256x256 / 128x128, by tiles of 256x256 (2048 rows):
    //                      160    192    224    256    320    384    448    512    640    768
    //   fold, rank 64      1.03   0.97   0.93   0.88   1.23   1.12   1.00   1.16   1.08   0.98
    //         256          0.98   0.97   0.88   0.87   1.21   1.08   0.98   1.07   1.02   0.92
    //         512          0.98   0.97   0.89   0.89   1.22   1.07   0.97   1.04   1.00   0.89
    //         1024         0.95   0.96   0.86   0.87   1.16   1.05   0.91   0.94   0.94   0.83
    //   merge, rank 64     1.17   1.07   0.95   0.91   1.20   1.09   0.97   0.95   1.03   0.94
    //         256          1.09   1.01   0.93   0.90   1.15   1.06   0.94   0.90   0.98   0.90
    //         512          1.07   0.95   0.90   0.86   1.15   1.05   0.92   0.89   0.97   0.90
    //         1024         1.00   0.97   0.87   0.86   1.16   1.04   0.94   0.86   0.98   0.86
    //   unquantised merge, rank 256 / 1024
    //                      1.07 / 1.02   0.99 / 0.98   0.96 / 0.89   0.95 / 0.91   1.16   1.10 / 1.06   1.06 / 0.98   1.16 / 0.97   1.07 / 0.96   0.98 / 0.86
    // `per` is from 6000 random launches of 385 tiles of 128x128 and more (512 to 13824 rows and columns, ranks 16 to 1024).  Mean of
    // its choice against 128x128 everywhere and launches that it makes more than 2 % slower, and the same for lines by the fill of the
    // 256x256 rounds and a limit on their padding, which it has replaced:
    //   merge, B K x rows   0.980, 14 of 1705 (0.989, 42: 5632 x 10240, rank 306, 3.4 rounds against 6.9, 82 -> 89 us)
    //          rows x K     0.990, 13 of 879  (0.994, 16)
    //   fold,  B K x rows   0.977, 39 of 1695 (0.988, 22)
    //          rows x K     0.988, 14 of 874  (0.996, 14)
    //   unquantised merge   0.982, 7 of 870   (0.992, 1, but 1152 x 12288, rank 989, was left on 128x128 for its padding, 36 -> 41 us)
    // Over more than one round folds and unquantised merges of low rank are bound by their stores (fold, 5376 x 12068, rank 351, 112 us against 98;
    // merge, 8192 x 8192, rank 256, 75 against 68); in one round
    // folds with B stored K x rows are ahead as soon as 128x128 tiles need a second one (0.93 to 0.99 of the time on the mean).
    // Contractions shorter than a k-tile leave the epilogue, 1600 x 8768, rank 8, 23.4 -> 28.9.
    const int K = p.A[0].K;
    if ((epi == EPI_FOLD || epi == EPI_MERGE || epi == EPI_ACC_BF16) && K >= 64) {
        const int64_t t = tiles(128, 128), t256 = tiles(256, 256);
        const bool one = t256 <= 256;
        const double per = (epi == EPI_FOLD && b_rc && one ? 0.57 : 0.51) + 0.003 * (double)std::min((K + BK - 1) / BK, 16);
        if ((t > 640 || (t > 384 && t <= 512)) && (epi == EPI_MERGE || one || K >= 512) && rounds_of_256x256(t256) < per * rounds_of_128x128(t))
            return NT_256x256;
    }
    // 64x128 tiles on two stages, of which a compute unit holds three: where 128x128, two to a unit, leave room for the 64x128
    // to take no more rounds.  Time of the launch, 64x128 / 128x128, ranks of 96, 300 and 768, by tiles of 128x128:
    //                        208 to 384       448, 512         560, 620        680, 760
    //   fold                 0.86 to 1.02     1.10 to 1.24     0.86 to 1.02    0.99 to 1.16
    //   merge                0.86 to 0.96     1.12 to 1.26     0.86 to 0.97    0.91 to 1.05
    //   compensation step    0.81 to 0.92     1.04 to 1.19     0.87 to 0.96    0.94 to 1.08
    //   unquantised merge    0.96 to 1.06     1.01 to 1.07     0.94 to 1.01    1.02 to 1.13
    // (With three stages and two to a unit they took 1.03 to 1.28 of the time of two stages and three.)
    const int64_t t = tiles(128, 128);
    if (epi != EPI_FOLD_F32 && (t <= 384 || (t > 512 && t <= 640))) return NT_64x128;
    return NT_128x128;
}

// A small weight of low rank reads P as its codes: every work-group expands its 64 rows of P in LDS, which saves the launch that
// would write them out.  That pays as long as all tiles of 64x128 are resident at once, two to a unit (the panel of P costs the
// third); from there on the work-groups that follow each pay for their panel.  The call, us, rank 64 / 256, with the launch and
// without, by tiles:
//                      merge                              forward, 2048 tokens
//   32  (512 x 512)    9.6 -> 6.6,   9.4 -> 7.9           13.0 -> 11.1, 14.1 -> 13.0
//   192 (2048 x 768)   8.7 -> 6.1,   9.6 -> 8.0           20.1 -> 18.1, 20.5 -> 19.7
//   512 (2048 x 2048)  9.1 -> 7.1,   11.0 -> 9.6          31.2 -> 29.2, 32.7 -> 31.6
//   768 (2048 x 3072)  10.2 -> 10.8, 12.8 -> 15.3         42.0 -> 41.2, 44.2 -> 45.4
//   2048 (4096 x 4096) 19.2 -> 19.3, 25.1 -> 25.0         74.5 -> 74.1, 79.2 -> 78.3
bool weight_takes_codes(int64_t out, int64_t in, int64_t r) {
    return !g_nt_tile_override && r <= A_CODES_TILES * BK && codes_tiles(out, in) <= 512;
}
int64_t codes_tiles(int64_t out, int64_t in) { return ((out + 63) / 64) * ((in + 127) / 128); }
// (A group saves a longer launch; figures at launch_merge_grouped.)
bool group_takes_codes(int64_t r, int64_t tiles) {
    return !g_nt_tile_override && ((r <= A_CODES_TILES * BK && tiles <= 512) || (r <= 128 && tiles <= 900));
}

hipError_t launch_weight_product(int epi, bool b_rc, const GemmParams& p, hipStream_t st) {
    if (p.A[0].absmax) {
        if (!b_rc || p.A[0].K > A_CODES_TILES * BK) return hipErrorInvalidValue;
        if (epi == EPI_MERGE) return launch_nt<64, 128, EPI_MERGE, false, true, 2, false, true>(p, st);
        if (epi == EPI_FOLD) return launch_nt<64, 128, EPI_FOLD, false, true, 2, false, true>(p, st);
        return hipErrorInvalidValue;
    }
    switch (epi) {
        case EPI_MERGE: return b_rc ? launch_sized<EPI_MERGE, true>(p, st) : launch_sized<EPI_MERGE, false>(p, st);
        case EPI_FOLD: return b_rc ? launch_sized<EPI_FOLD, true>(p, st) : launch_sized<EPI_FOLD, false>(p, st);
        case EPI_COMP: return b_rc ? launch_sized<EPI_COMP, true>(p, st) : hipErrorInvalidValue;
        case EPI_FOLD_F32: return b_rc ? launch_sized<EPI_FOLD_F32, true>(p, st) : hipErrorInvalidValue;
        case EPI_ACC_BF16: return b_rc ? launch_sized<EPI_ACC_BF16, true>(p, st) : hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

}  // namespace loqt
