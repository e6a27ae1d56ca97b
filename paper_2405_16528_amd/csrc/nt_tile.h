// One output tile of the products of gemm_nt.hip and gemm_weight.hip:
//
//   C[M x N] = alpha * sum_seg  A_seg[M x K_seg] * B_seg[K_seg x N]        (fp32 accumulate)
//
// with both operands bf16, each stored either rows x K (K contiguous) or K x rows (rows contiguous).
// NF4 operands are dequantised to bf16 once per call (nf4_dequantize_kernel, or the fold epilogue
// below) instead of once per output tile; at thousands of tokens that costs a few per cent of the
// GEMM and keeps every VALU and LDS cycle of the inner loop for feeding the matrix cores.  The exception is the A of
// a small weight's fold or merge (ANF4), whose whole cost is its launches.
//
// Work-group: 4 waves that multiply (2 x 2), or 8 (2 x 4, NW), or 4 and as many that only load (LOADERS); tile BM x BN x 64,
// v_mfma_f32_16x16x32_bf16: the same flops per cycle and the same LDS bytes as v_mfma_f32_32x32x16_bf16, the same bits, but a
// quarter of the accumulator registers read and written per instruction (a few per cent of clock on this power-limited part) and
// independent accumulators for the small tiles.
//  * operand tiles go from global memory straight into LDS (global_load_lds_dwordx4, no registers, no
//    ds_write) into a ring of NS stages.  Where every wave loads, the loads of a tile are issued one by one between the MFMAs, spread
//    over the slots, never in a burst (the memory pipeline of a compute unit limits the requests in flight, and a
//    stalled load holds back the MFMAs behind it in the in-order wave).  Loads past the end of the range fetch the last
//    tile once more, into a stage nobody reads.  A k-tile that is not full (the last one of a K segment that is not a
//    multiple of 64) is loaded like any other, lanes past the end fetching a valid chunk, and what lies past the end is
//    cleared in LDS (cut_tile);
//  * two stages: two barriers per k-tile -- one as soon as the tile's last fragments are in registers, which frees its stage
//    for the tile after next, one that publishes the next tile -- so a load has 1.25 to 2 k-tiles to land.  Three or four
//    stages: the fragments of a whole k-tile are double-buffered, one barrier per k-tile publishes the next tile and frees the
//    stage of the running one, and a load has NS - 1 k-tiles to land;
//  * 16-byte chunks of an LDS row are XOR-swizzled so that fragment reads are free of bank conflicts; the swizzle is applied
//    on the global side (which chunk a lane fetches), the LDS side of a direct load is lane-linear;
//  * K-contiguous tiles are read back with one 16-byte read per fragment, row-contiguous tiles
//    with two transposing reads (ds_read_b64_tr_b16): no operand is ever transposed in memory;
//  * the instruction order of the loop is fixed by hand (a scheduling fence after every MFMA slot);
//  * the accumulators are kept transposed (lane = row m, registers = 4 consecutive n) so the
//    epilogues can pack along n: bf16 results are staged through LDS and leave as whole
//    16-byte-per-lane row segments; the fold epilogue adds the dequantised NF4 weight on the way;
//    the merge epilogue requantises 64-blocks in registers (paper sec. 5.1, Alg. 1 line 5);
//  * tiles are dealt to the 8 XCDs in contiguous ranges and walked in groups of 4 or 8 tile rows so that the
//    work-groups sharing an L2 also share operand panels.
// The 256x256 kernels use nearly every vector register; tests/test_isa_guard.py checks their generated loop.
#pragma once
#include <type_traits>

#include "loqt_internal.h"

namespace loqt {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

constexpr int BK = 64;
constexpr int ROWB = 128;  // bytes of one LDS row (64 bf16)

#define LOQT_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

// ANF4: A is NF4 and short (A_CODES_TILES k-tiles at most).  Its rows are expanded into a panel in LDS while the first tiles of B
// are on their way (a few hundred cycles of look-ups per work-group at rank 256), and the loop loads B alone.
constexpr int A_CODES_TILES = 4;

template <int BM, int BN, int NS = 2, bool ANF4 = false, int NW = 4>
struct NtCfg {
    static constexpr int THREADS = NW * 64, WAVES_N = NW / 2;  // that multiply; waves along the columns of the tile
    static constexpr int WTM = BM / 2, WTN = BN / WAVES_N;     // wave tile
    static constexpr int TM = WTM / 16, TN = WTN / 16; // 16x16 tiles per wave
    static constexpr int ASTAGE = ANF4 ? 0 : BM * ROWB; // bytes of A in a stage
    static constexpr int STAGE = ASTAGE + BN * ROWB;
    static constexpr int NCHA = ASTAGE / (THREADS * 16);         // 16-byte chunks per thread per stage that belong to A
    static constexpr int NCHB = BN * ROWB / (THREADS * 16);               // and to B
    static constexpr int NCH = NCHA + NCHB;
    static constexpr int PANEL = ANF4 ? A_CODES_TILES * BM * ROWB : 0;
    static constexpr int HEAD = PANEL + (ANF4 ? BM * BN / 2 : 0);  // the panel and the old codes of the tile, ahead of the ring
    static constexpr int EPITCH = WTN * 2 + 16;        // staging pitch of the bf16 epilogue: 16-byte rows, no bank conflicts beyond two lanes
    static constexpr int SMEM = HEAD + NS * STAGE;     // NS stages: tiles kt .. kt+NS-1 are in LDS or in flight
    static_assert(STAGE >= NW * 32 * EPITCH || HEAD >= NW * 32 * EPITCH, "room to stage 32 rows of each wave");
    static constexpr int PER_CU = SMEM <= 52 * 1024 ? 3 : SMEM <= 78 * 1024 ? 2 : 1;  // work-groups that share a compute unit
};

// the larger of a and of the value the lanes 16, 32 and 48 further on hold (all four lanes of a column of the wave get it)
__device__ __forceinline__ float max_over_lane_groups(float a) {
    const uint32_t u = __float_as_uint(a);
    const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(u, u, false, false));
    const uint32_t v = __float_as_uint(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
    const u32x2 q = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(v, v, false, false));
    return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

// One output tile.  L: index of the tile in the walk order described above (tiles past the end return at once);
// split: slice of the contraction (EPI_F32_SPLITK), else 0.
// NOTAIL: every K segment is a whole number of k-tiles, so no tile has to be cut (cut_tile).
// LOADERS: eight waves, of which four load.
// NW: waves that multiply, 2 x NW / 2 of them over the tile.  Eight: the 256x256 tiles whose epilogue walks the weight.  The loop is no
// faster for the second wave on a SIMD, the epilogue is: 28900 cycles with four waves, 13700 with eight (merge), 12300 and 9000
// (fold), of 65000 to 80000 in all at rank 1024.
template <int BM, int BN, int EPI, bool ARC, bool BRC, int NS = 2, bool NOTAIL = false, bool ANF4 = false, bool LOADERS = false, int NW = 4>
__device__ __forceinline__ void nt_gemm_tile(const GemmParams& p, const int L, const int split) {
    using Cfg = NtCfg<BM, BN, NS, ANF4, NW>;
    constexpr int NT = Cfg::THREADS, PASS = NT * 16;  // bytes of one chunk per thread
    static_assert(NW == 4 || (!LOADERS && !ANF4), "");
    constexpr int TM = Cfg::TM, TN = Cfg::TN, STAGE = Cfg::STAGE, WTM = Cfg::WTM, WTN = Cfg::WTN;
    constexpr bool ENCODES = EPI == EPI_MERGE || EPI == EPI_COMP;
    constexpr bool CODES = EPI == EPI_MERGE || EPI == EPI_FOLD || EPI == EPI_FOLD_F32;  // reads the old 4-bit weight
    // Epilogues that walk the weight: the columns of a wave are dealt to the accumulator tiles so that a lane ends up with
    // eight neighbours.  Within 64 columns, slot 4 g + e of tile t holds column 32 (t / 2) + 8 g + 4 ((t ^ g) & 1) + e, so
    // lane group g has columns 8 g .. 8 g + 7 of either half: the eight codes of one dword, 16 bytes in bf16.  (Which of the two
    // tiles holds the lower four alternates with g, because the transposing reads of one tile would otherwise all ask for the
    // same half of their 16-byte chunks, half of the banks.)
    constexpr bool WEIGHT = ENCODES || CODES || EPI == EPI_ACC_BF16;
    static_assert(!WEIGHT || WTN % 64 == 0, "");
    static_assert(!ANF4 || (CODES && !ARC && NS == 2), "");
    static_assert(!LOADERS || (!WEIGHT && (NS == 3 || NS == 4)), "");
    extern __shared__ __attribute__((aligned(16))) char smem[];

    // (LOADERS: the second four waves load, with the indexes of the first four)
    const int tid = LOADERS ? threadIdx.x & 255 : threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / Cfg::WAVES_N, wn = wave % Cfg::WAVES_N;
    const int wave_s = __builtin_amdgcn_readfirstlane(wave);
    const int frow = lane & 15, g4 = lane >> 4;  // lane = 16 g4 + frow

    // tables of the epilogues that decode or encode NF4, in static LDS (their reads need no base register) and filled here:
    // the barriers of the main loop lie between
    __shared__ Nf4EncTables enc_tables;
    __shared__ float2 level_table[256];
    // the levels of four codes in half `sh` (0 or 16) of cw (element e in byte e / 2, even e in the high nibble): a table entry
    // holds both levels of a byte
    auto levels4 = [&](uint32_t cw, int sh, float* q) {
        const uint32_t hw = cw >> sh;
        const char* const t = reinterpret_cast<const char*>(level_table);
        const float2 a = *reinterpret_cast<const float2*>(t + ((hw << 3) & 0x7f8u)), b = *reinterpret_cast<const float2*>(t + ((hw >> 5) & 0x7f8u));
        q[0] = a.x, q[1] = a.y, q[2] = b.x, q[3] = b.y;
    };
    if constexpr (ENCODES) {
        if (tid >= 64 && tid < 128) nf4_enc_tables_fill(&enc_tables, tid - 64);
    }
    if constexpr (ENCODES || CODES) {
        if (NT == 256 || tid < 256) level_table[tid] = make_float2(kNf4Levels[tid >> 4], kNf4Levels[tid & 15]);
    }

    // ---- tile of this work-group: contiguous range per XCD, groups of GM tile rows inside
    const int tiles_m = (p.M + BM - 1) / BM;
    const int tiles_n0 = (p.N + BN - 1) / BN, tiles_n = tiles_n0 + (p.Nx + BN - 1) / BN;
    if (L >= tiles_m * tiles_n) return;
    constexpr int GM = (EPI == EPI_BF16 && !ARC && !BRC) ? 4 : 8;  // measured per operand layout
    const int gid = L / (GM * tiles_n);
    const int first_m = gid * GM;
    const int gsz = min(tiles_m - first_m, GM);
    const int rem = L - gid * GM * tiles_n;
    const int tm = first_m + rem % gsz;
    int tn = rem / gsz;
    const bool part1 = tn >= tiles_n0;  // second column range
    if (part1) tn -= tiles_n0;
    const int m0 = tm * BM, n0 = tn * BN;
    const int N = part1 ? p.Nx : p.N;
    const float alpha = part1 ? p.alphax : p.alpha;

    const int nkt0 = (p.A[0].K + BK - 1) / BK;
    const int nkt1 = (p.A[1].K + BK - 1) / BK;
    int kt_begin = 0, kt_end = nkt0 + nkt1;
    if (EPI == EPI_F32_SPLITK) {
        const int per = (kt_end + p.splits - 1) / p.splits;
        kt_begin = split * per;
        kt_end = min(kt_end, kt_begin + per);
    }

    // 16x16 tiles (i, j) of the wave tile: lane = row 16 i + (lane & 15), register r = slot 4 (lane >> 4) + r of tile j
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

    // the old block scales of this lane's rows are fetched here, ahead of the product, so that the epilogue does not start with
    // a round trip to memory
    constexpr int NB = WTN / 64 > 0 ? WTN / 64 : 1;  // 64-blocks of the wave's columns
    float am_old[CODES ? TM : 1][NB];
    if constexpr (CODES) {
        const int64_t lda = p.w_ld >> 6;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int m = min(m0 + wm * WTM + i * 16 + frow, p.M - 1);
                const int nb = n0 + wn * WTN + b * 64;
                am_old[i][b] = p.w_absmax[m * lda + ((nb < p.w_ld ? nb : n0) >> 6)];
            }
    }

    // ---- staging.  Chunk i of this thread is LDS slot (i*256 + tid) of the operand tile (the LDS side
    // of a direct load is lane-linear); which 16 bytes of global memory go there carries the swizzle.
    //  K-contiguous operand (rows x K): tile [row][64 k], slot -> row slot>>3, physical chunk slot&7,
    //    logical chunk (slot&7) ^ swz(row); rows are i*32 apart, so the chunk column is the same for all i.
    //  row-contiguous operand (K x rows): tile [64 k][BR rows], slot -> k = slot / (BR/8), physical chunk
    //    slot % (BR/8), logical chunk physical ^ swz(k); read back transposed by ds_read_b64_tr_b16.  Half a
    //    wave of such a read touches 8 k rows x 32 bytes; a row of 128 or more rows is a multiple of 256 bytes (all 64
    //    banks), so the XOR has to move the eight k rows (kk & 3 and bit 3 of kk tell them apart) to eight different places.
    // Addresses are a wave-uniform 64-bit base (operand pointer + tile origin + K offset, scalar
    // registers) plus a 32-bit per-lane byte offset inside the tile's rows, so the loads use the
    // scalar-base form and no 64-bit address arithmetic runs on the vector unit.
    //
    // XOR of the chunk index of row `row` of a K-contiguous tile.  A 16-byte LDS read is served in sets of
    // 16 lanes, {0-3, 12-15, 20-23, 24-27} and {4-7, 8-11, 16-19, 28-31} of each half-wave (measured), and a row is
    // half the banks.  A set holds rows 0-3 and 12-15 of one chunk column and rows 4-11 of the next; with the columns dealt
    // out in eights (WEIGHT, B only) it holds four rows of each of four groups of eight.
    auto kc_swz = [](auto dealt_tag, int row) {
        if constexpr (decltype(dealt_tag)::value) {
            return ((row >> 1) & 1) | (((row >> 3) & 3) << 1);
        } else {
            const int e = (row >> 1) & 7;
            return (e & 1) | ((e & 2) << 1) | ((e & 4) >> 1);
        }
    };
    // XOR of the chunk index of k row kk of a row-contiguous tile of 8 cpr rows.  A 64-row tile has rows of 128 bytes, half the
    // banks: there bit 0 of kk tells two rows apart already.
    auto rc_swz = [](auto dealt_tag, int kk, int cpr) {
        if (cpr == 8) return 2 * ((kk >> 1) & 1) ^ 4 * ((kk >> 3) & 1);
        return (4 * (kk & 3)) ^ (decltype(dealt_tag)::value ? 1 : 2) * ((kk >> 3) & 1);
    };
    using PlainTag = std::integral_constant<bool, false>;
    using BTag = std::integral_constant<bool, WEIGHT>;
    // the operand of K segment `seg`, field by field (selects on scalars: a run-time index into the by-value
    // parameter block, or a copy of an Operand, would go through scratch memory)
    auto a_ptr = [&](bool seg) { return seg ? p.A[1].ptr : p.A[0].ptr; };
    auto a_ld = [&](bool seg) { return seg ? p.A[1].ld : p.A[0].ld; };
    auto a_rows = [&](bool seg) { return seg ? p.A[1].rows : p.A[0].rows; };
    auto b_ptr = [&](bool seg) { return part1 ? p.Bx.ptr : (seg ? p.B[1].ptr : p.B[0].ptr); };
    auto b_ld = [&](bool seg) { return part1 ? p.Bx.ld : (seg ? p.B[1].ld : p.B[0].ld); };
    auto b_rows = [&](bool seg) { return part1 ? p.Bx.rows : (seg ? p.B[1].rows : p.B[0].rows); };
    // index of the cut tile of each segment, or -1
    const int tail0 = (p.A[0].K % BK) ? nkt0 - 1 : -1, tail1 = (p.A[1].K % BK) ? nkt0 + nkt1 - 1 : -1;
    auto is_tail = [&](int t) { return !NOTAIL && (t == tail0 || t == tail1); };

    // The lane offsets of a thread's chunks are loop-invariant registers (per K segment) and the tile origin is a scalar
    // pointer that advances by a constant, so a load is one instruction plus scalar bookkeeping and can sit between MFMAs.
    constexpr int CCPR = BN / 32, CRPP = NT / CCPR, NCC = BM / CRPP;  // old codes: 16-byte chunks per row, rows per pass, passes
    uint32_t offA[ANF4 ? NCC : Cfg::NCHA], offB[Cfg::NCHB];
    const char *hotA = nullptr, *hotB = nullptr;  // operand bytes of the tile that is loaded next
    int64_t stepA = 0, stepB = 0;
    // (kleft: what is left of the segment's contraction from k0 on.  The loads of a tile that is not full repeat a
    // valid chunk or k row in place of those past the end; cut_tile then clears them.)
    auto hot_operand = [&](auto rc_tag, auto br_tag, auto dealt_tag, const void* optr, int64_t old, int orows, int row0, int k0,
                           int kleft, uint32_t* off, const char*& base, int64_t& step) {
        constexpr bool RC = decltype(rc_tag)::value;
        constexpr int BR = decltype(br_tag)::value;
        constexpr int NC = BR * ROWB / PASS;
        // a tile that lies wholly past the operand's last row (the merge walks the padding columns of the
        // code matrix, which can exceed `in` by more than a tile) reads the operand's first rows instead:
        // its products are never used, and the clamps below then never go negative
        if (row0 >= orows) row0 = 0;
        const uint32_t ld2 = (uint32_t)old * 2u;  // row pitch in bytes (a tile spans < 2^32 bytes)
        if constexpr (!RC) {
            const int r0 = tid >> 3;
            const int kc = (tid & 7) ^ kc_swz(dealt_tag, r0);
            const int rlast = orows - 1 - row0;  // rows past the end: any valid row
            const uint32_t kb = NOTAIL || kc * 8 < kleft ? (uint32_t)kc * 16u : 0u;
#pragma unroll
            for (int i = 0; i < NC; ++i) off[i] = (uint32_t)min(i * (NT / 8) + r0, rlast) * ld2 + kb;
            base = reinterpret_cast<const char*>(optr) + ((int64_t)row0 * old + k0) * 2;
            step = BK * 2;
        } else {
            constexpr int CPR = BR / 8;     // chunks per k row
            constexpr int KPI = NT / CPR;   // k rows covered by one pass of the threads
            const int kq = tid / CPR;
            const int clast = (((orows - 1) >> 3) << 3) - row0;  // columns past the end: any valid chunk
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                const int logical = (tid % CPR) ^ rc_swz(dealt_tag, kq + i * KPI, CPR);
                const int kr = NOTAIL ? kq + i * KPI : min(kq + i * KPI, kleft - 1);
                off[i] = (uint32_t)kr * ld2 + (uint32_t)min(logical * 8, clast) * 2u;
            }
            base = reinterpret_cast<const char*>(optr) + ((int64_t)k0 * old + row0) * 2;
            step = (int64_t)BK * old * 2;
        }
    };
    auto hot_setup = [&](int kt) {  // kt: a tile of the range
        const bool seg = kt >= nkt0;
        const int k0 = (kt - (seg ? nkt0 : 0)) * BK;
        const int kleft = (seg ? p.A[1].K : p.A[0].K) - k0;
        if constexpr (!ANF4)
            hot_operand(std::integral_constant<bool, ARC>{}, std::integral_constant<int, BM>{}, PlainTag{}, a_ptr(seg), a_ld(seg),
                        a_rows(seg), m0, k0, kleft, offA, hotA, stepA);
        hot_operand(std::integral_constant<bool, BRC>{}, std::integral_constant<int, BN>{}, BTag{}, b_ptr(seg), b_ld(seg),
                    b_rows(seg), n0, k0, kleft, offB, hotB, stepB);
    };
    // The old codes of the tile (BN / 2 bytes a row) follow the last k-tile as if they were the next one's A: they land under
    // the last k-tiles' products and wait in LDS for the epilogue (fetched by it, they took as long as two or three k-tiles).
    // The swizzle keeps the reads of 16 rows apart.
    auto code_swz = [](int row) { return CCPR == 8 ? (row >> 1) & 7 : (row >> 2) & 3; };
    auto codes_setup = [&]() {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));  // (else its results are worked out ahead of the loop and copied, or reloaded, in every iteration)
        const uint32_t ldb = (uint32_t)(p.w_ld >> 1);
#pragma unroll
        for (int i = 0; i < (ANF4 ? NCC : Cfg::NCHA); ++i) {
            const int row = (i < NCC ? i : 0) * CRPP + tid / CCPR;
            const int ch = (tid % CCPR) ^ code_swz(row);
            offA[i] = (uint32_t)min(row, p.M - 1 - m0) * ldb + (n0 + ch * 32 < p.w_ld ? (uint32_t)ch * 16u : 0u);
        }
        hotA = reinterpret_cast<const char*>(p.w_codes) + (int64_t)m0 * (p.w_ld >> 1) + (n0 >> 1);
    };
    auto hot_advance = [&](int kt) {  // move on to tile kt, the successor of the current one
        if (kt >= kt_end) {
            if constexpr (CODES && !ANF4) {
                if (kt == kt_end) codes_setup();
            }
            return;
        }
        if (kt == nkt0 || is_tail(kt)) hot_setup(kt);
        else hotA += stepA, hotB += stepB;
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)LOQT_LDS_PTR(smem);
    char* const ring = smem + Cfg::HEAD;
    // Load n of a tile (chunks of A, then of B) into `stage`.  Inline assembly: the compiler cannot tell that the LDS reads of
    // the running tile never touch the stage the loads in flight are writing, and would wait for all of them (vmcnt(0))
    // before every group of transposing reads; written this way it does not see them, and the loop waits for them itself
    // before each barrier.  No EXEC mask: a wave issues at most one instruction every four cycles, and the six-instruction
    // form between two MFMAs of sixteen cycles each holds the second one back.  Tiles past the end of the contraction
    // are not masked either: the tile pointers stop advancing, so such a load fetches the last tile once more
    // into a stage nobody reads again (the loop's exit waits for them before LDS is reused).
    // A load that takes its LDS address from M0 may not be the very next instruction after the write of M0 (one wait state; the
    // compiler keeps to it in its own code and does not look inside an assembly string).  So M0 gets the sum of the stage and the
    // chunk's place in it, which would be an instruction anyway, and an s_nop follows: as many instructions as the sum, a move and
    // the load.
    // M0 cannot be named as a clobber (the compiler reserves it and warns that a clobber is not honoured): it
    // never keeps a value in M0 across other code, it writes M0 right in front of each of its own uses.
    // tests/test_isa_guard.py checks that nothing else in the loop touches M0, and the wait state.
    auto direct_load = [&](uint32_t o, const char* base, uint32_t dst, uint32_t at) {
        asm volatile(
            "s_add_u32 m0, %2, %3\n\t"
            "s_nop 0\n\t"
            "global_load_lds_dwordx4 %0, %1"
            :
            : "v"(o), "s"(base), "s"(dst), "i"(at)
            : "memory", "scc");
    };
    auto hot_load = [&](int n, char* stage) {
        const bool isA = n < Cfg::NCHA;
        const int i = isA ? n : n - Cfg::NCHA;
        const uint32_t dst = lds0 + (uint32_t)(stage - smem) + (uint32_t)(wave_s * 1024);
        direct_load(isA ? offA[i] : offB[i], isA ? hotA : hotB, dst, (uint32_t)((isA ? 0 : Cfg::ASTAGE) + i * PASS));
    };
    // Tile kt of the range has landed in `stage` by direct loads and ends past its segment's contraction: clears
    // everything from there on, in both operands (what came instead is finite, but the padding of a row need not be).
    // The slots of LDS are those of the staging above.  A barrier has to follow.
    auto cut_operand = [&](auto rc_tag, auto br_tag, auto dealt_tag, int kleft, char* tile) {
        constexpr bool RC = decltype(rc_tag)::value;
        constexpr int BR = decltype(br_tag)::value;
        constexpr int NC = BR * ROWB / PASS;
        if constexpr (!RC) {
            const int nv = kleft - 8 * ((tid & 7) ^ kc_swz(dealt_tag, tid >> 3));  // valid elements of this thread's chunk column
            if (nv < 8) {
                uint32_t keep[4];
#pragma unroll
                for (int d = 0; d < 4; ++d) keep[d] = 2 * d + 1 < nv ? 0xffffffffu : 2 * d < nv ? 0xffffu : 0u;
#pragma unroll 1
                for (int i = 0; i < NC; ++i) {
                    uint4* q = reinterpret_cast<uint4*>(tile + i * PASS + tid * 16);
                    const uint4 v = *q;
                    *q = make_uint4(v.x & keep[0], v.y & keep[1], v.z & keep[2], v.w & keep[3]);
                }
            }
        } else {
            constexpr int CPR = BR / 8, KPI = NT / CPR;
#pragma unroll 1
            for (int i = 0; i < NC; ++i)
                if (i * KPI + tid / CPR >= kleft) *reinterpret_cast<uint4*>(tile + i * PASS + tid * 16) = make_uint4(0, 0, 0, 0);
        }
    };
    auto cut_tile = [&](int kt, char* stage) {
        const bool seg = kt >= nkt0;
        const int kleft = (seg ? p.A[1].K : p.A[0].K) - (kt - (seg ? nkt0 : 0)) * BK;
        if constexpr (!ANF4) cut_operand(std::integral_constant<bool, ARC>{}, std::integral_constant<int, BM>{}, PlainTag{}, kleft, stage);
        cut_operand(std::integral_constant<bool, BRC>{}, std::integral_constant<int, BN>{}, BTag{}, kleft, stage + Cfg::ASTAGE);
    };
    // ANF4: the panel of A.  Chunk i of this thread is the same slot of the same tile layout as above; the codes of all k-tiles are
    // asked for at once, ahead of the first tiles of B.
    constexpr int PR = ANF4 ? BM / 32 : 1, PT = ANF4 ? A_CODES_TILES : 1;
    uint32_t pcode[PR][PT];
    float pscale[PR][PT];
    const int pk = ((tid & 7) ^ kc_swz(PlainTag{}, tid >> 3)) * 8;  // first k of this thread's chunks in a k-tile
    auto panel_load = [&]() {
        const Operand& a = p.A[0];
#pragma unroll
        for (int i = 0; i < PR; ++i) {
            const int64_t row = min(m0 + i * 32 + (tid >> 3), a.rows - 1);  // rows past the end: any valid row
            const uint8_t* c = reinterpret_cast<const uint8_t*>(a.ptr) + row * (a.ld >> 1) + (pk >> 1);
            const float* s = a.absmax + row * (a.ld >> 6);
#pragma unroll
            for (int t = 0; t < PT; ++t) {
                const int kt = min(t, nkt0 - 1);
                pcode[i][t] = *reinterpret_cast<const uint32_t*>(c + kt * (BK / 2));
                pscale[i][t] = s[kt];
            }
        }
    };
    auto panel_expand = [&]() {  // (the same products and the same rounding as nf4_dequantize_kernel's)
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            if (t >= nkt0) break;
            const int left = p.A[0].K - t * BK - pk;  // elements of this thread's chunks that exist
#pragma unroll
            for (int i = 0; i < PR; ++i) {
                float q[8];
                levels4(pcode[i][t], 0, q);
                levels4(pcode[i][t], 16, q + 4);
#pragma unroll
                for (int e = 0; e < 8; ++e) q[e] = e < left ? pscale[i][t] * q[e] : 0.f;
                *reinterpret_cast<uint4*>(smem + t * (BM * ROWB) + i * 4096 + tid * 16) =
                    make_uint4(pack_bf16(q[0], q[1]), pack_bf16(q[2], q[3]), pack_bf16(q[4], q[5]), pack_bf16(q[6], q[7]));
            }
        }
    };

    // ---- fragments.  A lane holds row (lane & 15) of a 16-row fragment and the 8 k-values 32*ks + 8*(lane >> 4) .. +7.
    // K-contiguous tiles: one 16-byte read of logical chunk 4*ks + (lane >> 4).  Row-contiguous tiles: two transposing 8-byte
    // reads; within a group of 16 lanes, lane 4*jj + q supplies the address of k row 8*(lane >> 4) + jj, slots 4q..4q+3, and
    // receives the four k of slot (lane & 15).
    auto read_tr = [&](const char* ptr, int pitch) -> bf16x8 {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4*)(ptr));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4*)(ptr + 4 * pitch));
        const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, v);
    };
    uint32_t a_ko[2], b_ko[2][WEIGHT ? 2 : 1];  // K-contiguous tiles: byte offset of this lane's fragment row and chunk per k32 step
    int a_rc[ARC ? TM : 1], b_rc[BRC ? TN : 1];
    {
        const int jj = (lane >> 2) & 3, q = lane & 3;
        const int g = frow >> 2;  // group of four slots of this lane's B row
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            a_ko[ks] = (uint32_t)((wm * WTM + frow) * ROWB + (((4 * ks + g4) ^ kc_swz(PlainTag{}, frow)) << 4));
            if constexpr (WEIGHT) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {  // even and odd tiles
                    const int row = 8 * g + 4 * ((t ^ g) & 1) + (frow & 3);
                    b_ko[ks][t] = (uint32_t)(Cfg::ASTAGE + (wn * WTN + row) * ROWB + (((4 * ks + g4) ^ kc_swz(BTag{}, row)) << 4));
                }
            } else {
                b_ko[ks][0] = (uint32_t)(Cfg::ASTAGE + (wn * WTN + frow) * ROWB + (((4 * ks + g4) ^ kc_swz(BTag{}, frow)) << 4));
            }
        }
        if constexpr (ARC) {
#pragma unroll
            for (int u = 0; u < TM; ++u) {
                const int chunk = ((wm * WTM + u * 16) >> 3) + (q >> 1);
                a_rc[u] = (8 * g4 + jj) * (BM * 2) + ((chunk ^ rc_swz(PlainTag{}, 8 * g4 + jj, BM / 8)) << 4) + (q & 1) * 8;
            }
        }
        if constexpr (BRC) {
#pragma unroll
            for (int u = 0; u < TN; ++u) {
                const int col = WEIGHT ? (u >> 2) * 64 + ((u >> 1) & 1) * 32 + 8 * q + 4 * ((u ^ q) & 1) : u * 16 + 4 * q;
                const int chunk = (wn * WTN + col) >> 3;
                b_rc[u] = Cfg::ASTAGE + (8 * g4 + jj) * (BN * 2) + ((chunk ^ rc_swz(BTag{}, 8 * g4 + jj, BN / 8)) << 4) + (col & 4) * 2;
            }
        }
    }
    const char* panel = smem;  // ANF4: the running k-tile of A
    // fragment u (those of A first) of k32 step ks of the tile at `stage`
    auto read_frag = [&](int ks, int u, const char* stage) -> bf16x8 {
        if (u < TM) {
            if constexpr (ARC) return read_tr(stage + a_rc[u] + 32 * ks * (BM * 2), BM * 2);
            else return *reinterpret_cast<const bf16x8*>((ANF4 ? panel : stage) + a_ko[ks] + u * 16 * ROWB);
        } else {
            const int j = u - TM;
            if constexpr (BRC) return read_tr(stage + b_rc[j] + 32 * ks * (BN * 2), BN * 2);
            else if constexpr (WEIGHT) return *reinterpret_cast<const bf16x8*>(stage + b_ko[ks][j & 1] + ((j >> 2) * 64 + ((j >> 1) & 1) * 32) * ROWB);
            else return *reinterpret_cast<const bf16x8*>(stage + b_ko[ks][0] + j * 16 * ROWB);
        }
    };
    constexpr int NM = TM * TN, NU = TM + TN;  // MFMAs and fragments of a k32 step
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    if constexpr (LOADERS) {
        // ---- waves of their own for the loads.  A wave issues in order, and a direct load holds it up while the memory pipeline of the
        // compute unit is busy, so of the 1031 to 1100 cycles per k-tile of a 128x128 tile with one wave to a SIMD the matrix units were
        // busy for 512; the products alone took 620, the loads alone 570, the fragment reads alone 420.  Here one wave of a SIMD
        // multiplies and another one loads, with one barrier per k-tile between them: 670 and 760 cycles (B rows x K, K x rows), 256x128
        // 1160 and 1210 instead of 1390 and 1430 (1024 of products), 64x128 590 instead of 720, 64x64 460 instead of 500.  The
        // accumulators of 256x256 leave no registers for a second wave.  Four waves of products, fragments of one k32 step ahead: the
        // barrier of k-tile kt, between its two steps, says that its fragments are in registers, which frees its stage for tile
        // kt + NS, and that tile kt + 1 has landed.
        constexpr int NCH = Cfg::NCH;
        const int nkt = kt_end - kt_begin;
        // all but `later` of the tiles asked for have landed
        auto landed = [&](int later) {
            if (later >= NS - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * NCH) : "memory");
            else if (NS > 3 && later == NS - 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * NCH) : "memory");
            else if (later == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NCH) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        };
        if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 8)) {
            if (nkt > 0) {
                hot_setup(kt_begin);
                for (int t = 0; t < NS && t < nkt; ++t) {
                    if (t > 0) hot_advance(kt_begin + t);
#pragma unroll
                    for (int n = 0; n < NCH; ++n) hot_load(n, smem + t * STAGE);
                }
                landed(min(NS, nkt) - 1);
                __syncthreads();
                if (is_tail(kt_begin)) {
                    cut_tile(kt_begin, smem);
                    __syncthreads();
                }
                int si = 0;
                for (int kt = kt_begin; kt < kt_end; ++kt) {
                    char* const cur = smem + si * STAGE;
                    si = si + 1 == NS ? 0 : si + 1;
                    landed(min(kt_end - 2 - kt, NS - 2));
                    __syncthreads();
                    if (is_tail(kt + 1)) {
                        cut_tile(kt + 1, smem + si * STAGE);
                        __syncthreads();
                    }
                    if (kt + NS < kt_end) {
                        hot_advance(kt + NS);
#pragma unroll
                        for (int n = 0; n < NCH; ++n) hot_load(n, cur);
                    }
                }
            }
            __syncthreads();
            return;
        }
        // 64x64: a k32 step is four products, less than the latency of a read, so the fragments of a whole k-tile are kept ahead and the
        // barrier is between the k-tiles (64 x 64 x 4096 15.0 -> 14.6 us, 1024 x 1024 x 2048 10.5 -> 10.2)
        constexpr bool WHOLE = NM < 8;
        if (nkt > 0) {
            __syncthreads();
            if (is_tail(kt_begin)) __syncthreads();
        }
        int si = 0;
        if constexpr (WHOLE) {
            constexpr int NSL = 2 * NM, RSL = NSL * 3 / 4;  // slots of one MFMA; those that carry fragment reads
            bf16x8 f[2][2][NU];
            if (nkt > 0) {
#pragma unroll
                for (int u = 0; u < 2 * NU; ++u) f[0][u / NU][u % NU] = read_frag(u / NU, u % NU, smem);
            }
            auto ktile = [&](auto par_tag, int kt) {
                constexpr int P = decltype(par_tag)::value;
                si = si + 1 == NS ? 0 : si + 1;
                const char* const nxt = smem + si * STAGE;
                __syncthreads();
                if (is_tail(kt + 1)) __syncthreads();
#pragma unroll
                for (int sl = 0; sl < NSL; ++sl) {
                    const int ks = sl / NM, i = sl % NM / TN, j = sl % TN;
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[P][ks][TM + j], f[P][ks][i], acc[i][j], 0, 0, 0);
                    if (sl < RSL) {
#pragma unroll
                        for (int u = sl * 2 * NU / RSL; u < (sl + 1) * 2 * NU / RSL; ++u) f[P ^ 1][u / NU][u % NU] = read_frag(u / NU, u % NU, nxt);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            for (int kt = kt_begin; kt < kt_end; ++kt) {
                ktile(I0{}, kt);
                if (++kt >= kt_end) break;
                ktile(I1{}, kt);
            }
        } else {
            constexpr int RSL = NM * 5 / 8;  // slots (of one MFMA) that carry fragment reads: the last ones have time to arrive
            bf16x8 f[2][NU];
            // the order in which a step's products ask for the fragments: A's first, B's, the rest of A's
            auto nth = [](int n) { return n == 0 ? 0 : n <= TN ? TM + n - 1 : n - TN; };
            auto step = [&](auto cb_tag, const char* rstage) {  // the MFMAs of k32 step CB, under them the reads of the next step
                constexpr int CB = decltype(cb_tag)::value;
#pragma unroll
                for (int sl = 0; sl < NM; ++sl) {
                    const int i = sl / TN, j = sl % TN;
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[CB][TM + j], f[CB][i], acc[i][j], 0, 0, 0);
                    if (sl < RSL) {
#pragma unroll
                        for (int n = sl * NU / RSL; n < (sl + 1) * NU / RSL; ++n) f[CB ^ 1][nth(n)] = read_frag(CB ^ 1, nth(n), rstage);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            if (nkt > 0) {
#pragma unroll
                for (int n = 0; n < NU; ++n) f[0][nth(n)] = read_frag(0, nth(n), smem);
            }
            for (int kt = kt_begin; kt < kt_end; ++kt) {
                const char* const cur = smem + si * STAGE;
                si = si + 1 == NS ? 0 : si + 1;
                step(I0{}, cur);
                __syncthreads();
                if (is_tail(kt + 1)) __syncthreads();
                step(I1{}, smem + si * STAGE);
            }
        }
    } else if constexpr (NS == 2) {
        // ---- two stages.  A stage is free as soon as the fragments of its second k32 step sit in
        // registers, a quarter of the way into its tile, so its refill does not have to wait for the barrier
        // that publishes the next tile.  Per k-tile kt, in slots of two MFMAs:
        //   first half of k32 step 0 : the fragment reads of step 1
        //   barrier X                : every wave has tile kt in registers, its stage is free
        //   second half of step 0    : the loads of tile kt+2 into that stage, one every LSP-th slot from here on
        //   first half of step 1     : loads
        //   barrier Y                : tile kt+1 has landed (loads return in order: all but those of kt+2 issued so far)
        //   second half of step 1    : loads, and the fragment reads of step 0 of tile kt+1
        // A load so has 1.25 to 1.5 k-tiles (256x256: about 3000 cycles) to land: measured against a library GEMM of the same
        // tile shape, instruction mix and cache traffic, the loop with one barrier per tile (loads issued 0.25 to 1 tile
        // ahead) spent 27 % of its wave cycles waiting where that kernel spent 6 %.
        constexpr int NSL = NM / 2;                              // slots of a k32 step
        constexpr int LSP = (3 * NSL / 2) / Cfg::NCH;            // 256x256: 16 loads over 48 slots
        constexpr int LBY = (NSL + LSP - 1) / LSP < Cfg::NCH ? (NSL + LSP - 1) / LSP : Cfg::NCH;  // of which precede barrier Y
        constexpr int RPQ = (NU + NSL / 2 - 1) / (NSL / 2);      // fragment reads per slot over a quarter of the slots
        static_assert(LSP >= 1, "");
        bf16x8 fa[2][TM], fb[2][TN];
        auto rd = [&](int ks, int nb, int u, const char* stage) {
            if (u < TM) fa[nb][u] = read_frag(ks, u, stage);
            else fb[nb][u - TM] = read_frag(ks, u, stage);
        };
        // slots S0..S1-1 (two MFMAs each) of a k32 step on fragment buffer CB.  RPS > 0: the fragment reads of k32 step
        // RKS of the tile at `rstage` into the other buffer, RPS per slot from the first slot of the range on.  LD >= 0:
        // this range starts at slot LD of the schedule of loads (of the tile at hotA / hotB, into `lstage`), one every
        // LSP-th slot.
        auto slots = [&](auto cb_tag, auto s0_tag, auto s1_tag, auto rd_tag, auto rks_tag, auto ld_tag, const char* rstage,
                         char* lstage) {
            constexpr int CB = decltype(cb_tag)::value, S0 = decltype(s0_tag)::value, S1 = decltype(s1_tag)::value;
            constexpr int RPS = decltype(rd_tag)::value;                 // fragment reads per slot
            constexpr int RKS = decltype(rks_tag)::value, LD = decltype(ld_tag)::value;
#pragma unroll
            for (int sl = S0; sl < S1; ++sl) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int m = 2 * sl + e, i = m / TN, j = m % TN;
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[CB][j], fa[CB][i], acc[i][j], 0, 0, 0);
                }
                const int t = sl - S0;
                if constexpr (RPS > 0) {
#pragma unroll
                    for (int u = t * RPS; u < (t + 1) * RPS && u < NU; ++u) rd(RKS, CB ^ 1, u, rstage);
                }
                if constexpr (LD >= 0) {
                    const int g = LD + t;
                    if (g % LSP == 0 && g / LSP < Cfg::NCH) hot_load(g / LSP, lstage);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        using SH = std::integral_constant<int, NSL / 2>;
        using SE = std::integral_constant<int, NSL>;
        using RQ = std::integral_constant<int, RPQ>;
        using NOLD = std::integral_constant<int, -1>;
        if (kt_begin < kt_end) {
            if constexpr (ANF4) {
                panel_load();
                codes_setup();
#pragma unroll
                for (int i = 0; i < NCC; ++i) direct_load(offA[i], hotA, lds0 + (uint32_t)(wave_s * 1024), (uint32_t)(Cfg::PANEL + i * 4096));
            }
            hot_setup(kt_begin);
#pragma unroll
            for (int n = 0; n < Cfg::NCH; ++n) hot_load(n, ring);
            hot_advance(kt_begin + 1);  // (a range of one tile loads it twice; nobody reads the second copy)
#pragma unroll
            for (int n = 0; n < Cfg::NCH; ++n) hot_load(n, ring + STAGE);
            if constexpr (ANF4) {
                __syncthreads();  // the table of levels
                panel_expand();
            }
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(Cfg::NCH) : "memory");
            __syncthreads();
            if (is_tail(kt_begin)) {
                cut_tile(kt_begin, ring);
                __syncthreads();
            }
#pragma unroll
            for (int u = 0; u < NU; ++u) rd(0, 0, u, ring);
        }
        for (int kt = kt_begin; kt < kt_end; ++kt) {
            char* cur = ring + ((kt - kt_begin) & 1) * STAGE;
            char* nxt = ring + (((kt - kt_begin) & 1) ^ 1) * STAGE;
            slots(I0{}, I0{}, SH{}, RQ{}, I1{}, NOLD{}, cur, cur);
            __syncthreads();  // X: nobody reads `cur` any more
            hot_advance(kt + 2);
            slots(I0{}, SH{}, SE{}, I0{}, I0{}, I0{}, cur, cur);
            slots(I1{}, I0{}, SH{}, I0{}, I0{}, SH{}, cur, cur);
            // tile kt+1 must have landed; the loads of tile kt+2 issued so far came after it and may stay in flight
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LBY) : "memory");
            __syncthreads();  // Y
            if (is_tail(kt + 1)) {
                cut_tile(kt + 1, nxt);
                __syncthreads();
            }
            // harmless stale reads after the last tile
            if constexpr (ANF4) panel += BM * ROWB;
            slots(I1{}, SH{}, SE{}, RQ{}, I0{}, SE{}, nxt, cur);
        }
    } else {
        // ---- three or more stages.  One work-group per compute unit is a chain of barrier, fragment reads and MFMAs per
        // k-tile, so the chain is cut to one of each: the fragments of a whole k-tile are double-buffered in registers, and the
        // one barrier of k-tile kt says both that tile kt+1 has landed and that nobody reads the stage of tile kt any more
        // (its fragments came into registers during tile kt-1).  Under the MFMAs of tile kt go the fragment reads of tile
        // kt+1 and the loads of tile kt+NS into the stage of tile kt.
        constexpr int PER = NM >= 32 ? 2 : 1;     // MFMAs per slot
        constexpr int NSL = 2 * NM / PER;         // slots of a k-tile
        constexpr int RSL = NSL >= 16 ? NSL / 2 : NSL * 3 / 4;  // slots that carry fragment reads, the first ones
        bf16x8 f[2][2][NU];                       // [parity of the tile][k32 step][fragment]
        int si = 0;                               // stage of tile kt
        if (kt_begin < kt_end) {
            hot_setup(kt_begin);
#pragma unroll
            for (int t = 0; t < NS; ++t) {
                if (t > 0) hot_advance(kt_begin + t);
#pragma unroll
                for (int n = 0; n < Cfg::NCH; ++n) hot_load(n, smem + t * STAGE);
            }
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * Cfg::NCH) : "memory");
            __syncthreads();
            if (is_tail(kt_begin)) {
                cut_tile(kt_begin, smem);
                __syncthreads();
            }
#pragma unroll
            for (int u = 0; u < 2 * NU; ++u) f[0][u / NU][u % NU] = read_frag(u / NU, u % NU, smem);
        }
        auto ktile = [&](auto par_tag, int kt) {
            constexpr int P = decltype(par_tag)::value;
            char* cur = smem + si * STAGE;
            si = si + 1 == NS ? 0 : si + 1;
            char* nxt = smem + si * STAGE;
            // tile kt+1 must have landed; the NS - 2 tiles after it may stay in flight
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * Cfg::NCH) : "memory");
            __syncthreads();
            if (is_tail(kt + 1)) {
                cut_tile(kt + 1, nxt);
                __syncthreads();
            }
            hot_advance(kt + NS);
#pragma unroll
            for (int sl = 0; sl < NSL; ++sl) {
#pragma unroll
                for (int e = 0; e < PER; ++e) {
                    const int q = PER * sl + e, ks = q / NM, i = q % NM / TN, j = q % NM % TN;
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[P][ks][TM + j], f[P][ks][i], acc[i][j], 0, 0, 0);
                }
                // (harmless stale reads after the last tile)
                if (sl < RSL) {
#pragma unroll
                    for (int u = sl * 2 * NU / RSL; u < (sl + 1) * 2 * NU / RSL; ++u) f[P ^ 1][u / NU][u % NU] = read_frag(u / NU, u % NU, nxt);
                }
#pragma unroll
                for (int n = sl * Cfg::NCH / NSL; n < (sl + 1) * Cfg::NCH / NSL; ++n) hot_load(n, cur);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        for (int kt = kt_begin; kt < kt_end; ++kt) {
            ktile(I0{}, kt);
            if (++kt >= kt_end) break;
            ktile(I1{}, kt);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loads past the end, before LDS is reused
    __syncthreads();                                  // LDS is free for the epilogue

    // ------------------------------------------------------------------ epilogues
    // where the old codes are: the stage of the k-tile after the last one; the stage after that one is free
    const int nkt = kt_end - kt_begin;
    char* const cbuf = ANF4 ? smem + Cfg::PANEL : smem + (CODES ? nkt % NS : 0) * STAGE;
    char* const ebase = ANF4 ? smem : smem + (CODES ? (nkt + 1) % NS : ENCODES ? 1 : 0) * STAGE;
    // byte offset of the dword of codes of this lane in row 16 i + frow of its wave, columns 32 c + 8 g4 .. +7 of the tile
    auto code_at = [&](int i, int c) {
        return cbuf + (wm * WTM + i * 16 + frow) * (BN / 2) + ((c ^ code_swz(frow)) << 4) + 4 * g4;
    };
    const int sh0 = 16 * (g4 & 1), sh1 = 16 - sh0;  // the half of a dword that belongs to an even and to an odd tile
    // first column (in the tile of the work-group) of this lane's four of accumulator tile j
    auto col_of = [&](int j) {
        if constexpr (WEIGHT) return wn * WTN + (j >> 2) * 64 + ((j >> 1) & 1) * 32 + 8 * g4 + 4 * ((j ^ g4) & 1);
        else return wn * WTN + j * 16 + 4 * g4;
    };

    if constexpr (EPI == EPI_BF16 || EPI == EPI_FOLD || EPI == EPI_ACC_BF16) {
        // 32 rows at a time are staged through the wave's private LDS region and leave as whole 16-byte row segments (LDS operations
        // of one wave complete in order, so no barrier), the stores of one block under way while the next one is computed.  All segments
        // of a block are asked for at once, and a wave that lies inside the matrix (wave-uniform) walks a pointer; with the bounds of
        // every segment tested beside its read, each store waited for its own read and for a 64-bit product (256x256, bf16: the
        // epilogue 13300 cycles before, 6400 to 7900 now).  The same at the edges, by which a launch of one round is held up (y of
        // 2816 x 5862 x 768 36.8 us with one segment after the other there, 33.2 this way).
        constexpr int EPITCH = Cfg::EPITCH;
        char* ebuf = ebase + wave_s * (32 * EPITCH);
        constexpr int CPR = WTN / 8, RPI = 64 / CPR, NIT = 32 / RPI;  // 16-byte chunks per row; rows per store of the wave; stores per block
        uint16_t* C = reinterpret_cast<uint16_t*>(part1 ? p.Cx : p.C);
        const int64_t ldc = part1 ? p.ldcx : p.ldc;
        // (256x256, four waves: asked for anew, so that nothing of the stores has to be kept through the loop.  Elsewhere that costs: an
        // unquantised merge of 7808 x 9793, rank 128, 64.5 us, 69.3 with it.)
        int slane = lane;
        if constexpr (BM == 256 && BN == 256 && NW == 4) asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(slane));
        const int swm = wave_s / Cfg::WAVES_N, swn = wave_s % Cfg::WAVES_N;
        const int srow = slane / CPR, sch = slane % CPR;
        const char* const sread = ebuf + srow * EPITCH + sch * 16;
        const bool inside = m0 + (swm + 1) * WTM <= p.M && n0 + (swn + 1) * WTN <= N;
        uint16_t* sdst = C + (int64_t)(m0 + swm * WTM + srow) * ldc + (n0 + swn * WTN + sch * 8);
        const int64_t sstep = RPI * ldc;
        // rows row0 .. row0+31 of the wave tile
        auto store_rows = [&](int row0) {
            u32x4 v[NIT];
#pragma unroll
            for (int it = 0; it < NIT; ++it) v[it] = *reinterpret_cast<const u32x4*>(sread + it * RPI * EPITCH);
            if (inside) {
#pragma unroll
                for (int it = 0; it < NIT; ++it, sdst += sstep) __builtin_nontemporal_store(v[it], reinterpret_cast<u32x4*>(sdst));
                return;
            }
            const int rows = p.M - (m0 + swm * WTM + srow), cols = N - (n0 + swn * WTN + sch * 8);  // left, from the lane's first segment on
            if (cols >= 8) {
#pragma unroll
                for (int it = 0; it < NIT; ++it)
                    if (row0 + it * RPI < rows) __builtin_nontemporal_store(v[it], reinterpret_cast<u32x4*>(sdst + it * sstep));
            } else if (cols > 0) {  // the end of the rows: four, two and one elements
#pragma unroll
                for (int it = 0; it < NIT; ++it) {
                    if (row0 + it * RPI >= rows) continue;
                    uint16_t* const d = sdst + it * sstep;
                    if (cols & 4) *reinterpret_cast<u32x2*>(d) = u32x2{v[it][0], v[it][1]};
                    if (cols & 2) *reinterpret_cast<uint32_t*>(d + (cols & 4)) = cols & 4 ? v[it][2] : v[it][0];
                    if (cols & 1) d[cols & 6] = (uint16_t)(cols & 4 ? cols & 2 ? v[it][3] : v[it][2] : cols & 2 ? v[it][1] : v[it][0]);
                }
            }
            sdst += NIT * sstep;
        };
        // Unquantised merge (M = out, N = in): the old bf16 weight, 16 bytes per lane (n < N stays inside the row's pitch, a
        // multiple of 8 elements), two rows of tiles ahead of their turn.  (Fetched four columns at a time where they are
        // added, a launch on 6374 x 2304, rank 160, took 41 us; this way 24.5.)
        constexpr bool OLD = EPI == EPI_ACC_BF16;
        uint4 old[OLD ? 2 : 1][2][OLD ? TN / 2 : 1];
        auto fetch_old = [&](int i) {
            const int64_t row = min(m0 + wm * WTM + i * 16 + frow, p.M - 1);
#pragma unroll
            for (int c = 0; c < TN / 2; ++c) {
                const int n = n0 + wn * WTN + 32 * c + 8 * g4;
                old[(i >> 1) & 1][i & 1][c] = *reinterpret_cast<const uint4*>(p.w_bf16 + row * p.w_bf16_ld + (n < N ? n : n0));
            }
        };
        if constexpr (OLD) fetch_old(0), fetch_old(1);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if constexpr (OLD)
                if (i % 2 == 0 && i + 2 < TM) fetch_old(i + 2), fetch_old(i + 3);
            const int m = m0 + wm * WTM + i * 16 + frow;
            uint32_t cw[EPI == EPI_FOLD ? TN / 2 : 1];
            if constexpr (EPI == EPI_FOLD) {
#pragma unroll
                for (int c = 0; c < TN / 2; ++c) cw[c] = *reinterpret_cast<const uint32_t*>(code_at(i, wn * (WTN / 32) + c));
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                float v0 = alpha * acc[i][j][0], v1 = alpha * acc[i][j][1], v2 = alpha * acc[i][j][2], v3 = alpha * acc[i][j][3];
                if constexpr (OLD) {
                    const uint4 o = old[(i >> 1) & 1][i & 1][j >> 1];
                    const bool hi = (j ^ g4) & 1;
                    const uint32_t o0 = hi ? o.z : o.x, o1 = hi ? o.w : o.y;
                    v0 += bf16_lo(o0), v1 += bf16_hi(o0), v2 += bf16_lo(o1), v3 += bf16_hi(o1);
                }
                if constexpr (EPI == EPI_FOLD) {  // folded weight (M = out, N = in)
                    const float am = am_old[i][j >> 2];
                    float q[4];
                    levels4(cw[j >> 1], j & 1 ? sh1 : sh0, q);
                    v0 += am * q[0], v1 += am * q[1], v2 += am * q[2], v3 += am * q[3];
                }
                const uint2 v = make_uint2(pack_bf16(v0, v1), pack_bf16(v2, v3));
                *reinterpret_cast<uint2*>(ebuf + ((i & 1) * 16 + frow) * EPITCH + (col_of(j) - wn * WTN) * 2) = v;
            }
            if (i & 1) store_rows((i - 1) * 16);
        }
    } else if constexpr (EPI == EPI_F32_SPLITK || EPI == EPI_FOLD_F32) {
        // fp32 results, 16 bytes per lane (row m, 4 consecutive n).  EPI_F32_SPLITK: slice `split` of the
        // contraction.  EPI_FOLD_F32 (M = out, N = in): the dense merged weight of Alg. 1 line 5,
        // fma(alpha, acc, fl32(absmax * q[code])), the same expression the merge epilogue quantises.
        // A tile inside the matrix tests no bounds and walks a pointer (a slice on 256x128: the epilogue 12700 cycles before, 8600 now).
        float* C = reinterpret_cast<float*>(p.C);
        if (EPI == EPI_F32_SPLITK) C += (int64_t)split * p.M * p.ldc;
        if (EPI == EPI_F32_SPLITK && m0 + BM <= p.M && n0 + BN <= p.N) {
            float* dst = C + (int64_t)(m0 + wm * WTM + frow) * p.ldc + (n0 + col_of(0));
            const int64_t step = 16 * p.ldc;
#pragma unroll
            for (int i = 0; i < TM; ++i, dst += step)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = p.alpha * acc[i][j][e];
                    *reinterpret_cast<float4*>(dst + 16 * j) = make_float4(v[0], v[1], v[2], v[3]);
                }
            return;
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = m0 + wm * WTM + i * 16 + frow;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int n = n0 + col_of(j);
                float v[4];
                if constexpr (EPI == EPI_FOLD_F32) {
                    float lev[4];
                    const uint32_t cw = *reinterpret_cast<const uint32_t*>(code_at(i, wn * (WTN / 32) + (j >> 1)));
                    levels4(cw, j & 1 ? sh1 : sh0, lev);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = __builtin_fmaf(p.alpha, acc[i][j][e], am_old[i][j >> 2] * lev[e]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = p.alpha * acc[i][j][e];
                }
                if (m < p.M) {
                    float* dst = C + (int64_t)m * p.ldc + n;
                    if (n + 4 <= p.N) {
                        *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                    } else {
                        for (int e = 0; e < 4; ++e)
                            if (n + e < p.N) dst[e] = v[e];
                    }
                }
            }
        }
    } else {
        // merge (M = out, N = in): W_new = fl32(absmax * q[code]) + alpha * acc, requantised per
        // 64-block along n (Alg. 1 line 5).  A block of row m is 16 values in each of four lanes.
        // compensation step (Alg. 2 lines 8-10): the same with W_hat = w_f32 + alpha * acc; the residual
        // w_f32 - deq(q(W_hat)) leaves as bf16.
        // The new codes take the place of the old ones in LDS, dword by dword, and leave from there 16 bytes per lane.
        // One wave per SIMD has nobody to hide a latency behind, so all blocks of 16 rows go through every stage together and
        // what the next 16 rows need is read ahead.
        const Nf4EncTables* const enc = &enc_tables;
        const int64_t ldb = p.w_ld >> 1, lda = p.w_ld >> 6;
        constexpr int CPW = WTN / 32, RPS = 64 / CPW;  // chunks of codes per row of the wave; rows per store
        // Old levels of the running 16 rows and of the next; compensation: the weights, from memory, of all rows at once.
        constexpr int AHEAD = EPI == EPI_COMP ? TM : 2;
        float src[AHEAD][NB][16];
        auto fetch = [&](int i) {
            const int m = m0 + wm * WTM + i * 16 + frow;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                float* const q = src[i % AHEAD][b];
                if constexpr (EPI == EPI_COMP) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const int n = n0 + col_of(4 * b + t);
                        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                        if (m < p.M && n < p.w_f32_ld) v = *reinterpret_cast<const float4*>(p.w_f32 + (int64_t)m * p.w_f32_ld + n);
                        q[4 * t] = v.x, q[4 * t + 1] = v.y, q[4 * t + 2] = v.z, q[4 * t + 3] = v.w;
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const uint32_t cw = *reinterpret_cast<const uint32_t*>(code_at(i, wn * CPW + 2 * b + u));
                        levels4(cw, sh0, q + 8 * u);
                        levels4(cw, sh1, q + 8 * u + 4);
                    }
                }
            }
        };
        // columns of the wave from nlast on do not exist
        const int nlast = p.w_cols - (n0 + (wave_s % Cfg::WAVES_N) * WTN);
#pragma unroll
        for (int i = 0; i < AHEAD - 1; ++i) fetch(i);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = m0 + wm * WTM + i * 16 + frow;
            if (i + AHEAD - 1 < TM) fetch(i + AHEAD - 1);
            float v[NB][16];
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float a = acc[i][4 * b + e / 4][e % 4], o = src[i % AHEAD][b][e];
                    v[b][e] = __builtin_fmaf(p.alpha, a, EPI == EPI_COMP ? o : am_old[CODES ? i : 0][b] * o);
                }
            // columns past the end count as 0.  (The condition in scalar registers and the empty
            // assembly keep it a branch: turned into selects it costs as much as the whole encoder.)
            if (nlast < WTN) {
                asm volatile("");
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (col_of(4 * b + e / 4) - wn * WTN + e % 4 >= nlast) {
                            v[b][e] = 0.f;
                            if constexpr (EPI == EPI_COMP) src[i % AHEAD][b][e] = 0.f;
                        }
            }
            Nf4BlockEncoder be[NB];
            float amax[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                amax[b] = 0.f;
#pragma unroll
                for (int e = 0; e < 16; ++e) amax[b] = fmaxf(amax[b], fabsf(v[b][e]));
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) amax[b] = max_over_lane_groups(amax[b]), be[b].set(amax[b]);
            // single-precision encoder first; the exact one again for all of them when any lane of the
            // wave has an element within rounding of a decision point (about one block in 10^4)
            uint32_t word[NB][2];
            bool near = false;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                uint32_t code[16];
                float nearest = __builtin_inff();
#pragma unroll
                for (int e = 0; e < 16; ++e) code[e] = be[b].encode_fast(enc, v[b][e], nearest);
                near |= be[b].near(nearest);
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    word[b][u] = nf4_pack4(code[8 * u], code[8 * u + 1], code[8 * u + 2], code[8 * u + 3]) << sh0 |
                                 nf4_pack4(code[8 * u + 4], code[8 * u + 5], code[8 * u + 6], code[8 * u + 7]) << sh1;
            }
            if (__any(near)) {  // (rolled up, the values through LDS: unrolled, the rare path is half of the kernel's instructions)
                float* const sc = reinterpret_cast<float*>(ebase) + wave * (16 * NB * 64) + lane;
#pragma unroll
                for (int e = 0; e < 16 * NB; ++e) sc[e * 64] = v[e / 16][e % 16];
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        uint32_t w = 0;
#pragma unroll 1
                        for (int k = 0; k < 8; ++k)
                            w |= be[b].encode(enc, sc[(16 * b + 8 * u + k) * 64]) << (((k >> 1) & 1) * 8 + 4 - 4 * (k & 1) + (k & 4 ? sh1 : sh0));
                        word[b][u] = w;
                    }
            }
            float am_new = 0.f;  // of block g4
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                am_new = b == 0 || b == g4 ? amax[b] : am_new;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    *reinterpret_cast<uint32_t*>(code_at(i, wn * CPW + 2 * b + u)) = word[b][u];
                    if constexpr (EPI == EPI_COMP) {  // the residuals of the eight columns, 16 bytes
                        uint2 half[2];
#pragma unroll
                        for (int t = 0; t < 2; ++t) {
                            float lev[4], e[4];
                            levels4(word[b][u], t ? sh1 : sh0, lev);
#pragma unroll
                            for (int k = 0; k < 4; ++k) e[k] = src[i % AHEAD][b][8 * u + 4 * t + k] - amax[b] * lev[k];
                            half[t] = make_uint2(pack_bf16(e[0], e[1]), pack_bf16(e[2], e[3]));
                        }
                        const uint2 lo = sh0 ? half[1] : half[0], hi = sh0 ? half[0] : half[1];
                        const int n = n0 + wn * WTN + 64 * b + 32 * u + 8 * g4;
                        if (m < p.M && n < p.e_ld)
                            *reinterpret_cast<uint4*>(p.e_out + (int64_t)m * p.e_ld + n) = make_uint4(lo.x, lo.y, hi.x, hi.y);
                    }
                }
            }
            if (m < p.M && g4 < NB && n0 + wn * WTN + g4 * 64 < p.w_ld) p.out_absmax[m * lda + ((n0 + wn * WTN) >> 6) + g4] = am_new;
            if ((i + 1) * 16 % RPS == 0) {  // rows that are complete: (i + 1) 16 - RPS on
                asm volatile("" ::: "memory");
                const int row = wm * WTM + (i + 1) * 16 - RPS + lane / CPW, c = wn * CPW + lane % CPW;
                const uint4 o = *reinterpret_cast<const uint4*>(cbuf + row * (BN / 2) + ((c ^ code_swz(row)) << 4));
                if (m0 + row < p.M && n0 + c * 32 < p.w_ld)
                    *reinterpret_cast<uint4*>(p.out_codes + (m0 + row) * ldb + (n0 >> 1) + c * 16) = o;
            }
        }
    }
}

// Work-groups are dealt to the 8 XCDs round-robin by the hardware; each XCD walks a contiguous range of tiles.
template <int BM, int BN, int EPI, bool ARC, bool BRC, int NS = 2, bool NOTAIL = false, bool ANF4 = false, bool LOADERS = false, int NW = 4>
__global__ __launch_bounds__(LOADERS ? 512 : 64 * NW, (LOADERS ? 2 : NW / 4) * (NtCfg<BM, BN, NS, ANF4, NW>::PER_CU)) void nt_gemm_kernel(const GemmParams p) {
    const int per_xcd = gridDim.x >> 3;
    nt_gemm_tile<BM, BN, EPI, ARC, BRC, NS, NOTAIL, ANF4, LOADERS, NW>(p, (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3), blockIdx.y);
}

// 128x128 tiles: with waves of their own for the loads a compute unit holds one work-group, without two.  One is enough, and faster, while
// no XCD (an eighth of the tiles of every slice, rounded up) has more than its 32 units: 4096 x 768 x 2048 21.4 -> 17.5 us, 2048 x 2048 x
// 4096 36.8 -> 31.3.  From there on two hide each other's first loads and results (512 tiles of 4096 x 2048 x 5461: 103.7 either way).
template <int EPI>
bool one_to_a_unit(const GemmParams& p) {
    const int64_t tiles = (int64_t)((p.M + 127) / 128) * ((p.N + 127) / 128 + (p.Nx + 127) / 128);
    return (tiles + 7) / 8 * (EPI == EPI_F32_SPLITK ? p.splits : 1) <= 32;
}

// the kernel's LDS size has to be raised above the default once per process (first launch, or loqt_prepare)
template <int BM, int BN, int EPI, bool ARC, bool BRC, int NS = 2, bool NOTAIL = false, bool ANF4 = false, bool LOADERS = false, int NW = 4>
hipError_t ensure_attr() {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(nt_gemm_kernel<BM, BN, EPI, ARC, BRC, NS, NOTAIL, ANF4, LOADERS, NW>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, NtCfg<BM, BN, NS, ANF4, NW>::SMEM);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    return hipSuccess;
}

template <int BM, int BN, int EPI, bool ARC, bool BRC, int NS = 2, bool NOTAIL = false, bool ANF4 = false, bool LOADERS = false, int NW = 4>
hipError_t launch_nt(const GemmParams& p, hipStream_t st) {
    if constexpr (BM == 256 && (EPI == EPI_BF16 || (EPI == EPI_F32_SPLITK && BN == 128) || NW == 8) && !NOTAIL) {
        // 256-row tiles have a variant for contractions that are whole k-tiles
        if (p.A[0].K % BK == 0 && p.A[1].K % BK == 0) return launch_nt<BM, BN, EPI, ARC, BRC, NS, true, ANF4, LOADERS, NW>(p, st);
    }
    hipError_t e0 = ensure_attr<BM, BN, EPI, ARC, BRC, NS, NOTAIL, ANF4, LOADERS, NW>();
    if (e0 != hipSuccess) return e0;
    const int tiles = ((p.M + BM - 1) / BM) * ((p.N + BN - 1) / BN + (p.Nx + BN - 1) / BN);
    dim3 grid((tiles + 7) / 8 * 8, EPI == EPI_F32_SPLITK ? p.splits : 1);
    hipLaunchKernelGGL((nt_gemm_kernel<BM, BN, EPI, ARC, BRC, NS, NOTAIL, ANF4, LOADERS, NW>), grid, dim3(LOADERS ? 512 : 64 * NW), (NtCfg<BM, BN, NS, ANF4, NW>::SMEM), st, p);
    return hipGetLastError();
}

}  // namespace
}  // namespace loqt
