// Products of a few hundred tokens with a 4-bit weight:  C[T x N] = alpha * sum_seg A_seg[T x K_seg] * deq(B_seg)[K_seg x N]
// in fp32 slices of the contraction, the codes expanded on the way from LDS to LDS.
//
// With T <= 256 an expansion of the weight to bf16 costs as much as the product (13824 x 5120: 37 us, 40 MB read and 141 MB
// written, and the product reads the 141 MB back).  Here the codes and block scales of a k-tile come into LDS by direct
// loads (5 KB instead of 16 KB for 64 x 128 weights), each thread expands its 16 (level table in LDS, one fp32 multiply,
// round to nearest even bf16: the bits of nf4_dequantize) and stores them where the plain kernels' direct loads would have
// put them; with up to 256 tokens in a tile every weight is expanded once per call.
//
// Work-group: four waves that multiply (2 x 2 of them over the tile BM x 128 x 64, v_mfma_f32_16x16x32_bf16, the loop of nt_tile.h
// with waves of their own for the loads) and four, or with up to 128 tokens eight, that feed them; three stages of operands.  The one
// barrier of k-tile kt falls between its two k32 steps and says that its fragments are in registers and that tile kt+1 is in
// place.  After it the feeding waves write tile kt+2 out, whose levels they have looked up in the iteration before, look up those of
// tile kt+3, ask for its A (direct loads into the stage of tile kt) between the look-ups and for the codes of tile kt+6, and take the
// codes of tile kt+4 out of their ring of three slots.  A wave takes the codes it has asked for itself, so only its own loads have
// to have landed.  The codes come from HBM and have two k-tiles for that, A has two.
// dx = dy deq(W) + Z B has a bf16 operand stored K x rows beside the 4-bit one: the work-groups of one more slice take that
// product, with direct loads of B in place of the codes, instead of a launch of their own (16 us at 256 x 5120 x 1024).
// What bounds it is the feeding: a k-tile takes 2000 cycles with 256 tokens and 1200 with 64 on a chip that is otherwise empty, 1440 and
// 700 with the expansion left out, 1850 and 1100 without look-ups, 1750 and 1130 without A, 1900 and 1220 without the matrix
// instructions (1024 and 256).  With every wave doing both, two to a SIMD, it was 2400 and 1800: there the instructions of the
// expansion stood between the matrix instructions.  Products with the sums of their slices left out, us, before and now: y of 13824 x 5120
// + 1024, 256 tokens 65 / 55, dx of it 52 / 47; 128 tokens 54 / 44; 64 tokens 45 / 35; 4096 x 5120, 256 tokens 23.9 / 22.0, 64 tokens
// 14.2 / 12.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "loqt_internal.h"

namespace loqt {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

constexpr int BN = 128, BK = 64, ROWB = 128;
constexpr int QBYTES = 256 * 16 + 256 * 4;  // codes and scales of one k-tile: 16 and 4 bytes for each of 256 lanes
constexpr int NS = 3, NQ = 3;               // stages of operands, slots of the ring of codes

#define LOQT_LDS_ADDR(p) ((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)(p))

template <int BM>
struct Cfg {
    static constexpr int WTM = BM / 2, WTN = BN / 2;    // wave tile
    static constexpr int TM = WTM / 16, TN = WTN / 16;  // 16x16 tiles per wave
    static constexpr int FEED = BM == 256 ? 256 : 512;  // threads that feed (the accumulators of 256 rows leave registers for four waves)
    static constexpr int THREADS = 256 + FEED;
    static constexpr int NA = BM * ROWB / (FEED * 16);  // direct loads of A per thread and k-tile
    static constexpr int CODES = 8192 / FEED;           // codes per thread and k-tile
    static constexpr int STAGE = (BM + BN) * ROWB;
    static constexpr int SMEM = NS * STAGE + NQ * QBYTES;
};

// waits until no more than `c` of this wave's loads are on their way, or fewer: C0, the count of the steady state, first
template <int C0, int NA>
__device__ __forceinline__ void wait_loads(int c) {
    if (c >= C0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(C0) : "memory");
    else if (c >= NA + 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NA + 2) : "memory");
    else if (c >= NA) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NA) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// slices of the contraction, and the one of the second segment
template <bool BRC>
__host__ __device__ __forceinline__ int slices_of(const GemmParams& p) {
    return p.splits + (BRC && p.A[1].K > 0 ? 1 : 0);
}
// an eighth of the tiles with all their slices on the 32 compute units of an XCD
__host__ __device__ __forceinline__ bool one_round(int tiles, int slices) { return ((tiles + 7) >> 3) * slices <= 32; }

// BRC: the weight is stored K x rows (its blocks run along the output columns), else rows x K
template <int BM, bool BRC>
__global__ __launch_bounds__(Cfg<BM>::THREADS, Cfg<BM>::THREADS / 256) void nf4_tile_kernel(const GemmParams p) {
    using C = Cfg<BM>;
    constexpr int TM = C::TM, TN = C::TN, STAGE = C::STAGE, NA = C::NA, FEED = C::FEED, CODES = C::CODES, PASS = FEED * 16;
    extern __shared__ __attribute__((aligned(256))) char smem[];
    __shared__ __attribute__((aligned(256))) float lut[64];  // (static: its reads then need no base register)
    char* const qring = smem + NS * STAGE;
    const bool feeds = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) != 0;
    const int tid = feeds ? threadIdx.x - 256 : threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
    // An XCD takes a contiguous range of tiles, row tiles of one column next to each other (they share its codes), with all their slices
    // where that is one round, else of the tiles of all slices: an eighth of the tiles, rounded up, leaves XCDs idle while others
    // take two rounds (forward, 192 tokens, 10335 x 2548 in three slices 64.3 -> 44.2 us, 96 tokens, 1131 x 5689 34.7 -> 27.1), but where one round holds them the spread has nothing to give, and backward calls of a few
    // tokens were 1 to 2 us slower with their slices spread (7872 x 636, one token, 26.2 -> 28.1).
    const int tiles = tiles_m * tiles_n, slices = slices_of<BRC>(p), per_x = (tiles + 7) >> 3, x = blockIdx.x & 7, j = blockIdx.x >> 3;
    const bool fits = one_round(tiles, slices);
    const int all = fits ? j : x * (gridDim.x >> 3) + j, of = fits ? per_x : tiles;
    const int slice = all / of, L = all - slice * of + (fits ? x * per_x : 0);
    if (L >= tiles || slice >= slices) return;
    const int m0 = (L % tiles_m) * BM, n0 = (L / tiles_m) * BN;

    // K x rows: the second segment is the bf16 one, a slice of its own after the others
    const bool extra = BRC && slice == p.splits;
    const int nkt0 = (p.A[0].K + BK - 1) / BK, nkt1 = (p.A[1].K + BK - 1) / BK;
    const int per = ((BRC ? nkt0 : nkt0 + nkt1) + p.splits - 1) / p.splits;
    const int kt_begin = extra ? nkt0 : slice * per;
    const int kt_end = extra ? nkt0 + nkt1 : min(BRC ? nkt0 : nkt0 + nkt1, kt_begin + per);
    const int n = kt_end - kt_begin;  // k-tiles of this work-group
    const int tail0 = (p.A[0].K % BK) ? nkt0 - 1 : -1, tail1 = (p.A[1].K % BK) ? nkt0 + nkt1 - 1 : -1;

    // chunk swizzles of nt_tile.h
    auto kc_swz = [](int row) {
        const int e = (row >> 1) & 7;
        return (e & 1) | ((e & 2) << 1) | ((e & 4) >> 1);
    };
    auto rc_swz = [](int kk) { return (4 * (kk & 3)) ^ (2 * ((kk >> 3) & 1)); };

    if (feeds) {
        // ---- direct loads.  A: chunk i of a thread is row i*FEED/8 + tid/8, physical chunk tid%8 of the [row][64 k] tile.
        // Codes: lane ql of 256 (all, or the first 32 of every wave) fetches 32 of them, half ql%2 of row ql/2 of the 128 rows, or, K x rows,
        // columns 32*(ql%4) on of k row ql/4.
        const int ql = FEED == 256 ? tid : wave * 32 + (lane & 31);
        uint32_t offA[NA], offQ = 0, offS = 0;
        const char *baseA = nullptr, *baseQ = nullptr, *baseS = nullptr;
        int64_t stepQ = 0, stepS = 0;
        auto setup_a = [&](int kt) {
            const bool seg = kt >= nkt0;
            const int k0 = (kt - (seg ? nkt0 : 0)) * BK, kleft = (seg ? p.A[1].K : p.A[0].K) - k0;
            const int64_t ld = seg ? p.A[1].ld : p.A[0].ld;
            const int r0 = tid >> 3, kc = (tid & 7) ^ kc_swz(r0), rlast = p.M - 1 - m0;
            const uint32_t kb = kc * 8 < kleft ? (uint32_t)kc * 16u : 0u;  // past the end: a valid chunk, cleared later
#pragma unroll
            for (int i = 0; i < NA; ++i) offA[i] = (uint32_t)min(i * (FEED / 8) + r0, rlast) * (uint32_t)(ld * 2) + kb;
            baseA = reinterpret_cast<const char*>(seg ? p.A[1].ptr : p.A[0].ptr) + ((int64_t)m0 * ld + k0) * 2;
        };
        auto setup_q = [&](int kt) {
            const bool seg = kt >= nkt0;
            const int k0 = (kt - (seg ? nkt0 : 0)) * BK, kleft = (seg ? p.B[1].K : p.B[0].K) - k0;
            const int64_t ldb = (seg ? p.B[1].ld : p.B[0].ld) >> 1, lds = (seg ? p.B[1].ld : p.B[0].ld) >> 6;
            const char* codes = reinterpret_cast<const char*>(seg ? p.B[1].ptr : p.B[0].ptr);
            const char* scales = reinterpret_cast<const char*>(seg ? p.B[1].absmax : p.B[0].absmax);
            if constexpr (!BRC) {
                const int row = min(ql >> 1, p.N - 1 - n0);
                offQ = (uint32_t)row * (uint32_t)ldb + (uint32_t)(ql & 1) * 16u;
                offS = (uint32_t)row * (uint32_t)(lds * 4);
                baseQ = codes + (int64_t)n0 * ldb + (k0 >> 1);
                baseS = scales + ((int64_t)n0 * lds + (k0 >> 6)) * 4;
                stepQ = BK / 2, stepS = 4;
            } else {
                const int k = min(ql >> 2, kleft - 1);  // k rows past the end meet zeros of A
                const int c = n0 + 32 * (ql & 3) < 2 * ldb ? ql & 3 : 0;
                offQ = (uint32_t)k * (uint32_t)ldb + (uint32_t)c * 16u;
                offS = (uint32_t)k * (uint32_t)(lds * 4) + (uint32_t)(c >> 1) * 4u;
                baseQ = codes + (int64_t)k0 * ldb + (n0 >> 1);
                baseS = scales + ((int64_t)k0 * lds + (n0 >> 6)) * 4;
                stepQ = BK * ldb, stepS = BK * lds * 4;
            }
        };
        // B in bf16 (extra): chunk i of a thread is k row i*FEED/16 + tid/16, physical chunk tid%16 of the [64 k][128] tile
        constexpr int NBL = 64 * BN * 2 / PASS;
        uint32_t offB[NBL];
        const char* baseB = nullptr;
        auto setup_b = [&](int kt) {
            const int k0 = (kt - nkt0) * BK, kleft = p.B[1].K - k0;
            const int clast = (((p.N - 1) >> 3) << 3) - n0;  // columns past the end: any valid chunk
#pragma unroll
            for (int i = 0; i < NBL; ++i) {
                const int k = i * (FEED / 16) + (tid >> 4), logical = (tid & 15) ^ rc_swz(k);
                offB[i] = (uint32_t)min(k, kleft - 1) * (uint32_t)(p.B[1].ld * 2) + (uint32_t)min(logical * 8, clast) * 2u;
            }
            baseB = reinterpret_cast<const char*>(p.B[1].ptr) + ((int64_t)k0 * p.B[1].ld + n0) * 2;
        };
        auto is_tail = [&](int t) { return t == tail0 || t == tail1; };
        const uint32_t lds0 = LOQT_LDS_ADDR(smem), lwave = (uint32_t)wave * 1024u;
        // Inline assembly (M0: the LDS address, and one wait state between its write and the load) for the reasons given in nt_tile.h:
        // the compiler would wait for all of the loads in front of LDS reads.
        auto direct_load = [&](uint32_t o, const char* base, uint32_t dst, uint32_t at) {
            asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(o), "s"(base), "s"(dst), "i"(at) : "memory", "scc");
        };
        // t: k-tile of this work-group's range, asked for in order, from 0 on; past the end nothing is
        // A in four parts, which go between the look-ups of the codes: a load holds the wave up while the memory pipeline is busy
        auto next_a = [&](int t) {
            if (t >= n) return;
            const int kt = kt_begin + t;
            if (t == 0 || kt == nkt0 || is_tail(kt)) setup_a(kt);
            else baseA += BK * 2;
        };
        auto part_a = [&](int t, int part) {
            if (t >= n) return;
            const uint32_t adst = lds0 + (uint32_t)(t % NS * STAGE) + lwave;
#pragma unroll
            for (int i = part * NA / 4; i < (part + 1) * NA / 4; ++i) direct_load(offA[i], baseA, adst, (uint32_t)(i * PASS));
        };
        auto ask_a = [&](int t) {
            next_a(t);
#pragma unroll
            for (int part = 0; part < 4; ++part) part_a(t, part);
        };
        auto load_q = [&](uint32_t slot) {
            if constexpr (FEED == 256) {
                direct_load(offQ, baseQ, slot + lwave, 0);
                asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(offS), "s"(baseS), "s"(slot + (uint32_t)wave * 256u),
                             "i"(4096) : "memory", "scc");
            } else {  // by half of the lanes (EXEC is all ones before and after: uniform control flow)
                asm volatile(
                    "s_mov_b32 m0, %2\n\t"
                    "s_mov_b32 exec_hi, 0\n\t"
                    "global_load_lds_dwordx4 %0, %1\n\t"
                    "s_mov_b32 m0, %5\n\t"
                    "s_nop 0\n\t"
                    "global_load_lds_dword %3, %4\n\t"
                    "s_mov_b32 exec_hi, -1"
                    ::"v"(offQ), "s"(baseQ), "s"(slot + (uint32_t)wave * 512u), "v"(offS), "s"(baseS), "s"(slot + 4096u + (uint32_t)wave * 128u) : "memory");
            }
        };
        auto ask_q = [&](int t) {
            if (t >= n) return;
            const int kt = kt_begin + t;
            if (t == 0 || kt == nkt0 || (BRC && is_tail(kt))) setup_q(kt);
            else baseQ += stepQ, baseS += stepS;
            load_q(LOQT_LDS_ADDR(qring) + (uint32_t)(t % NQ * QBYTES));
        };
        auto ask_b = [&](int t) {
            if (t >= n) return;
            const int kt = kt_begin + t;
            if (t == 0 || is_tail(kt)) setup_b(kt);
            else baseB += (int64_t)BK * p.B[1].ld * 2;
            const uint32_t dst = lds0 + (uint32_t)(t % NS * STAGE) + lwave;
#pragma unroll
            for (int i = 0; i < NBL; ++i) direct_load(offB[i], baseB, dst, (uint32_t)(BM * ROWB + i * PASS));
        };
        // tile t has landed: clears A past the end of the contraction (codes past it are finite weights, or k rows repeated).  A thread
        // clears the chunks it has loaded itself, and waits for that: the next barrier may be one that lets LDS operations pass.
        auto cut = [&](int t) {
            const int kt = kt_begin + t;
            if (t >= n || !is_tail(kt)) return;
            const bool seg = kt >= nkt0;
            const int kleft = (seg ? p.A[1].K : p.A[0].K) - (kt - (seg ? nkt0 : 0)) * BK;
            const int nv = kleft - 8 * ((tid & 7) ^ kc_swz(tid >> 3));
            if (nv < 8) {
                uint32_t keep[4];
#pragma unroll
                for (int d = 0; d < 4; ++d) keep[d] = 2 * d + 1 < nv ? 0xffffffffu : 2 * d < nv ? 0xffffu : 0u;
#pragma unroll 1
                for (int i = 0; i < NA; ++i) {
                    uint4* q = reinterpret_cast<uint4*>(smem + t % NS * STAGE + i * PASS + tid * 16);
                    const uint4 v = *q;
                    *q = make_uint4(v.x & keep[0], v.y & keep[1], v.z & keep[2], v.w & keep[3]);
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        };
        // ---- expansion of the thread's codes: byte offsets into the table of levels, look-ups, products with the scale, two to a dword,
        // four dwords to a chunk of 16 bytes.  All look-ups of a k-tile are under way before the first product.
        int wbase, wsw;  // where the thread's chunks go: row (or k row) of the tile, its swizzle
        constexpr int PER_ROW = (BRC ? BN : BK) / CODES, NCK = CODES / 8;  // threads to a row, chunks per thread
        wbase = BM * ROWB + (tid / PER_ROW) * (BRC ? BN * 2 : ROWB);
        wsw = BRC ? rc_swz(tid / PER_ROW) : kc_swz(tid / PER_ROW);
        uint32_t cw[NCK];
        float am = 0.f, scale = 0.f, v[CODES];
        auto take = [&](const char* slot) {  // the codes of a tile, out of the ring
            if constexpr (NCK == 4) {
                const uint4 c = *reinterpret_cast<const uint4*>(slot + tid * 16);
                cw[0] = c.x, cw[1] = c.y, cw[2] = c.z, cw[3] = c.w;
            } else {
                const uint2 c = *reinterpret_cast<const uint2*>(slot + tid * 8);
                cw[0] = c.x, cw[1] = c.y;
            }
            am = *reinterpret_cast<const float*>(slot + 4096 + (FEED == 256 ? tid : tid >> 1) * 4);
        };
        auto look_up = [&](int c) {  // chunk c: a dword of codes, even elements in the high nibbles
            const uint32_t even = (cw[c] >> 2) & 0x3c3c3c3cu, odd = (cw[c] << 2) & 0x3c3c3c3cu;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                v[8 * c + e] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(lut) + (((e & 1 ? odd : even) >> (8 * (e / 2))) & 0xffu));
        };
        auto put = [&](char* stage) {
#pragma unroll
            for (int c = 0; c < NCK; ++c) {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[8 * c + e] *= scale;
                const int logical = (tid % PER_ROW) * NCK + c;
                const float* const w = v + 8 * c;
                *reinterpret_cast<uint4*>(stage + wbase + ((logical ^ wsw) << 4)) =
                    make_uint4(pack_bf16(w[0], w[1]), pack_bf16(w[2], w[3]), pack_bf16(w[4], w[5]), pack_bf16(w[6], w[7]));
            }
        };
        auto slot_of = [&](int t) { return qring + t % NQ * QBYTES; };
        if (tid < 16) lut[tid] = kNf4Levels[tid];
        __syncthreads();
        if (n > 0) {
            // what is on its way after tile t, of `each` loads to a tile, up to tile `last` (loads are asked for in order)
            auto some = [&](int t, int each) { return t < n ? each : 0; };
            if (!extra) {
                for (int t = 0; t < NQ; ++t) ask_q(t);
                for (int t = 0; t < NS; ++t) ask_a(t);
                wait_loads<3 * NA, NA>(some(0, NA) + some(1, NA) + some(2, NA));  // the codes
                // (past the end: whatever is in the ring, for nobody.  A slot is free when its codes have been used.)
                auto ahead = [&](int t) {
                    take(slot_of(t));
#pragma unroll
                    for (int c = 0; c < NCK; ++c) look_up(c);
                    scale = am;
                    ask_q(t + 3);
                };
                ahead(0);
                put(smem);
                wait_loads<2 * NA + 2, NA>(some(1, NA) + some(2, NA) + some(3, 2));
                cut(0);
                __syncthreads();  // tile 0 is in place
                ahead(1);
                put(smem + STAGE);
                ahead(2);
                wait_loads<4, NA>(some(4, 2) + some(5, 2));  // A of tiles 1 and 2, the codes of tile 3
                take(slot_of(3));
                cut(1);
                // Iteration k: write out tile k + 2, whose levels are in registers; look up those of tile k + 3, whose codes are; ask for A
                // of tile k + 3 and the codes of tile k + 6 (into the slot of tile k + 3); take the codes of tile k + 4, which are on
                // their way ahead of A of tile k + 2 (behind it at first); wait for A of tile k + 2.  So no look-up is waited for
                // in the iteration that makes it.
                // Where no tile in question is the first of its segment or cut, three at a time, with the stages as constants and no
                // branch: the other form spends half of its 300 instructions on the scalar unit.  Past the end the last tile is asked for
                // once more, into stages and slots that nobody reads.  Behind the writes of a tile there are 16 LDS reads or
                // more, which need not have arrived at the barrier.
                auto fast = [&](auto phase_tag, auto first_tag, int k) {
                    constexpr int P = decltype(phase_tag)::value;
                    asm volatile("s_waitcnt lgkmcnt(15)\n\ts_barrier" ::: "memory");
                    put(smem + (P + 2) % 3 * STAGE);
                    if (k + 3 < n) baseA += BK * 2;
#pragma unroll
                    for (int part = 0; part < 4; ++part) {
                        if (part < NCK) look_up(part < NCK ? part : 0);
#pragma unroll
                        for (int i = part * NA / 4; i < (part + 1) * NA / 4; ++i) direct_load(offA[i], baseA, lds0 + lwave, (uint32_t)(P * STAGE + i * PASS));
                    }
                    scale = am;
                    if (k + 6 < n) baseQ += stepQ, baseS += stepS;
                    load_q(LOQT_LDS_ADDR(qring) + P * QBYTES);
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(first_tag)::value ? NA + 4 : 2 * NA + 4) : "memory");
                    take(qring + (P + 1) % 3 * QBYTES);
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NA + 4) : "memory");
                };
                const int s0 = nkt0 - kt_begin, s1 = tail0 - kt_begin, s2 = tail1 - kt_begin;
                auto plain = [&](int k) {  // k + 2 < n, no special tile among k + 2 .. k + 8
                    auto far = [&](int t) { return t < 0 || t >= n || (unsigned)(t - (k + 2)) > 6u; };
                    return k + 2 < n && far(s0) && far(s1) && far(s2);
                };
                using True = std::true_type;
                using False = std::false_type;
                for (int k = 0; k < n; ++k) {
                    if (k % 3 == 0) {
                        // The counts of the waits take it that every load up to now was made: k + 5 < n, or the three before were fast.
                        bool all = k + 5 < n;
                        if (k == 0 && all && plain(0)) {
                            fast(std::integral_constant<int, 0>{}, True{}, 0);
                            fast(std::integral_constant<int, 1>{}, False{}, 1);
                            fast(std::integral_constant<int, 2>{}, False{}, 2);
                            k = 3;
                        }
                        while (k > 0 && all && plain(k)) {
                            fast(std::integral_constant<int, 0>{}, False{}, k);
                            fast(std::integral_constant<int, 1>{}, False{}, k + 1);
                            fast(std::integral_constant<int, 2>{}, False{}, k + 2);
                            k += 3;
                        }
                        if (k >= n) break;
                    }
                    __syncthreads();  // tile k is in registers, tile k + 1 in place
                    if (k + 2 >= n) continue;
                    put(smem + (k + 2) % NS * STAGE);
                    next_a(k + 3);
#pragma unroll
                    for (int part = 0; part < 4; ++part) {
                        if (part < NCK) look_up(part < NCK ? part : 0);
                        part_a(k + 3, part);
                    }
                    scale = am;
                    ask_q(k + 6);
                    wait_loads<2 * NA + 4, NA>((k > 0 ? some(k + 2, NA) : 0) + some(k + 5, 2) + some(k + 3, NA) + some(k + 6, 2));
                    take(slot_of(k + 4));
                    wait_loads<NA + 4, NA>(some(k + 5, 2) + some(k + 3, NA) + some(k + 6, 2));
                    cut(k + 2);
                }
            } else {
                for (int t = 0; t < NS; ++t) ask_a(t), ask_b(t);
                constexpr int NL = NA + NBL;
                wait_loads<2 * NL, NL>(some(1, NL) + some(2, NL));
                cut(0);
                __syncthreads();
                wait_loads<NL, NL>(some(2, NL));
                cut(1);
                for (int k = 0; k < n; ++k) {
                    __syncthreads();
                    ask_a(k + 3), ask_b(k + 3);
                    wait_loads<NL, NL>(some(k + 3, NL));
                    cut(k + 2);
                }
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loads past the end
        return;
    }

    // ---- products
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int wm = wave >> 1, wn = wave & 1;
    // fragments (nt_tile.h)
    const int frow = lane & 15, q4 = lane >> 4;
    uint32_t a_ko[2], b_ko[2];
    int b_rc[BRC ? TN : 1];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int coff = ((4 * ks + q4) ^ kc_swz(frow)) << 4;
        a_ko[ks] = (uint32_t)((wm * C::WTM + frow) * ROWB + coff);
        b_ko[ks] = (uint32_t)(BM * ROWB + (wn * C::WTN + frow) * ROWB + coff);
    }
    if constexpr (BRC) {
        const int jj = (lane >> 2) & 3, q = lane & 3;
#pragma unroll
        for (int u = 0; u < TN; ++u) {
            const int chunk = ((wn * C::WTN + u * 16) >> 3) + (q >> 1);
            b_rc[u] = BM * ROWB + (8 * q4 + jj) * (BN * 2) + ((chunk ^ rc_swz(8 * q4 + jj)) << 4) + (q & 1) * 8;
        }
    }
    constexpr int NU = TM + TN, NM = TM * TN, RSL = NM * 5 / 8;
    bf16x8 f[2][NU];
    auto read_frag = [&](int ks, int u, const char* stage) {
        if (u < TM) {
            f[ks][u] = *reinterpret_cast<const bf16x8*>(stage + a_ko[ks] + u * 16 * ROWB);
        } else if constexpr (BRC) {
            const char* ptr = stage + b_rc[u - TM] + 32 * ks * (BN * 2);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(ptr));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(ptr + 4 * (BN * 2)));
            f[ks][u] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        } else {
            f[ks][u] = *reinterpret_cast<const bf16x8*>(stage + b_ko[ks] + (u - TM) * 16 * ROWB);
        }
    };
    auto nth = [](int i) { return i == 0 ? 0 : i <= TN ? TM + i - 1 : i - TN; };  // the order in which the products ask for them
    auto step = [&](auto cb_tag, const char* rstage) {  // the products of k32 step CB, under them the reads of the next step
        constexpr int CB = decltype(cb_tag)::value;
#pragma unroll
        for (int sl = 0; sl < NM; ++sl) {
            const int i = sl / TN, j = sl % TN;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[CB][TM + j], f[CB][i], acc[i][j], 0, 0, 0);
            if (sl < RSL) {
#pragma unroll
                for (int u = sl * NU / RSL; u < (sl + 1) * NU / RSL; ++u) read_frag(CB ^ 1, nth(u), rstage);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    __syncthreads();  // the table of levels
    if (n > 0) {
        __syncthreads();  // tile 0 is in place
#pragma unroll
        for (int u = 0; u < NU; ++u) read_frag(0, nth(u), smem);
    }
    int si = 0;
    for (int k = 0; k < n; ++k) {
        const char* const cur = smem + si * STAGE;
        si = si + 1 == NS ? 0 : si + 1;
        step(std::integral_constant<int, 0>{}, cur);
        __syncthreads();
        step(std::integral_constant<int, 1>{}, smem + si * STAGE);  // (past the last tile: harmless stale reads)
    }

    // lane: row 16 i + (lane & 15), columns 16 j + 4 (lane >> 4) .. +3
    float* out = reinterpret_cast<float*>(p.C) + (int64_t)slice * p.M * p.ldc;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + wm * C::WTM + i * 16 + frow;
        float* const row = out + (int64_t)m * p.ldc + n0 + wn * C::WTN + 4 * q4;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            // (the pitch is a multiple of 4: columns N .. ldc-1 of the slices are scratch)
            if (m < p.M && n0 + wn * C::WTN + j * 16 + 4 * q4 < p.ldc)
                *reinterpret_cast<float4*>(row + j * 16) = make_float4(p.alpha * acc[i][j][0], p.alpha * acc[i][j][1], p.alpha * acc[i][j][2], p.alpha * acc[i][j][3]);
        }
    }
}

template <int BM, bool BRC>
hipError_t ensure_attr() {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(nf4_tile_kernel<BM, BRC>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, Cfg<BM>::SMEM);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    return hipSuccess;
}
template <int BM, bool BRC>
hipError_t launch(const GemmParams& p, hipStream_t st) {
    hipError_t e = ensure_attr<BM, BRC>();
    if (e != hipSuccess) return e;
    const int tiles = ((p.M + BM - 1) / BM) * ((p.N + BN - 1) / BN);
    const int slices = slices_of<BRC>(p), per_xcd = one_round(tiles, slices) ? (tiles + 7) / 8 * slices : (tiles * slices + 7) / 8;
    hipLaunchKernelGGL((nf4_tile_kernel<BM, BRC>), dim3(per_xcd * 8), dim3(Cfg<BM>::THREADS), Cfg<BM>::SMEM, st, p);
    return hipGetLastError();
}

}  // namespace

hipError_t prepare_nf4_tile_kernels() {
    hipError_t e;
    if ((e = ensure_attr<256, false>()) != hipSuccess) return e;
    if ((e = ensure_attr<128, false>()) != hipSuccess) return e;
    if ((e = ensure_attr<64, false>()) != hipSuccess) return e;
    if ((e = ensure_attr<256, true>()) != hipSuccess) return e;
    if ((e = ensure_attr<128, true>()) != hipSuccess) return e;
    return ensure_attr<64, true>();
}

// Slices of the contraction: microseconds per k-tile with few work-groups and with one on every compute unit, plus the
// rest of a tile, as in plan_nt.  The slices it takes against the best of 1 to 32, over 4500 random products (1 to 256 tokens, 64 to 13824
// columns and as long a contraction): 1.011 on the mean, one in ninety more than 10 % off.  Tiles of 64 rows are priced above their own
// 0.45 to 0.58 us per k-tile: with those, dx (whose slice of Z B is short, but counts as another one) came in half as many slices
// (47 tokens, 6078 x 8448, rank 64, the backward call 46.8 -> 53.8 us; 7 tokens, 3650 x 8453, 35.9 -> 40.5), 1.0113 of the best with
// them, 1.0099 with these.
int nf4_tile_splits(int64_t M, int64_t N, int64_t nkt, int extra, int64_t max_splits) {
    const int64_t bm = M <= 64 ? 64 : M <= 128 ? 128 : 256;
    const double alone = bm == 128 ? 0.55 : 0.80, full = bm == 64 ? 0.95 : bm == 128 ? 0.75 : 1.0, rest = bm == 64 ? 6.0 : bm == 128 ? 7.0 : 10.0;
    const int64_t tiles = (M + bm - 1) / bm * ((N + BN - 1) / BN);
    int best = 1;
    double best_cost = 0.0;
    for (int64_t s = 1; s <= std::min<int64_t>(max_splits, NT_MAX_SPLITS); ++s) {
        const int64_t per = (nkt + s - 1) / s, wgs = tiles * (s + extra);
        if (s > 1 && (per < 4 || (nkt + per - 1) / per != s)) continue;
        auto one = [&](int64_t w) { return (double)per * (alone + (full - alone) * (double)w / 256.0) + rest; };
        const double cost = (double)(wgs / 256) * one(256) + (wgs % 256 ? one(wgs % 256) : 0.0) +
                            (double)(s + extra) * (double)M * (double)N * 4.0 * (1.0 / 6.0e6 + 1.0 / 7.0e6);
        if (s == 1 || cost < best_cost) best = (int)s, best_cost = cost;
    }
    return best;
}

hipError_t launch_nf4_tile(bool b_rc, const GemmParams& p, hipStream_t st) {
    if (p.M <= 64) return b_rc ? launch<64, true>(p, st) : launch<64, false>(p, st);
    if (p.M <= 128) return b_rc ? launch<128, true>(p, st) : launch<128, false>(p, st);
    return b_rc ? launch<256, true>(p, st) : launch<256, false>(p, st);
}

}  // namespace loqt
