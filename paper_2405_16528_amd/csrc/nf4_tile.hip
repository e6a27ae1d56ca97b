// Products of a few hundred tokens with a 4-bit weight:  C[T x N] = alpha * sum_seg A_seg[T x K_seg] * deq(B_seg)[K_seg x N]
// in fp32 slices of the contraction, the codes expanded on the way from LDS to LDS.
//
// With T <= 512 an expansion of the weight to bf16 costs as much as the product (13824 x 5120: 37 us, 40 MB read and 141 MB
// written, and the product reads the 141 MB back).  Here the codes and block scales of a k-tile come into LDS by direct
// loads (5 KB instead of 16 KB for 64 x 128 weights), each thread expands its 16 (level table in LDS, one fp32 multiply,
// round to nearest even bf16: the bits of nf4_dequantize) and stores them where the plain kernels' direct loads would have
// put them; with up to 256 tokens in a tile every weight is expanded once per call.
//
// Work-group: 8 waves, two per SIMD (4 x 2 of them over the tile, 2 x 4 with 64 rows), tile BM x 128 x 64,
// v_mfma_f32_16x16x32_bf16, two stages of operands and two barriers per k-tile as in nt_tile.h.  In the iteration of k-tile kt
//   first quarter          : fragment reads of its second k32 step
//   barrier X              : nobody reads stage kt any more
//   after it               : direct loads of A of tile kt+2 into that stage, then of the codes of tile kt+4
//   first three quarters   : codes of tile kt+1 expanded into the other stage
//   barrier Y              : tile kt+1 and the codes of tile kt+2 are in place
//   last quarter           : fragment reads of tile kt+1
// dx = dy deq(W) + Z B has a bf16 operand stored K x rows beside the 4-bit one: the work-groups of one more slice take that
// product, with direct loads of B in place of the codes, instead of a launch of their own (16 us at 256 x 5120 x 1024).
// A wave issues one instruction in four cycles and a matrix instruction keeps its unit for sixteen, so everything else
// goes between the matrix instructions in portions of about three, with a scheduling fence after each.  The codes come from
// HBM and have a ring of four slots: loads return in order, and those of an iteration are issued after its loads of A, so
// barrier Y can leave them in flight for one iteration more.
// What bounds it is the instructions around the matrix units: y of 13824 x 5120 + 1024 with 64 / 128 / 256 tokens takes 52 / 60 /
// 75 us with the sum of its slices, 34 / 42 / 60 without the expansion, 51 / 54 / 65 without the matrix instructions, 47 / 55 / 70
// without the loads of codes, 48 / 54 / 66 without those of A.  Two waves per SIMD cover for each other's look-ups and
// barriers: forward + backward, us, four waves / eight: 4096 x 4096, rank 1024, 256 tokens 126 / 104; 5120 x 5120 152 / 117;
// 13824 x 5120 201 / 190, 64 tokens 164 / 129.  Three stages, one barrier and fragments a step ahead were no faster (128 tokens,
// y 57 against 59) and leave no registers for 256 rows.
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
constexpr int THREADS = 512;
constexpr int QBYTES = 256 * 16 + 256 * 4;  // codes and scales of one k-tile: 16 and 4 bytes for each of 256 lanes
constexpr int NQ = 4;                       // slots of their ring

#define LOQT_LDS_ADDR(p) ((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)(p))

template <int BM>
struct Cfg {
    static constexpr int WM = BM == 64 ? 2 : 4, WN = 8 / WM;  // waves along the rows and columns of the tile
    static constexpr int WTM = BM / WM, WTN = BN / WN;        // wave tile
    static constexpr int TM = WTM / 16, TN = WTN / 16;        // 16x16 tiles per wave
    static constexpr int NA = BM / 64;                        // direct loads of A per thread and k-tile
    static constexpr int STAGE = (BM + BN) * ROWB;
    static constexpr int SMEM = 2 * STAGE + NQ * QBYTES;
};

template <int F, int... I, class Fn>
__device__ __forceinline__ void each(std::integer_sequence<int, I...>, Fn& f) {
    (f(std::integral_constant<int, F + I>{}), ...);
}

// BRC: the weight is stored K x rows (its blocks run along the output columns), else rows x K
template <int BM, bool BRC>
__global__ __launch_bounds__(THREADS, 2) void nf4_tile_kernel(const GemmParams p) {
    using C = Cfg<BM>;
    constexpr int TM = C::TM, TN = C::TN, STAGE = C::STAGE, U = 2 * TM * TN;  // slots: one matrix instruction each
    extern __shared__ __attribute__((aligned(256))) char smem[];
    __shared__ __attribute__((aligned(256))) float lut[64];  // (static: its reads then need no base register)
    char* const qring = smem + 2 * STAGE;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
    // contiguous ranges of tiles per XCD; row tiles of one column run next to each other and share its codes
    const int L = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (L >= tiles_m * tiles_n) return;
    const int m0 = (L % tiles_m) * BM, n0 = (L / tiles_m) * BN;

    // K x rows: the second segment is the bf16 one, a slice of its own after the others
    const bool extra = BRC && (int)blockIdx.y == p.splits;
    const int nkt0 = (p.A[0].K + BK - 1) / BK, nkt1 = (p.A[1].K + BK - 1) / BK;
    const int per = ((BRC ? nkt0 : nkt0 + nkt1) + p.splits - 1) / p.splits;
    const int kt_begin = extra ? nkt0 : blockIdx.y * per;
    const int kt_end = extra ? nkt0 + nkt1 : min(BRC ? nkt0 : nkt0 + nkt1, kt_begin + per);
    const int tail0 = (p.A[0].K % BK) ? nkt0 - 1 : -1, tail1 = (p.A[1].K % BK) ? nkt0 + nkt1 - 1 : -1;

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // chunk swizzles of nt_tile.h
    auto kc_swz = [](int row) {
        const int e = (row >> 1) & 7;
        return (e & 1) | ((e & 2) << 1) | ((e & 4) >> 1);
    };
    auto rc_swz = [](int kk) { return (4 * (kk & 3)) ^ (2 * ((kk >> 3) & 1)); };

    // ---- direct loads.  A: chunk i of a thread is row i*64 + tid/8, physical chunk tid%8 of the [row][64 k] tile.
    // Codes: the first 32 lanes of every wave, ql of 256, fetch 32 of row ql/2 (half ql%2) of the 128 rows, or, K x rows, of k row
    // ql/4, columns 32*(ql%4) on.
    const int ql = wave * 32 + (lane & 31);
    uint32_t offA[C::NA], offQ = 0, offS = 0;
    const char *baseA = nullptr, *baseQ = nullptr, *baseS = nullptr;
    int64_t stepQ = 0, stepS = 0;
    auto setup_a = [&](int kt) {
        const bool seg = kt >= nkt0;
        const int k0 = (kt - (seg ? nkt0 : 0)) * BK, kleft = (seg ? p.A[1].K : p.A[0].K) - k0;
        const int64_t ld = seg ? p.A[1].ld : p.A[0].ld;
        const int r0 = tid >> 3, kc = (tid & 7) ^ kc_swz(r0), rlast = p.M - 1 - m0;
        const uint32_t kb = kc * 8 < kleft ? (uint32_t)kc * 16u : 0u;  // past the end: a valid chunk, cleared later
#pragma unroll
        for (int i = 0; i < C::NA; ++i) offA[i] = (uint32_t)min(i * 64 + r0, rlast) * (uint32_t)(ld * 2) + kb;
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
    // B in bf16 (extra): chunk i of a thread is k row i*32 + tid/16, physical chunk tid%16 of the [64 k][128] tile
    constexpr int NBL = 2;
    uint32_t offB[NBL];
    const char* baseB = nullptr;
    auto setup_b = [&](int kt) {
        const int k0 = (kt - nkt0) * BK, kleft = p.B[1].K - k0;
        const int clast = (((p.N - 1) >> 3) << 3) - n0;  // columns past the end: any valid chunk
#pragma unroll
        for (int i = 0; i < NBL; ++i) {
            const int k = i * 32 + (tid >> 4), logical = (tid & 15) ^ rc_swz(k);
            offB[i] = (uint32_t)min(k, kleft - 1) * (uint32_t)(p.B[1].ld * 2) + (uint32_t)min(logical * 8, clast) * 2u;
        }
        baseB = reinterpret_cast<const char*>(p.B[1].ptr) + ((int64_t)k0 * p.B[1].ld + n0) * 2;
    };
    auto is_tail = [&](int t) { return t == tail0 || t == tail1; };
    auto advance_a = [&](int kt) {  // to tile kt, the successor
        if (kt == nkt0 || is_tail(kt)) setup_a(kt);
        else baseA += BK * 2;
    };
    auto advance_q = [&](int kt) {
        if (kt == nkt0 || (BRC && is_tail(kt))) setup_q(kt);
        else baseQ += stepQ, baseS += stepS;
    };
    auto advance_b = [&](int kt) {
        if (is_tail(kt)) setup_b(kt);
        else baseB += (int64_t)BK * p.B[1].ld * 2;
    };
    const uint32_t lds0 = LOQT_LDS_ADDR(smem), lwave = (uint32_t)wave * 1024u;
    // Inline assembly (M0: the LDS address, and one wait state between its write and the load) for the reasons given in nt_tile.h:
    // the compiler would wait for all of the loads in front of LDS reads.
    auto direct_load = [&](uint32_t o, const char* base, uint32_t dst, uint32_t at) {
        asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(o), "s"(base), "s"(dst), "i"(at) : "memory", "scc");
    };
    auto load_a = [&](int n, const char* stage) {
        direct_load(offA[n], baseA, lds0 + (uint32_t)(stage - smem) + lwave, (uint32_t)(n * 8192));
    };
    auto load_b = [&](int i, const char* stage) {
        direct_load(offB[i], baseB, lds0 + (uint32_t)(stage - smem) + lwave, (uint32_t)(BM * ROWB + i * 8192));
    };
    // codes and scales: two loads by half of the lanes (EXEC is all ones before and after: uniform control flow)
    auto load_q = [&](const char* slot) {
        const uint32_t dst = lds0 + (uint32_t)(slot - smem) + (uint32_t)wave * 512u;
        const uint32_t dsts = lds0 + (uint32_t)(slot - smem) + 4096u + (uint32_t)wave * 128u;
        asm volatile(
            "s_mov_b32 m0, %2\n\t"
            "s_mov_b32 exec_hi, 0\n\t"
            "global_load_lds_dwordx4 %0, %1\n\t"
            "s_mov_b32 m0, %5\n\t"
            "s_nop 0\n\t"
            "global_load_lds_dword %3, %4\n\t"
            "s_mov_b32 exec_hi, -1"
            ::"v"(offQ), "s"(baseQ), "s"(dst), "v"(offS), "s"(baseS), "s"(dsts) : "memory");
    };
    // clears A past the end of the contraction (codes past it are finite weights, or k rows repeated)
    auto cut_tile = [&](int kt, char* stage) {
        const bool seg = kt >= nkt0;
        const int kleft = (seg ? p.A[1].K : p.A[0].K) - (kt - (seg ? nkt0 : 0)) * BK;
        const int nv = kleft - 8 * ((tid & 7) ^ kc_swz(tid >> 3));
        if (nv < 8) {
            uint32_t keep[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) keep[d] = 2 * d + 1 < nv ? 0xffffffffu : 2 * d < nv ? 0xffffu : 0u;
#pragma unroll 1
            for (int i = 0; i < C::NA; ++i) {
                uint4* q = reinterpret_cast<uint4*>(stage + i * 8192 + tid * 16);
                const uint4 v = *q;
                *q = make_uint4(v.x & keep[0], v.y & keep[1], v.z & keep[2], v.w & keep[3]);
            }
        }
    };

    // ---- expansion of the thread's 16 codes, one per step: look-up of code t, then, eight steps later, its product with
    // the scale; two products make a dword, eight a chunk of 16 bytes.  Thread tid has codes 16*(tid%4) on of row tid/4, or,
    // K x rows, of k row tid/8, columns 16*(tid%8) on.
    uint32_t cw[2], odd = 0, even = 0, o[4];
    float am = 0.f, lv[16];
    auto fetch_codes = [&](const char* slot) {
        const uint2 c = *reinterpret_cast<const uint2*>(slot + tid * 8);
        cw[0] = c.x, cw[1] = c.y;
        am = *reinterpret_cast<const float*>(slot + 4096 + (tid >> 1) * 4);
    };
    int wbase, wsw;  // where the thread's chunks go: row (or k row) of the tile, its swizzle
    if constexpr (!BRC) {
        wbase = BM * ROWB + (tid >> 2) * ROWB;
        wsw = kc_swz(tid >> 2);
    } else {
        wbase = BM * ROWB + (tid >> 3) * (BN * 2);
        wsw = rc_swz(tid >> 3);
    }
    constexpr int STEPS = 24;
    auto step = [&](auto t_tag, char* stage) {
        constexpr int t = decltype(t_tag)::value;
        if constexpr (t < 16) {
            if constexpr (t % 8 == 0) {  // even elements in the high nibbles; byte offsets into the table
                even = (cw[t / 8] >> 2) & 0x3c3c3c3cu;
                odd = (cw[t / 8] << 2) & 0x3c3c3c3cu;
            }
            lv[t] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(lut) + (((t & 1 ? odd : even) >> (8 * ((t % 8) / 2))) & 0xffu));
        }
        if constexpr (t >= 8) {
            constexpr int c = t - 8;
            lv[c] *= am;
            if constexpr (c % 2 == 1) o[(c % 8) / 2] = pack_bf16(lv[c - 1], lv[c]);
            if constexpr (c % 8 == 7) {
                const int logical = (BRC ? (tid & 7) * 2 : (tid & 3) * 2) + c / 8;
                *reinterpret_cast<uint4*>(stage + wbase + ((logical ^ wsw) << 4)) = make_uint4(o[0], o[1], o[2], o[3]);
            }
        }
    };

    // ---- fragments (nt_tile.h)
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
    bf16x8 fa[2][TM], fb[2][TN];
    auto read_frag = [&](int ks, int nb, int u, const char* stage) {
        if (u < TM) {
            fa[nb][u] = *reinterpret_cast<const bf16x8*>(stage + a_ko[ks] + u * 16 * ROWB);
        } else if constexpr (BRC) {
            const char* ptr = stage + b_rc[u - TM] + 32 * ks * (BN * 2);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(ptr));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(ptr + 4 * (BN * 2)));
            fb[nb][u - TM] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        } else {
            fb[nb][u - TM] = *reinterpret_cast<const bf16x8*>(stage + b_ko[ks] + (u - TM) * 16 * ROWB);
        }
    };

    if (tid < 16) lut[tid] = kNf4Levels[tid];
    constexpr int NU = TM + TN, Q = U / 4, LS = 3 * Q;  // fragments; a quarter of the slots; slots that carry loads
    auto run = [&](auto codes_tag) {
        constexpr bool CODES = decltype(codes_tag)::value;
        constexpr int NL = C::NA + (CODES ? 1 : NBL);  // loads of a k-tile (codes and scales count once, and come last)
        constexpr int LBY = 2 * Q * NL / LS;           // of which precede barrier Y
        static_assert(!CODES || LBY <= C::NA, "");
        // A of two tiles, codes of four (past the range the last one again, into slots nobody reads)
        setup_a(kt_begin);
        if constexpr (CODES) setup_q(kt_begin);
        else setup_b(kt_begin);
#pragma unroll
        for (int t = 0; t < (CODES ? NQ : 2); ++t) {
            if (t > 0 && kt_begin + t < kt_end) {
                if (t < 2) advance_a(kt_begin + t);
                if constexpr (CODES) advance_q(kt_begin + t);
                else advance_b(kt_begin + t);
            }
            if (t < 2) {
#pragma unroll
                for (int n = 0; n < C::NA; ++n) load_a(n, smem + t * STAGE);
            }
            if constexpr (CODES) {
                load_q(qring + t * QBYTES);
            } else {
#pragma unroll
                for (int i = 0; i < NBL; ++i) load_b(i, smem + t * STAGE);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (is_tail(kt_begin)) cut_tile(kt_begin, smem);
        if constexpr (CODES) {
            fetch_codes(qring);
            auto here = [&](auto t) { step(t, smem); };
            each<0>(std::make_integer_sequence<int, STEPS>{}, here);
            fetch_codes(qring + QBYTES);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < TM + TN; ++u) read_frag(0, 0, u, smem);
        for (int kt = kt_begin; kt < kt_end; ++kt) {
            const int it = kt - kt_begin;
            char* cur = smem + (it & 1) * STAGE;
            char* nxt = smem + ((it & 1) ^ 1) * STAGE;
            const char* qnext = qring + ((it + 2) % NQ) * QBYTES;  // codes of tile kt+2
            const char* qload = qring + (it % NQ) * QBYTES;        // those of tile kt are used up: tile kt+4
            auto slot = [&](auto s_tag) {
                constexpr int s = decltype(s_tag)::value, CB = s / (U / 2), m = s % (U / 2), i = m / TN, j = m % TN;
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[CB][j], fa[CB][i], acc[i][j], 0, 0, 0);
                if constexpr (s < Q) {
#pragma unroll
                    for (int u = s * NU / Q; u < (s + 1) * NU / Q; ++u) read_frag(1, 1, u, cur);
                } else {
                    constexpr int g = s - Q;
#pragma unroll
                    for (int n = g * NL / LS; n < (g + 1) * NL / LS; ++n) {
                        if (n < C::NA) load_a(n, cur);
                        else if (CODES) load_q(qload);
                        else load_b(n - C::NA, cur);
                    }
                }
                if constexpr (s < 3 * Q) {
                    if constexpr (CODES) {
                        auto there = [&](auto t) { step(t, nxt); };
                        each<s * STEPS / (3 * Q)>(std::make_integer_sequence<int, (s + 1) * STEPS / (3 * Q) - s * STEPS / (3 * Q)>{}, there);
                    }
                } else {
                    constexpr int r = s - 3 * Q;
#pragma unroll
                    for (int u = r * NU / Q; u < (r + 1) * NU / Q; ++u) read_frag(0, 0, u, nxt);
                    if constexpr (CODES && r == Q - 1) fetch_codes(qnext);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            each<0>(std::make_integer_sequence<int, Q>{}, slot);
            __syncthreads();  // X
            if (kt + 2 < kt_end) {
                advance_a(kt + 2);
                if constexpr (!CODES) advance_b(kt + 2);
            }
            if constexpr (CODES) {
                if (kt + NQ < kt_end) advance_q(kt + NQ);
            }
            each<Q>(std::make_integer_sequence<int, 2 * Q>{}, slot);
            // of the iteration before, A (and B) must have landed and the two loads of codes, its last ones, need not; the
            // loads of this iteration so far may stay in flight as well
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LBY + (CODES ? 2 : 0)) : "memory");
            __syncthreads();  // Y
            if (is_tail(kt + 1)) {
                cut_tile(kt + 1, nxt);
                __syncthreads();
            }
            each<3 * Q>(std::make_integer_sequence<int, Q>{}, slot);
        }
    };
    if (kt_begin < kt_end) {
        if (BRC && extra) run(std::integral_constant<bool, !BRC>{});
        else run(std::integral_constant<bool, true>{});
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loads past the end

    // lane: row 16 i + (lane & 15), columns 16 j + 4 (lane >> 4) .. +3
    float* out = reinterpret_cast<float*>(p.C) + (int64_t)blockIdx.y * p.M * p.ldc;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + wm * C::WTM + i * 16 + frow;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + wn * C::WTN + j * 16 + 4 * q4;
            // (the pitch is a multiple of 4: columns N .. ldc-1 of the slices are scratch)
            if (m < p.M && n < p.ldc)
                *reinterpret_cast<float4*>(out + (int64_t)m * p.ldc + n) =
                    make_float4(p.alpha * acc[i][j][0], p.alpha * acc[i][j][1], p.alpha * acc[i][j][2], p.alpha * acc[i][j][3]);
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
    hipLaunchKernelGGL((nf4_tile_kernel<BM, BRC>), dim3((tiles + 7) / 8 * 8, p.splits + (BRC && p.A[1].K > 0 ? 1 : 0)), dim3(THREADS), Cfg<BM>::SMEM, st, p);
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
// rest of a tile, as in plan_nt
int nf4_tile_splits(int64_t M, int64_t N, int64_t nkt, int extra, int64_t max_splits) {
    const int64_t bm = M <= 64 ? 64 : M <= 128 ? 128 : 256;
    const double alone = bm == 64 ? 0.80 : bm == 128 ? 0.85 : 0.95, full = bm == 64 ? 0.95 : bm == 128 ? 1.05 : 1.35;
    const int64_t tiles = (M + bm - 1) / bm * ((N + BN - 1) / BN);
    int best = 1;
    double best_cost = 0.0;
    for (int64_t s = 1; s <= std::min<int64_t>(max_splits, NT_MAX_SPLITS); ++s) {
        const int64_t per = (nkt + s - 1) / s, wgs = tiles * (s + extra);
        if (s > 1 && (per < 4 || (nkt + per - 1) / per != s)) continue;
        auto one = [&](int64_t w) { return (double)per * (alone + (full - alone) * (double)w / 256.0) + 6.0; };
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
