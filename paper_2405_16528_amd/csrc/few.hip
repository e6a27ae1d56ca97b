// Forward products with few tokens (T <= 32): y = x deq(W)^T + U deq(P)^T and U = s x B^T, the weight streamed once.
//
// With a handful of tokens the product is a read of the weight: 0.5625 bytes per element from HBM, a few matrix
// instructions on the way.  Expanding the weight to bf16 first moves 2.56 + 2 bytes per element and then feeds 64-row
// tiles of which a quarter is tokens.  Here a lane reads 32 codes (16 bytes) of one weight row, looks their levels up
// (bf16 table in LDS) and hands them to v_mfma_f32_16x16x32_bf16 as they are; a block of 64 is summed on its own and
// then scaled by the block's absmax in fp32.  (The levels are rounded to bf16 before the scaling instead of after it:
// 1.4e-3 rms of the weight against 1.7e-3.)  The matrix instruction wants the eight k from 32 j + 8 q on in lane group q;
// the group has read 32 q .. 32 q + 31, so the four dwords of codes are transposed across the four groups of 16 lanes
// first (two lane swaps per pair).  Neither operand passes through LDS.
//
// A work-group owns 16 * RT weight rows over the whole contraction; its 16 waves take every 16th chunk of 128 and their
// sums meet in LDS in a fixed order, so there are no slices in memory and no second launch.  What bounds it is a chain inside
// the wave, not a rate: a wave has two or three chunks and loads x of one only after the products of the one before, the
// codes of the next two after both.  At 11008 x 5056 and 16 tokens a work-group of 48 rows reads 162 KB of x and 137 KB of
// codes and scales in 13.8 us, 9 bytes per cycle and unit; by the counters (11008 x 4096) its waves wait for loads and barriers
// in 46 % of their cycles and for a place to issue (look-ups and their addresses) in 40 %, the matrix units are busy in 5 %.
// More rows per work-group share the chain, until the last work-groups start late: so RT grows with the number of rows.
// Kernel, us, contraction 5056, the same weight each time / 24 weights in turn (by 750 MB at 11008 rows):
//   16 tokens    RT 1          RT 2          RT 3          RT 4            32 tokens   RT 1          RT 2          RT 3          RT 4
//   4096 rows     9.4 / 10.1   11.2 / 12.2   13.4 / 15.2   15.8 / 18.4                 12.7 / 14.1   14.3 / 16.1   16.7 / 18.9   24.6 / 27.3
//   11008 rows   19.4 / 20.6   19.2 / 22.1   13.8 / 16.3   16.2 / 19.6                 36.6 / 37.3   28.8 / 31.1   18.2 / 20.4   26.7 / 30.2
// U = s x B^T needs a launch before y, and the chip is nearly idle in it.  So where the work-groups of both fit on the chip at once and the contraction is long U
// goes out beside x deq(W)^T, which does not need it, whose sums wait in fp32 for the second launch, U deq(P)^T.
// The whole call at 16 x 11008 x 4096, rank 1024: 165 -> 23.3 (expanded weight -> this; 78 with the expanded weight on the
// narrow tiles of gemm_nt.hip), 160 -> 51 on buffers that nothing has read before.  From 33 tokens on x costs more than the expanded weight (4096 x 11008, 64 tokens: 98 against 79).
#include <type_traits>

#include "loqt_internal.h"

namespace loqt {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int CH = 128;  // contraction of one chunk
constexpr int NW = 16;   // waves of a work-group

// The levels are kept in 64ths, and the sums of NF4 products with them: a block's 64 products, which have no scale yet, then
// stay in fp32's range for every x that bf16 holds.  (A power of two: no other bit changes.)
constexpr float UNIT = 64.f;

typedef __attribute__((ext_vector_type(8))) short s16x8;

// the bf16 levels of 8 codes (element e in byte e / 2, even e in the high nibble)
__device__ __forceinline__ bf16x8 levels8(uint32_t w, const char* lut) {
    const uint32_t odd = (w << 1) & 0x1e1e1e1eu, even = (w >> 3) & 0x1e1e1e1eu;  // byte offsets into the table
    s16x8 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = *reinterpret_cast<const short*>(lut + ((even >> (8 * i)) & 0xffu));
        v[2 * i + 1] = *reinterpret_cast<const short*>(lut + ((odd >> (8 * i)) & 0xffu));
    }
    return __builtin_bit_cast(bf16x8, v);
}

// elements k .. k+7 of a bf16 row (16-byte aligned pieces, the pitch a multiple of 8); MASK: those from K on as zero.
// Always one unconditional load: a branch around it would make every load wait for the ones before.
template <bool MASK>
__device__ __forceinline__ bf16x8 load8(const uint16_t* row, int k, int K) {
    if constexpr (!MASK) return *reinterpret_cast<const bf16x8*>(row + k);
    uint4 v = *reinterpret_cast<const uint4*>(row + (k < K ? k : 0));
    uint32_t* w = reinterpret_cast<uint32_t*>(&v);
#pragma unroll
    for (int d = 0; d < 4; ++d) w[d] &= k + 2 * d + 1 < K ? 0xffffffffu : k + 2 * d < K ? 0xffffu : 0u;
    return __builtin_bit_cast(bf16x8, v);
}

typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
// lanes 32-63 of a change places with lanes 0-31 of b; rows 1 and 3 of 16 lanes of a with rows 0 and 2 of b
__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b) {
    const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(a, b, false, false));
    a = r[0], b = r[1];
}
__device__ __forceinline__ void swap16(uint32_t& a, uint32_t& b) {
    const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(a, b, false, false));
    a = r[0], b = r[1];
}

struct Seg {  // one K segment: x (bf16, T x K) and the weight rows (NF4 or bf16, N x K)
    const uint16_t* a;
    int64_t lda;
    const void* w;
    const float* absmax;
    int64_t ldw;
    int K;
};

template <bool NF4>
struct Weights;  // one chunk of 16 rows: what a lane holds of its row; k0: start of the chunk
template <>
struct Weights<true> {
    uint32_t d[4];
    float am[2];
    // Padding nibbles are levels like any other and meet zeros of x; a block wholly past K has no scale to rely on.
    template <bool MASK>
    __device__ __forceinline__ void load(const Seg& s, int row, int k0, int q) {
        int k = k0 + 32 * q, k1 = k0 + 64;
        if (MASK) k = k < s.ldw ? k : k0, k1 = k1 < s.K ? k1 : k0;
        const uint4 c = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint8_t*>(s.w) + (int64_t)row * (s.ldw >> 1) + (k >> 1));
        d[0] = c.x, d[1] = c.y, d[2] = c.z, d[3] = c.w;
        const float* a = s.absmax + (int64_t)row * (s.ldw >> 6);
        am[0] = a[k0 >> 6], am[1] = a[k1 >> 6];
    }
    __device__ __forceinline__ void ready() {  // dword j of lane group q becomes dword q of group j
        swap32(d[0], d[2]);
        swap32(d[1], d[3]);
        swap16(d[0], d[1]);
        swap16(d[2], d[3]);
    }
    __device__ __forceinline__ bf16x8 frag(int j, const char* lut) const { return levels8(d[j], lut); }
    __device__ __forceinline__ float scale(int h) const { return am[h]; }
};
template <>
struct Weights<false> {
    bf16x8 v[4];
    template <bool MASK>
    __device__ __forceinline__ void load(const Seg& s, int row, int k0, int q) {
        const uint16_t* r = reinterpret_cast<const uint16_t*>(s.w) + (int64_t)row * s.ldw;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = load8<MASK>(r, k0 + 32 * j + 8 * q, s.K);
    }
    __device__ __forceinline__ void ready() {}
    __device__ __forceinline__ bf16x8 frag(int j, const char*) const { return v[j]; }
    __device__ __forceinline__ float scale(int) const { return 1.f; }
};

// what becomes of the sums: bf16 result; fp32 sums for a later launch (four tokens of a row side by side: [T / 4][N]); bf16 result of
// them and those of an earlier launch
enum { TO_BF16, TO_SUMS, ADD_SUMS };

// C[T x N] = alpha * sum over both segments of A_seg[T x K_seg] * B_seg[N x K_seg]^T; A bf16, B NF4 or bf16.  blk: which 16 RT rows of
// B; lds: NW / 2 * RT * NT * 64 elements
template <bool NF4, int NT, int RT, int OUT>
__device__ __forceinline__ void few_tokens_rows(const GemmParams& p, const int blk, f32x4* const lds) {
    f32x4(*const red)[RT * NT][64] = reinterpret_cast<f32x4(*)[RT * NT][64]>(lds);
    uint16_t* lut = reinterpret_cast<uint16_t*>(red);  // until the sums need the place
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const char* lutc = reinterpret_cast<const char*>(lut);
    const int q = lane >> 4, l16 = lane & 15;
    const int n0 = blk * (16 * RT);
    int row[RT], tok[NT];
#pragma unroll
    for (int i = 0; i < RT; ++i) row[i] = min(n0 + 16 * i + l16, p.N - 1);  // rows and tokens past the end: any valid one
#pragma unroll
    for (int t = 0; t < NT; ++t) tok[t] = min(16 * t + l16, p.M - 1);
    f32x4 acc[RT][NT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    // the place in the result of this thread's four sums, in the end
    const int um = 16 * ((tid >> 6) % NT) + 4 * q, un = n0 + 16 * ((tid >> 6) / NT) + l16;
    static_assert(RT * NT <= NW, "one place per thread");
    f32x4* const sums = reinterpret_cast<f32x4*>(p.split_ws) + (int64_t)(um >> 2) * p.N + un;
    const bool mine = tid < RT * NT * 64 && un < p.N && um < p.M;
    f32x4 before{0.f, 0.f, 0.f, 0.f};
    if constexpr (OUT == ADD_SUMS)
        if (mine) before = *sums;

    const Seg s0{reinterpret_cast<const uint16_t*>(p.A[0].ptr), p.A[0].ld, p.B[0].ptr, p.B[0].absmax, p.B[0].ld, p.A[0].K};
    const Seg s1{reinterpret_cast<const uint16_t*>(p.A[1].ptr), p.A[1].ld, p.B[1].ptr, p.B[1].absmax, p.B[1].ld, p.A[1].K};
    auto seg = [&](bool second) {  // (scalar selects; a run-time index would go through memory)
        return Seg{second ? s1.a : s0.a, second ? s1.lda : s0.lda, second ? s1.w : s0.w, second ? s1.absmax : s0.absmax,
                   second ? s1.ldw : s0.ldw, second ? s1.K : s0.K};
    };
    // chunks whose weights a wave has in flight
    constexpr int NB = !NF4 && RT == 3 ? 1 : 2;
    Weights<NF4> w[NB][RT];
    bf16x8 x[NT][4];
    auto load_w = [&](auto mask, int b, const Seg& s, int k0) {
#pragma unroll
        for (int i = 0; i < RT; ++i) w[b][i].template load<decltype(mask)::value>(s, row[i], k0, q);
    };
    auto load_x = [&](auto mask, const Seg& s, int k0) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                x[t][j] = load8<decltype(mask)::value>(s.a + tok[t] * s.lda, k0 + 32 * j + 8 * q, s.K);
    };
    auto multiply = [&](int b) {
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            w[b][i].ready();
#pragma unroll
            for (int h = 0; h < 2; ++h) {  // blocks of 64
                const bf16x8 f0 = w[b][i].frag(2 * h, lutc), f1 = w[b][i].frag(2 * h + 1, lutc);
                const float sc = w[b][i].scale(h);
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    f32x4 a = NF4 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[i][t];
                    a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[t][2 * h], f0, a, 0, 0, 0);
                    a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[t][2 * h + 1], f1, a, 0, 0, 0);
                    if (NF4) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[i][t][e] = __builtin_fmaf(sc, a[e], acc[i][t][e]);
                    } else {
                        acc[i][t] = a;
                    }
                }
            }
        }
    };
    constexpr std::integral_constant<bool, false> WHOLE{};
    constexpr std::integral_constant<bool, true> CUT{};
    // whole chunks: batches of NB per wave.  Past the last one nothing is loaded either (scalar branches): a wave that
    // fetches a chunk it has no use for holds up the loads of the others.  Repeating the last chunk instead, whole calls in us
    // on bf16 weights (in brackets the plain products of gemm_nt.hip): 7232 x 128, rank 24, 32 tokens 21.7 -> 6.5 (8.7);
    // 2112 x 128, rank 112, 16 tokens 14.8 -> 5.7 (9.0); 512 x 512, rank 128, 32 tokens 17.1 -> 8.0 (11.7).
    const int f0 = s0.K / CH, full = f0 + s1.K / CH;
    auto whole = [&](int c, auto&& f) {
        if (c >= full) return;
        const bool second = c >= f0;
        f(seg(second), (second ? c - f0 : c) * CH);
    };
    auto batch = [&](int c0) {
#pragma unroll
        for (int b = 0; b < NB; ++b) whole(c0 + b * NW, [&](const Seg& s, int k0) { load_w(WHOLE, b, s, k0); });
        whole(c0, [&](const Seg& s, int k0) { load_x(WHOLE, s, k0); });
    };
    batch(wave);
    if (NF4) {
        if (tid < 16) lut[tid] = (uint16_t)(pack_bf16(kNf4Levels[tid] / UNIT, 0.f) & 0xffffu);
        __syncthreads();
    }
    for (int c0 = wave; c0 < full;) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (c0 + b * NW < full) multiply(b);
            if (b + 1 < NB) whole(c0 + (b + 1) * NW, [&](const Seg& s, int k0) { load_x(WHOLE, s, k0); });
        }
        c0 += NB * NW;
        if (c0 < full) batch(c0);
    }
    // what is left of a segment that does not end on a chunk
#pragma unroll 1
    for (int t = 0; t < 2; ++t) {
        const Seg s = seg(t == 1);
        if (s.K % CH == 0 || wave != (full + t) % NW) continue;
        load_w(CUT, 0, s, s.K / CH * CH);
        load_x(CUT, s, s.K / CH * CH);
        multiply(0);
    }
    // lane: row 16 i + (lane & 15), tokens 16 t + 4 (lane >> 4) .. +3.  The upper half of the waves hands over to the
    // lower half first (half the LDS).
    auto put = [&](int slot, bool add) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t) red[slot][i * NT + t][lane] = add ? red[slot][i * NT + t][lane] + acc[i][t] : acc[i][t];
    };
    __syncthreads();
    if (wave >= NW / 2) put(wave - NW / 2, false);
    __syncthreads();
    if (wave < NW / 2) put(wave, true);
    __syncthreads();
    if (!mine) return;
    f32x4 s = red[0][tid >> 6][lane];
#pragma unroll
    for (int v = 1; v < NW / 2; ++v) s += red[v][tid >> 6][lane];
    if constexpr (NF4) s *= UNIT;
    if constexpr (OUT == TO_SUMS) {
        *sums = s;
    } else {
        if constexpr (OUT == ADD_SUMS) s += before;
        uint16_t* dst = reinterpret_cast<uint16_t*>(p.C) + (int64_t)um * p.ldc + un;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (um + e < p.M) dst[e * p.ldc] = (uint16_t)(pack_bf16(p.alpha * s[e], 0.f) & 0xffffu);
    }
}

template <bool NF4, int NT, int RT, int OUT>
__global__ __launch_bounds__(64 * NW) void few_tokens_kernel(const GemmParams p) {
    __shared__ f32x4 lds[NW / 2 * RT * NT * 64];
    few_tokens_rows<NF4, NT, RT, OUT>(p, blockIdx.x, lds);
}

// U on the first u_blocks work-groups (16 RU rows each), the sums of x deq(W)^T on the others
template <int NT, int RT, int RU>
__global__ __launch_bounds__(64 * NW) void few_beside_kernel(const GemmParams u, const int u_blocks, const GemmParams w) {
    __shared__ f32x4 lds[NW / 2 * (RT > RU ? RT : RU) * NT * 64];
    if ((int)blockIdx.x < u_blocks) few_tokens_rows<false, NT, RU, TO_BF16>(u, blockIdx.x, lds);
    else few_tokens_rows<true, NT, RT, TO_SUMS>(w, (int)blockIdx.x - u_blocks, lds);
}

template <bool NF4, int NT, int RT, int OUT>
hipError_t launch_rows(const GemmParams& p, hipStream_t st) {
    hipLaunchKernelGGL((few_tokens_kernel<NF4, NT, RT, OUT>), dim3((p.N + 16 * RT - 1) / (16 * RT)), dim3(64 * NW), 0, st, p);
    return hipGetLastError();
}

// Rows per work-group (16 RT): as few as leave at most one work-group of 16 waves for a compute unit.  Beyond that the one of
// 48 and 64 whose rounds are cheaper by their rows (64 rows of two token tiles are 20 registers short and count for 80: 32
// tokens on 13568 x 5376, us, 55 in two rounds of 48 and 45 in one of 64; on 18752 x 7872 61 and 82 in two rounds of either).
// Rows in bf16 take 64 of the 128 registers at two chunks in flight; so 48 of them go with one chunk, and there is no form of 64.
template <bool NF4, int NT, int OUT = TO_BF16>
hipError_t launch_tokens(const GemmParams& p, hipStream_t st) {
    const int tiles = (p.N + 15) / 16;
    if (tiles <= 256) return launch_rows<NF4, NT, 1, OUT>(p, st);
    if (tiles <= 512) return launch_rows<NF4, NT, 2, OUT>(p, st);
    if constexpr (NF4 && (NT == 1 || OUT != ADD_SUMS))  // (sums of two token tiles come from 768 tiles of rows at most: rows_beside)
        if ((tiles + 1023) / 1024 * (NT == 1 ? 4 : 5) < (tiles + 767) / 768 * 3) return launch_rows<NF4, NT, 4, OUT>(p, st);
    return launch_rows<NF4, NT, 3, OUT>(p, st);
}

// Rows per work-group of W and of U, 16 each: the fewest with which both together leave at most one work-group for a compute unit.
// Whole calls, us, U first / U beside W, 1, 16 and 32 tokens:
//   11008 x 4096, rank 512   19.9 / 17.2   23.4 / 19.3   27.4 / 24.2
//   4096 x 4096, rank 1024   13.7 / 12.9   19.3 / 15.0   23.7 / 19.7       13824 x 5120, rank 1024   26.0 / 22.7   29.4 / 25.5   (no room)
//   5120 x 5120, rank 1024   18.6 / 13.9   22.9 / 17.0   28.3 / 22.8       4096 x 11008, rank 1024   23.3 / 19.6   30.1 / 26.6   39.6 / 36.7
// U on 48 rows was no faster than U first (11008 x 4096, rank 1024: 20.1 / 21.0, 24.7 / 24.3, 29.3 / 29.5).  64 rows of W where 48 do
// without U's work-groups pay from 9 tokens up (the same: 20.4 / 21.4 at one token, 22.2 / 22.5 at 8, 24.6 / 23.3 at 16).
struct Beside {
    int rt, ru;
};
Beside rows_beside(int T, int N, int r) {
    const int tw = (N + 15) / 16, tu = (r + 15) / 16;
    for (const Beside b : {Beside{1, 1}, Beside{2, 1}, Beside{3, 1}, Beside{3, 2}, Beside{4, 1}, Beside{4, 2}})
        if ((b.rt < 4 || (T <= 16 && (tw > 768 || T > 8))) && (tw + b.rt - 1) / b.rt + (tu + b.ru - 1) / b.ru <= 256) return b;
    return {0, 0};
}

template <int NT, int RT, int RU>
hipError_t launch_beside(const GemmParams& u, const GemmParams& w, hipStream_t st) {
    const int ub = (u.N + 16 * RU - 1) / (16 * RU);
    hipLaunchKernelGGL((few_beside_kernel<NT, RT, RU>), dim3(ub + (w.N + 16 * RT - 1) / (16 * RT)), dim3(64 * NW), 0, st, u, ub, w);
    return hipGetLastError();
}

template <int NT>
hipError_t launch_beside(const GemmParams& u, const GemmParams& w, hipStream_t st) {
    const Beside b = rows_beside(w.M, w.N, u.N);
    if constexpr (NT == 1)
        if (b.rt == 4) return b.ru == 1 ? launch_beside<NT, 4, 1>(u, w, st) : launch_beside<NT, 4, 2>(u, w, st);
    if (b.rt == 1) return launch_beside<NT, 1, 1>(u, w, st);
    if (b.rt == 2) return launch_beside<NT, 2, 1>(u, w, st);
    if (b.rt == 3) return b.ru == 1 ? launch_beside<NT, 3, 1>(u, w, st) : launch_beside<NT, 3, 2>(u, w, st);
    return hipErrorInvalidValue;
}

}  // namespace

// It pays where U's chain over the contraction is long against the work-groups' other costs, the more rows the later: random calls of 1 to
// 32 tokens, beside / first, by contraction:
//                          800 to 1100    1400 to 1800    1800 to 2300    2300 to 3000    4000 to 5500
//   to 4096 rows           1.01           0.94 to 1.01    0.88 to 1.00    0.83 to 0.96    0.81 to 0.83
//   to 8192                1.03 to 1.08   0.99 to 1.03    0.95 to 1.00    0.87 to 0.93    0.83 to 0.84
//   beyond                 1.11 to 1.12   1.04 to 1.08    1.00 to 1.04    0.95 to 0.98    0.88 to 0.90
// Beside at any length, 4832 of 45000 calls were slower by more than 3 % than with U first (11600 x 218, 21 tokens, 8.6 / 10.7 us); with
// these lines 354 are.
bool few_layer_fits(int T, int N, int K, int r, size_t ws_bytes) {
    return K >= (N <= 4096 ? 1300 : N <= 8192 ? 1800 : 2300) && rows_beside(T, N, r).rt > 0 && ws_bytes >= (size_t)((T + 3) / 4) * N * 16;
}

hipError_t launch_few_layer(const GemmParams& u, const GemmParams& w, const GemmParams& q, hipStream_t st) {
    if (w.M < 1 || w.M > FEW_TOKENS_MAX) return hipErrorInvalidValue;
    {
        TimedLaunch tl(SLOT_GEMM_U, st);
        const hipError_t e = w.M <= 16 ? launch_beside<1>(u, w, st) : launch_beside<2>(u, w, st);
        if (e != hipSuccess) return e;
    }
    TimedLaunch tl(SLOT_GEMM_Y, st);
    return w.M <= 16 ? launch_tokens<true, 1, ADD_SUMS>(q, st) : launch_tokens<true, 2, ADD_SUMS>(q, st);
}

hipError_t launch_few_tokens(int slot, bool nf4, const GemmParams& p, hipStream_t st) {
    if (p.M < 1 || p.M > FEW_TOKENS_MAX) return hipErrorInvalidValue;
    TimedLaunch tl(slot, st);
    if (p.M <= 16) return nf4 ? launch_tokens<true, 1>(p, st) : launch_tokens<false, 1>(p, st);
    return nf4 ? launch_tokens<true, 2>(p, st) : launch_tokens<false, 2>(p, st);
}

}  // namespace loqt
