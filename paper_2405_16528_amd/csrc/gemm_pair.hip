// Products that do not need each other as one launch: the gradient of the factor beside dx, Z = s dy deq(P) (or V = s x deq(Q))
// beside the fold of the weight, U = s x B^T beside the bf16 copies of W and P.
//
// Below a few thousand tokens a product is one partly filled round of small tiles for 5 to 20 us, a launch costs 3 to 4 us of
// them (2.6 of host time, 1.4 between kernels, the first loads of every work-group on top), and the small products (a few
// dozen work-groups with long contractions) leave most of the chip idle.  One grid over the tiles of both: the first work-groups
// belong to the product with the longer tiles, the others follow it onto whatever compute unit is free.  Both keep the slices
// they have alone, and but for the fold, which has two work-groups to a unit here and a rule for that in launch_z_fold, their tiles.
// Any tile sums k in the same order, so the results are the same bits.  Only tiles of up to 128x128 take
// part; larger products run for hundreds of microseconds.
#include <string.h>

#include <algorithm>

#include "nt_tile.h"

namespace loqt {

namespace {

template <int BM_, int BN_, int EPI_, bool ARC_, bool BRC_, int NS_, bool LOADERS_ = false>
struct Part {
    static constexpr int BM = BM_, BN = BN_, EPI = EPI_, NS = NS_, SMEM = NtCfg<BM, BN, NS>::SMEM, PER_CU = NtCfg<BM, BN, NS>::PER_CU;
    static constexpr bool ARC = ARC_, BRC = BRC_, LOADERS = LOADERS_;
    static_assert(PER_CU >= 2 || LOADERS, "");
    static int grid(const GemmParams& p) { return (((p.M + BM - 1) / BM) * ((p.N + BN - 1) / BN) + 7) / 8 * 8; }
    // `b`: work-group of this part; `per`: of them belong to a slice (a multiple of 8, so that b % 8 is the XCD)
    static __device__ __forceinline__ void run(const GemmParams& p, int b, int per) {
        const int split = EPI == EPI_F32_SPLITK ? b / per : 0, r = b - split * per;
        nt_gemm_tile<BM, BN, EPI, ARC, BRC, NS, false, false, LOADERS>(p, (r & 7) * (per >> 3) + (r >> 3), split);
    }
};
template <int EPI, bool ARC, bool BRC>
using T64x64 = Part<64, 64, EPI, ARC, BRC, 4>;
template <int EPI, bool ARC, bool BRC>
using T64x128 = Part<64, 128, EPI, ARC, BRC, 3>;
template <int EPI, bool ARC, bool BRC>
using T128x128 = Part<128, 128, EPI, ARC, BRC, 2>;

// with waves of their own for the loads (nt_tile.h), as they have alone
template <int EPI, bool ARC, bool BRC>
using L64x64 = Part<64, 64, EPI, ARC, BRC, 4, true>;
template <int EPI, bool ARC, bool BRC>
using L64x128 = Part<64, 128, EPI, ARC, BRC, 3, true>;
template <int EPI, bool ARC, bool BRC>
using L128x128 = Part<128, 128, EPI, ARC, BRC, 3, true>;

template <class A, class B>
constexpr int pair_smem = A::SMEM > B::SMEM ? A::SMEM : B::SMEM;
template <class A, class B>
constexpr int pair_threads = A::LOADERS ? 512 : 256;
template <class A, class B>
constexpr int pair_per_simd = (A::LOADERS ? 2 : 1) * (A::PER_CU >= 2 && B::PER_CU >= 2 ? 2 : 1);  // waves

template <class A, class B>
__global__ __launch_bounds__((pair_threads<A, B>), (pair_per_simd<A, B>)) void nt_pair_kernel(const GemmParams a, const GemmParams b, const int a_per, const int a_all,
                                                         const int b_per) {
    static_assert(A::LOADERS == B::LOADERS, "");
    if ((int)blockIdx.x < a_all) A::run(a, blockIdx.x, a_per);
    else B::run(b, blockIdx.x - a_all, b_per);
}

template <class A, class B>
hipError_t ensure_pair() {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(nt_pair_kernel<A, B>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, pair_smem<A, B>);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    return hipSuccess;
}

// without parameters it only makes the kernel ready
template <class A, class B>
hipError_t launch(const GemmParams* a, const GemmParams* b, hipStream_t st) {
    hipError_t e = ensure_pair<A, B>();
    if (e != hipSuccess || a == nullptr) return e;
    const int a_per = A::grid(*a), b_per = B::grid(*b);
    const int a_all = a_per * (A::EPI == EPI_F32_SPLITK ? a->splits : 1), b_all = b_per * (B::EPI == EPI_F32_SPLITK ? b->splits : 1);
    hipLaunchKernelGGL((nt_pair_kernel<A, B>), dim3(a_all + b_all), dim3(pair_threads<A, B>), (pair_smem<A, B>), st, *a, *b, a_per, a_all, b_per);
    return hipGetLastError();
}

// dx on tile `ta`, the gradient on tile `tb` (fp32 slices, or, BF16, straight to its destination).  Waves of their own for the loads
// but beside 128x128 tiles that a unit has to share (`crowded`).
template <int EPI_B>
hipError_t dx_gradient(int ta, int tb, bool crowded, const GemmParams* a, const GemmParams* b, hipStream_t st) {
    using B64 = L64x64<EPI_B, true, true>;
    using B128 = L64x128<EPI_B, true, true>;
    const bool wide = tb == NT_64x128;
    if (ta == NT_64x64) return wide ? launch<L64x64<EPI_BF16, false, true>, B128>(a, b, st) : launch<L64x64<EPI_BF16, false, true>, B64>(a, b, st);
    if (ta == NT_64x128) return wide ? launch<L64x128<EPI_BF16, false, true>, B128>(a, b, st) : launch<L64x128<EPI_BF16, false, true>, B64>(a, b, st);
    if (!crowded) return wide ? launch<L128x128<EPI_BF16, false, true>, B128>(a, b, st) : launch<L128x128<EPI_BF16, false, true>, B64>(a, b, st);
    using A = T128x128<EPI_BF16, false, true>;
    return wide ? launch<A, T64x128<EPI_B, true, true>>(a, b, st) : launch<A, T64x64<EPI_B, true, true>>(a, b, st);
}

// Z (bf16 or fp32 slices, always 64x64 tiles) and the fold on tile `tb`
template <int EPI_A, int EPI_B, bool BRC>
hipError_t z_fold(int tb, const GemmParams* a, const GemmParams* b, hipStream_t st) {
    using A = T64x64<EPI_A, false, true>;
    if (tb == NT_64x128) return launch<A, Part<64, 128, EPI_B, false, BRC, 2>>(a, b, st);
    return launch<A, T128x128<EPI_B, false, BRC>>(a, b, st);
}
template <int EPI_A>
hipError_t z_fold_kind(int epi, bool b_rc, int tb, const GemmParams* a, const GemmParams* b, hipStream_t st) {
    if (epi == EPI_ACC_BF16) return b_rc ? z_fold<EPI_A, EPI_ACC_BF16, true>(tb, a, b, st) : hipErrorInvalidValue;
    return b_rc ? z_fold<EPI_A, EPI_FOLD, true>(tb, a, b, st) : z_fold<EPI_A, EPI_FOLD, false>(tb, a, b, st);
}

// Bf16 copies of two NF4 matrices beside U = s x B^T, which does not need them.  A work-group of the copy takes eight codes per
// thread and four such pieces at a time: the product's LDS leaves only two of them on a compute unit.
struct CopyPair {
    DequantGroupItem it[2];
    int blocks[2];
};
constexpr int COPY_PIECES = 4;
// ... which costs a large weight more than the launch saves.  Forward calls, us, two launches / one: 1.6 million elements (300
// tokens) 19.4 / 14.8, 2.8 million 26.7 / 22.8, 6.4 million (500) 36.4 / 34.2, 9 million (300, 1000) 35.2 / 34.5 and 52.4 /
// 52.0, 16.8 million 53.3 / 53.4 and 77.6 / 75.2, 25 million 58.6 / 61.6 and 67.8 / 70.9, 45 million (500) 90.2 / 98.4.
constexpr int64_t COPY_BESIDE_MAX = 12000000;

template <class A>
__global__ __launch_bounds__(256, 2) void nt_copy_kernel(const GemmParams a, const CopyPair c, const int a_per, const int a_all) {
    if ((int)blockIdx.x < a_all) {
        // Nothing is on its way here.  The compiler orders the branches one behind the other and else takes it that loads of the
        // copy could be, and waits for all loads in every k-tile (U beside copies, 768 x 896 x 3136, 16.6 us without, 24.0 with).
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
        A::run(a, blockIdx.x, a_per);
        return;
    }
    __shared__ float lut[16];
    if (threadIdx.x < 16) lut[threadIdx.x] = kNf4Levels[threadIdx.x];
    __syncthreads();
    const int b = (int)blockIdx.x - a_all, k = b >= c.blocks[0] ? 1 : 0;  // wave-uniform
    const DequantGroupItem& it = c.it[k];
    const int gpr = (it.cols + 7) >> 3;
    const int64_t groups = it.rows * gpr, first = (int64_t)(k ? b - c.blocks[0] : b) * (256 * COPY_PIECES) + threadIdx.x;
    uint32_t word[COPY_PIECES];
    float m[COPY_PIECES];
    int64_t row[COPY_PIECES];
    int j0[COPY_PIECES];
#pragma unroll
    for (int i = 0; i < COPY_PIECES; ++i) {
        const int64_t g = min(first + i * 256, groups - 1);  // (past the end: the last one again, not stored)
        row[i] = g / gpr;
        j0[i] = (int)(g - row[i] * gpr) * 8;
        word[i] = *reinterpret_cast<const uint32_t*>(it.codes + row[i] * (it.ld_q >> 1) + (j0[i] >> 1));
        m[i] = it.absmax[row[i] * (it.ld_q >> 6) + (j0[i] >> 6)];
    }
#pragma unroll
    for (int i = 0; i < COPY_PIECES; ++i) {
        if (first + i * 256 >= groups) break;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = m[i] * lut[(word[i] >> (8 * (e >> 1) + ((e & 1) ? 0 : 4))) & 15u];
        uint16_t* dst = it.out + row[i] * it.ld_out + j0[i];
        if (j0[i] + 8 <= it.cols) {
            *reinterpret_cast<uint4*>(dst) = make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
        } else {
            store_bf16_tail(dst, v, it.cols - j0[i]);
        }
    }
}

template <class A>
hipError_t launch_copy(const GemmParams* a, const DequantGroupItem* items, hipStream_t st) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(nt_copy_kernel<A>), hipFuncAttributeMaxDynamicSharedMemorySize, A::SMEM);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    if (a == nullptr) return hipSuccess;
    CopyPair c;
    int64_t blocks = 0;
    for (int i = 0; i < 2; ++i) {
        c.it[i] = items[i];
        c.blocks[i] = (int)((items[i].rows * ((items[i].cols + 7) / 8) + 256 * COPY_PIECES - 1) / (256 * COPY_PIECES));
        blocks += c.blocks[i];
    }
    const int per = A::grid(*a), all = per * (A::EPI == EPI_F32_SPLITK ? a->splits : 1);
    hipLaunchKernelGGL((nt_copy_kernel<A>), dim3((unsigned)(all + blocks)), dim3(256), A::SMEM, st, *a, c, per, all);
    return hipGetLastError();
}

bool small_tile(int t) { return t == NT_64x64 || t == NT_64x128 || t == NT_128x128; }

}  // namespace

hipError_t launch_dx_gradient(int slot_dx, const GemmParams& dx, int slot, int epi, const GemmParams& g, hipStream_t st) {
    const NtPlan plan = product_plan(dx);
    const int tb = gradient_tile(epi, g);
    if (small_tile(plan.tile) && plan.splits == 1 && (tb == NT_64x64 || tb == NT_64x128)) {
        TimedLaunch tl(slot_dx, st);
        // 128x128 tiles with waves of their own for the loads have a unit to themselves, and so has every work-group of the gradient
        // then: only where all of both find one (4096 x 768 x 2048 with a gradient of 256 x 768 x 4096 in 240 work-groups 25.7 us in twos,
        // 29 one by one).
        const int gw = tb == NT_64x64 ? 64 : 128;
        const int64_t gradient = (int64_t)((g.M + 63) / 64) * ((g.N + gw - 1) / gw), dxs = (int64_t)((dx.M + 127) / 128) * ((dx.N + 127) / 128);
        const bool crowded = (dxs + 7) / 8 + (gradient + 7) / 8 * (epi == EPI_F32_SPLITK ? g.splits : 1) > 32;
        return epi == EPI_BF16 ? dx_gradient<EPI_BF16>(plan.tile, tb, crowded, &dx, &g, st) : dx_gradient<EPI_F32_SPLITK>(plan.tile, tb, crowded, &dx, &g, st);
    }
    hipError_t e = launch_gemm_nt(slot_dx, EPI_BF16, false, true, dx, st, &plan);
    if (e != hipSuccess) return e;
    const NtPlan gradient{tb, g.splits, 0.0};
    return launch_gemm_nt(slot, epi, true, true, g, st, &gradient);
}

hipError_t launch_z_fold(int slot_z, const GemmParams& z, int slot, int epi, bool b_rc, const GemmParams& fold, hipStream_t st) {
    const NtPlan plan = product_plan(z);
    // (a fold that is ahead on 256x256 tiles by a few per cent only still shares: it has to fill the chip with them, at some rank)
    const int64_t t256 = ((fold.M + 255) / 256) * (int64_t)((fold.N + 255) / 256);
    const bool alone = weight_tile(epi, b_rc, fold) == NT_256x256 && t256 >= 216 && t256 <= 256 && fold.A[0].K > (epi == EPI_FOLD ? 128 : 512);
    if (plan.tile == NT_64x64 && !alone && (g_nt_tile_override == 0 || small_tile(weight_tile(epi, b_rc, fold)))) {
        // (a compute unit holds two of either here: 64x128 as long as 128x128 leave units idle)
        const int tb = ((fold.M + 127) / 128) * (int64_t)((fold.N + 127) / 128) <= 192 ? NT_64x128 : NT_128x128;
        TimedLaunch tl(slot, st);
        if (plan.splits == 1) return z_fold_kind<EPI_BF16>(epi, b_rc, tb, &z, &fold, st);
        const GemmParams c = product_slices(z, plan.splits);
        hipError_t e = z_fold_kind<EPI_F32_SPLITK>(epi, b_rc, tb, &c, &fold, st);
        if (e != hipSuccess) return e;
        return launch_reduce_db(z.split_ws, c.splits, z.M, z.N, c.ldc, z.C, LOQT_BF16, z.ldc, 0, st, false);
    }
    hipError_t e = launch_gemm_nt(slot_z, EPI_BF16, false, true, z, st, &plan);
    if (e != hipSuccess) return e;
    return launch_gemm_nt(slot, epi, false, b_rc, fold, st);
}

hipError_t launch_u_copies(int slot, const GemmParams& u, const DequantGroupItem* items, hipStream_t st) {
    const NtPlan plan = product_plan(u);
    if (plan.tile == NT_64x64 && items[0].rows * items[0].cols <= COPY_BESIDE_MAX) {
        TimedLaunch tl(slot, st);
        if (plan.splits == 1) return launch_copy<T64x64<EPI_BF16, false, false>>(&u, items, st);
        const GemmParams c = product_slices(u, plan.splits);
        hipError_t e = launch_copy<T64x64<EPI_F32_SPLITK, false, false>>(&c, items, st);
        if (e != hipSuccess) return e;
        return launch_reduce_db(u.split_ws, c.splits, u.M, u.N, c.ldc, u.C, LOQT_BF16, u.ldc, 0, st, false);
    }
    hipError_t e = launch_dequantize_grouped(items, 2, st, SLOT_PREPASS);
    if (e != hipSuccess) return e;
    return launch_gemm_nt(slot, EPI_BF16, false, false, u, st, &plan);
}

hipError_t prepare_pair_kernels() {
    hipError_t e;
    if ((e = launch_copy<T64x64<EPI_BF16, false, false>>(nullptr, nullptr, nullptr)) != hipSuccess) return e;
    if ((e = launch_copy<T64x64<EPI_F32_SPLITK, false, false>>(nullptr, nullptr, nullptr)) != hipSuccess) return e;
    for (int ta : {NT_64x64, NT_64x128, NT_128x128})
        for (int tb : {NT_64x64, NT_64x128}) {
            for (bool crowded : {false, true}) {
                if ((e = dx_gradient<EPI_BF16>(ta, tb, crowded, nullptr, nullptr, nullptr)) != hipSuccess) return e;
                if ((e = dx_gradient<EPI_F32_SPLITK>(ta, tb, crowded, nullptr, nullptr, nullptr)) != hipSuccess) return e;
            }
        }
    for (int tb : {NT_64x128, NT_128x128})
        for (int k = 0; k < 3; ++k) {
            const int epi = k == 2 ? EPI_ACC_BF16 : EPI_FOLD;
            if ((e = z_fold_kind<EPI_BF16>(epi, k != 1, tb, nullptr, nullptr, nullptr)) != hipSuccess) return e;
            if ((e = z_fold_kind<EPI_F32_SPLITK>(epi, k != 1, tb, nullptr, nullptr, nullptr)) != hipSuccess) return e;
        }
    return hipSuccess;
}

}  // namespace loqt
