// Two products that do not need each other as one launch: the gradient of the factor beside dx, and Z = s dy deq(P) (or
// V = s x deq(Q)) beside the fold of the weight.
//
// Below a few thousand tokens a product is one partly filled round of small tiles for 5 to 20 us, a launch costs 3 to 4 us of
// them (2.6 of host time, 1.4 between kernels, the first loads of every work-group on top), and the small products (a few
// dozen work-groups with long contractions) leave most of the chip idle.  One grid over the tiles of both: the first work-groups
// belong to the product with the longer tiles, the others follow it onto whatever compute unit is free.  Both keep the tile
// shape and slices they have alone, so the results are the same bits.  Only tiles of which a compute unit holds two take part;
// larger products run for hundreds of microseconds, and their tiles have a compute unit and its registers to themselves.
#include <string.h>

#include <algorithm>

#include "nt_tile.h"

namespace loqt {

namespace {

template <int BM_, int BN_, int EPI_, bool ARC_, bool BRC_, int NS_>
struct Part {
    static constexpr int BM = BM_, BN = BN_, EPI = EPI_, NS = NS_, SMEM = NtCfg<BM, BN, NS>::SMEM;
    static constexpr bool ARC = ARC_, BRC = BRC_;
    static_assert(NtCfg<BM, BN, NS>::PER_CU == 2, "");
    static int grid(const GemmParams& p) { return (((p.M + BM - 1) / BM) * ((p.N + BN - 1) / BN) + 7) / 8 * 8; }
    // `b`: work-group of this part; `per`: of them belong to a slice (a multiple of 8, so that b % 8 is the XCD)
    static __device__ __forceinline__ void run(const GemmParams& p, int b, int per) {
        const int split = EPI == EPI_F32_SPLITK ? b / per : 0, r = b - split * per;
        nt_gemm_tile<BM, BN, EPI, ARC, BRC, NS>(p, (r & 7) * (per >> 3) + (r >> 3), split);
    }
};
template <int EPI, bool ARC, bool BRC>
using T64x64 = Part<64, 64, EPI, ARC, BRC, 4>;
template <int EPI, bool ARC, bool BRC>
using T64x128 = Part<64, 128, EPI, ARC, BRC, 3>;
template <int EPI, bool ARC, bool BRC>
using T128x128 = Part<128, 128, EPI, ARC, BRC, 2>;

template <class A, class B>
constexpr int pair_smem = A::SMEM > B::SMEM ? A::SMEM : B::SMEM;

template <class A, class B>
__global__ __launch_bounds__(256, 2) void nt_pair_kernel(const GemmParams a, const GemmParams b, const int a_per, const int a_all,
                                                         const int b_per) {
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
    hipLaunchKernelGGL((nt_pair_kernel<A, B>), dim3(a_all + b_all), dim3(256), (pair_smem<A, B>), st, *a, *b, a_per, a_all, b_per);
    return hipGetLastError();
}

// dx on tile `ta`, the gradient on tile `tb` (fp32 slices, or, BF16, straight to its destination)
template <int EPI_B>
hipError_t dx_gradient(int ta, int tb, const GemmParams* a, const GemmParams* b, hipStream_t st) {
    using B64 = T64x64<EPI_B, true, true>;
    using B128 = T64x128<EPI_B, true, true>;
    const bool wide = tb == NT_64x128;
    if (ta == NT_64x64) return wide ? launch<T64x64<EPI_BF16, false, true>, B128>(a, b, st) : launch<T64x64<EPI_BF16, false, true>, B64>(a, b, st);
    if (ta == NT_64x128) return wide ? launch<T64x128<EPI_BF16, false, true>, B128>(a, b, st) : launch<T64x128<EPI_BF16, false, true>, B64>(a, b, st);
    return wide ? launch<T128x128<EPI_BF16, false, true>, B128>(a, b, st) : launch<T128x128<EPI_BF16, false, true>, B64>(a, b, st);
}

// Z (bf16 or fp32 slices, always 64x64 tiles) and the fold on tile `tb`
template <int EPI_A, int EPI_B, bool BRC>
hipError_t z_fold(int tb, const GemmParams* a, const GemmParams* b, hipStream_t st) {
    using A = T64x64<EPI_A, false, true>;
    if (tb == NT_64x128) return launch<A, T64x128<EPI_B, false, BRC>>(a, b, st);
    return launch<A, T128x128<EPI_B, false, BRC>>(a, b, st);
}
template <int EPI_A>
hipError_t z_fold_kind(int epi, bool b_rc, int tb, const GemmParams* a, const GemmParams* b, hipStream_t st) {
    if (epi == EPI_ACC_BF16) return b_rc ? z_fold<EPI_A, EPI_ACC_BF16, true>(tb, a, b, st) : hipErrorInvalidValue;
    return b_rc ? z_fold<EPI_A, EPI_FOLD, true>(tb, a, b, st) : z_fold<EPI_A, EPI_FOLD, false>(tb, a, b, st);
}

bool small_tile(int t) { return t == NT_64x64 || t == NT_64x128 || t == NT_128x128; }

}  // namespace

hipError_t launch_dx_gradient(int slot_dx, const GemmParams& dx, int slot, int epi, const GemmParams& g, hipStream_t st) {
    const NtPlan plan = product_plan(dx);
    const int tb = gradient_tile(epi, g);
    if (small_tile(plan.tile) && plan.splits == 1 && (tb == NT_64x64 || tb == NT_64x128)) {
        TimedLaunch tl(slot_dx, st);
        return epi == EPI_BF16 ? dx_gradient<EPI_BF16>(plan.tile, tb, &dx, &g, st) : dx_gradient<EPI_F32_SPLITK>(plan.tile, tb, &dx, &g, st);
    }
    hipError_t e = launch_gemm_nt(slot_dx, EPI_BF16, false, true, dx, st);
    if (e != hipSuccess) return e;
    return launch_gemm_nt(slot, epi, true, true, g, st);
}

hipError_t launch_z_fold(int slot_z, const GemmParams& z, int slot, int epi, bool b_rc, const GemmParams& fold, hipStream_t st) {
    const NtPlan plan = product_plan(z);
    const int tb = weight_tile(epi, fold);
    if (plan.tile == NT_64x64 && (tb == NT_64x128 || tb == NT_128x128)) {
        TimedLaunch tl(slot, st);
        if (plan.splits == 1) return z_fold_kind<EPI_BF16>(epi, b_rc, tb, &z, &fold, st);
        const GemmParams c = product_slices(z, plan.splits);
        hipError_t e = z_fold_kind<EPI_F32_SPLITK>(epi, b_rc, tb, &c, &fold, st);
        if (e != hipSuccess) return e;
        return launch_reduce_db(z.split_ws, c.splits, z.M, z.N, c.ldc, z.C, LOQT_BF16, z.ldc, 0, st, false);
    }
    hipError_t e = launch_gemm_nt(slot_z, EPI_BF16, false, true, z, st);
    if (e != hipSuccess) return e;
    return launch_gemm_nt(slot, epi, false, b_rc, fold, st);
}

hipError_t prepare_pair_kernels() {
    hipError_t e;
    for (int ta : {NT_64x64, NT_64x128, NT_128x128})
        for (int tb : {NT_64x64, NT_64x128}) {
            if ((e = dx_gradient<EPI_BF16>(ta, tb, nullptr, nullptr, nullptr)) != hipSuccess) return e;
            if ((e = dx_gradient<EPI_F32_SPLITK>(ta, tb, nullptr, nullptr, nullptr)) != hipSuccess) return e;
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
