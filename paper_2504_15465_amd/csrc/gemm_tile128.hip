// 128x128-tile instances of the mid-size MFMA GEMM: two workgroups per CU (64 KB of LDS in four stages; a split A, with two
// planes, 72 KB in three).  Beside them the 64-deep form of gemm_lds_kernel.
#include "gemm_lds.hpp"
#include "gemm_mid.hpp"

namespace lithos {

template <bool KSA, bool KSB>
static gemm_fn plain() { return (gemm_fn)gemm_mid_kernel<128, 128, 2, 2, 4, 2, KSA, KSB, false>; }
template <bool KSB>
static gemm_fn split_a() { return (gemm_fn)gemm_mid_kernel<128, 128, 2, 2, 3, 2, false, KSB, true>; }

// The 64-deep k-tiles of gemm_lds_kernel (two stages) read whole lines of k-contiguous operands, the 32-deep ones half lines: see gemm_plan.
gemm_fn gemm_tile128_deep_fn(bool st)
{
    return st ? (gemm_fn)gemm_lds_kernel<128, 128, 2, 2, 1, 64, 2, 2, false, true, false, true> : (gemm_fn)gemm_lds_kernel<128, 128, 2, 2, 1, 64, 2, 2, false, true, false, false>;
}

gemm_fn gemm_tile128_fn(bool ta, bool tb, bool split)
{
    if (split) return tb ? split_a<false>() : split_a<true>();
    if (ta) return tb ? plain<true, false>() : plain<true, true>();
    return tb ? plain<false, false>() : plain<false, true>();
}

} // namespace lithos
