// 128x128-tile instances of the mid-size MFMA GEMM: two workgroups per CU (64 KB of LDS in four stages; a split A, with two
// planes, 72 KB in three).
#include "gemm_mid.hpp"

namespace lithos {

template <bool KSA, bool KSB>
static gemm_fn plain() { return (gemm_fn)gemm_mid_kernel<128, 128, 2, 2, 4, 2, KSA, KSB, false>; }
template <bool KSB>
static gemm_fn split_a() { return (gemm_fn)gemm_mid_kernel<128, 128, 2, 2, 3, 2, false, KSB, true>; }

gemm_fn gemm_mid128_fn(bool ta, bool tb, bool split)
{
    if (split) return tb ? split_a<false>() : split_a<true>();
    if (ta) return tb ? plain<true, false>() : plain<true, true>();
    return tb ? plain<false, false>() : plain<false, true>();
}

} // namespace lithos
