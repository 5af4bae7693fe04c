// 128x128-tile instances of the mid-size MFMA GEMM: two workgroups per CU (64 KB of LDS in four stages; a split A, with two
// planes, 72 KB in three; 80 KB in the five stages of k-tiles that are fetched in pairs).
#include "gemm_mid.hpp"

namespace lithos {

template <int S, bool KSA, bool KSB>
static gemm_fn plain() { return (gemm_fn)gemm_mid_kernel<128, 128, S, KSA, KSB, false>; }
template <bool KSB>
static gemm_fn split_a() { return (gemm_fn)gemm_mid_kernel<128, 128, 3, false, KSB, true>; }

gemm_fn gemm_mid128_fn(bool ta, bool tb, bool split)
{
    if (split) return tb ? split_a<false>() : split_a<true>();
    if (ta) return tb ? plain<4, true, false>() : plain<4, true, true>();
    return tb ? plain<4, false, false>() : plain<4, false, true>();
}

gemm_fn gemm_mid128_pair_fn(bool ta, bool tb) { return !tb ? plain<5, false, true>() : ta ? plain<5, true, false>() : plain<5, false, false>(); }

} // namespace lithos
