// 64x64-tile instances of the direct-to-LDS MFMA GEMM.  With two groups of four wavefronts, which halve the chain of
// k-tiles, two workgroups run per CU (64 KB of LDS, 72 KB with the two planes of a split A).  With one group five do
// (32 KB; a split A three, with 48 KB): no second group that waits in the epilogue, and a chain hidden by the other
// workgroups.  gemm_plan says which.
#include "gemm_lds.hpp"

namespace lithos {

template <int KG, bool TA, bool TB, bool ST>
static gemm_fn plain() { return (gemm_fn)gemm_lds_kernel<64, 64, 2, 2, KG, 64, 2, 4, TA, TB, false, ST>; }
template <int KG, bool TB, bool ST>
static gemm_fn split_a()
{
    if constexpr (KG == 2) return (gemm_fn)gemm_lds_kernel<64, 64, 2, 2, 2, 32, 3, 4, false, TB, true, ST>;
    else return (gemm_fn)gemm_lds_kernel<64, 64, 2, 2, 1, 64, 2, 3, false, TB, true, ST>;
}

template <int KG>
static gemm_fn pick(bool ta, bool tb, bool split, bool st)
{
    if (split) return tb ? (st ? split_a<KG, true, true>() : split_a<KG, true, false>()) : (st ? split_a<KG, false, true>() : split_a<KG, false, false>());
    if (ta) return tb ? (st ? plain<KG, true, true, true>() : plain<KG, true, true, false>()) : (st ? plain<KG, true, false, true>() : plain<KG, true, false, false>());
    return tb ? (st ? plain<KG, false, true, true>() : plain<KG, false, true, false>()) : (st ? plain<KG, false, false, true>() : plain<KG, false, false, false>());
}

gemm_fn gemm_tile64_fn(bool ta, bool tb, bool split, bool st, bool two_groups)
{
    return two_groups ? pick<2>(ta, tb, split, st) : pick<1>(ta, tb, split, st);
}

} // namespace lithos
