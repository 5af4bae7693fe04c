// 64x64-tile instances of the direct-to-LDS MFMA GEMM: two groups of four wavefronts halve the chain of k-tiles;
// two workgroups per CU (64 KB of LDS, 72 KB with the two planes of a split A).
#include "gemm_lds.hpp"

namespace lithos {

template <bool TA, bool TB, bool ST>
static gemm_fn plain() { return (gemm_fn)gemm_lds_kernel<64, 64, 2, 2, 2, 64, 2, 4, TA, TB, false, ST>; }
template <bool TB, bool ST>
static gemm_fn split_a() { return (gemm_fn)gemm_lds_kernel<64, 64, 2, 2, 2, 32, 3, 4, false, TB, true, ST>; }

gemm_fn gemm_tile64_fn(bool ta, bool tb, bool split, bool st)
{
    if (split) return tb ? (st ? split_a<true, true>() : split_a<true, false>()) : (st ? split_a<false, true>() : split_a<false, false>());
    if (ta) return tb ? (st ? plain<true, true, true>() : plain<true, true, false>()) : (st ? plain<true, false, true>() : plain<true, false, false>());
    return tb ? (st ? plain<false, true, true>() : plain<false, true, false>()) : (st ? plain<false, false, true>() : plain<false, false, false>());
}

} // namespace lithos
