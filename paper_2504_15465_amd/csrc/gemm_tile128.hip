// 128x128-tile instances of the direct-to-LDS MFMA GEMM: two workgroups of four wavefronts per CU.  A plain
// k-tile is 64 deep in two stages (64 KB of LDS), a split one, with two planes of A, 32 deep in three (72 KB).
// 64-bit addresses and 64-deep k-tiles: gemm_plan says which of the 128 tiles they serve.
#include "gemm_lds.hpp"

namespace lithos {

template <bool TA, bool TB, bool ST>
static gemm_fn plain() { return (gemm_fn)gemm_lds_kernel<128, 128, 2, 2, 1, 64, 2, 2, TA, TB, false, ST>; }
template <bool TB, bool ST>
static gemm_fn split_a() { return (gemm_fn)gemm_lds_kernel<128, 128, 2, 2, 1, 32, 3, 2, false, TB, true, ST>; }

gemm_fn gemm_tile128_fn(bool ta, bool tb, bool split, bool st)
{
    if (split) return tb ? (st ? split_a<true, true>() : split_a<true, false>()) : (st ? split_a<false, true>() : split_a<false, false>());
    if (ta) return tb ? (st ? plain<true, true, true>() : plain<true, true, false>()) : (st ? plain<true, false, true>() : plain<true, false, false>());
    return tb ? (st ? plain<false, true, true>() : plain<false, true, false>()) : (st ? plain<false, false, true>() : plain<false, false, false>());
}

} // namespace lithos
