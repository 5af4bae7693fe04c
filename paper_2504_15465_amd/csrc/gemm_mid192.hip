// 64x192-tile instances of the mid-size MFMA GEMM for a split A: two workgroups per CU (60 KB of LDS in three stages).
#include "gemm_mid.hpp"

namespace lithos {

gemm_fn gemm_mid192_fn(bool tb)
{
    return tb ? (gemm_fn)gemm_mid_kernel<64, 192, 3, false, false, true> : (gemm_fn)gemm_mid_kernel<64, 192, 3, false, true, true>;
}

} // namespace lithos
