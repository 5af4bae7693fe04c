// 256x256-tile instances of the direct-to-LDS MFMA GEMM, A given as [K,M].
#include "gemm_lds256.hpp"

namespace lithos {

gemm_fn gemm_lds256_ta_fn(bool tb) { return tb ? (gemm_fn)gemm_lds256_kernel<true, false> : (gemm_fn)gemm_lds256_kernel<true, true>; }

} // namespace lithos
