// 256x256-tile instances of the direct-to-LDS MFMA GEMM, A given as [M,K].
#include "gemm_lds256.hpp"

namespace lithos {

gemm_fn gemm_lds256_fn(bool tb) { return tb ? (gemm_fn)gemm_lds256_kernel<false, false> : (gemm_fn)gemm_lds256_kernel<false, true>; }

} // namespace lithos
