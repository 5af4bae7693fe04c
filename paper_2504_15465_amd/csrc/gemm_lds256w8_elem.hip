// Eight-wavefront 256x256 GEMM, instances with the element-wise epilogue.
#include "gemm_lds256w8.hpp"

namespace lithos {

gemm_fn gemm_lds256w8_elem_fn(bool ta, bool tb) { return LITHOS_LDS256W8_PICK(false); }

} // namespace lithos
