// Eight-wavefront 256x256 GEMM, instances with the wide epilogue (full tiles through LDS / 16 bytes per lane).
#include "gemm_lds256w8.hpp"

namespace lithos {

gemm_fn gemm_lds256w8_wide_fn(bool ta, bool tb) { return LITHOS_LDS256W8_PICK(true); }

} // namespace lithos
