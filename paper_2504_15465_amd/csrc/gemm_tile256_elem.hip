// 256x256-tile instances (8 wavefronts, 2x4) of the register-staged MFMA GEMM that store element by element.
#include "gemm_tile.hpp"

namespace lithos {

gemm_fn gemm_tile256_elem_fn(bool ta, bool tb) { return LITHOS_TILE_PICK(false); }

} // namespace lithos
