// Slices streamed through a ring, one pass, 64 x 64 tiles and runs of 128 x 64: 4 ... 9 slices.
#include "gemm_passes_dev.h"

namespace oz {
OZ_DEFINE_GEMM_PASSES(4)
OZ_DEFINE_GEMM_PASSES(5)
OZ_DEFINE_GEMM_PASSES(6)
OZ_DEFINE_GEMM_PASSES(7)
OZ_DEFINE_GEMM_PASSES(8)
OZ_DEFINE_GEMM_PASSES(9)
}  // namespace oz
