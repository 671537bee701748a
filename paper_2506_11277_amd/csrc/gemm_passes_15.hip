// Slice products in passes: 15 ... 16 slices (a file for a few counts, so that they compile side by side).
#include "gemm_passes_dev.h"

namespace oz {
OZ_DEFINE_GEMM_PASSES(15)
OZ_DEFINE_GEMM_PASSES(16)
}  // namespace oz
