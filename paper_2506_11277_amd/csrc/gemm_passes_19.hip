// Slice products in passes: 19 ... 20 slices (a file for a few counts, so that they compile side by side).
#include "gemm_passes_dev.h"

namespace oz {
OZ_DEFINE_GEMM_PASSES(19)
OZ_DEFINE_GEMM_PASSES(20)
}  // namespace oz
