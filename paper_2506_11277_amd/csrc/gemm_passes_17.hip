// Slice products in passes: 17 ... 18 slices (a file for a few counts, so that they compile side by side).
#include "gemm_passes_dev.h"

namespace oz {
OZ_DEFINE_GEMM_PASSES(17)
OZ_DEFINE_GEMM_PASSES(18)
}  // namespace oz
