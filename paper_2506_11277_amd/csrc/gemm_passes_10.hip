// Slice products in passes: 10 ... 12 slices (a file for a few counts, so that they compile side by side).
#include "gemm_passes_dev.h"

namespace oz {
OZ_DEFINE_GEMM_PASSES(10)
OZ_DEFINE_GEMM_PASSES(11)
OZ_DEFINE_GEMM_PASSES(12)
}  // namespace oz
