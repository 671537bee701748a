// Slice products in passes: 13 ... 14 slices (a file for a few counts, so that they compile side by side).
#include "gemm_passes_dev.h"

namespace oz {
OZ_DEFINE_GEMM_PASSES(13)
OZ_DEFINE_GEMM_PASSES(14)
}  // namespace oz
