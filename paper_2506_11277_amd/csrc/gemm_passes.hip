// Slice products in passes over groups of diagonals: which shape runs, and the launch (kernels: gemm_passes_dev.h, instantiated
// in gemm_passes_4.hip ... gemm_passes_19.hip; 32 x 32 tiles: gemm_small.hip).
#include "oz_common.h"

namespace oz {

#define OZ_DECLARE(S_)                                                                                                      \
    hipError_t launch_gemm_passes_##S_(bool small, int m, int n, int kp, int stride, const int8_t *pA, const int8_t *pB,    \
                                       const int32_t *eA, const int32_t *eB, double *C, int ldc, int Q, hipStream_t st);
OZ_DECLARE(4) OZ_DECLARE(5) OZ_DECLARE(6) OZ_DECLARE(7) OZ_DECLARE(8) OZ_DECLARE(9)
OZ_DECLARE(10) OZ_DECLARE(11) OZ_DECLARE(12) OZ_DECLARE(13) OZ_DECLARE(14) OZ_DECLARE(15) OZ_DECLARE(16) OZ_DECLARE(17)
OZ_DECLARE(18) OZ_DECLARE(19) OZ_DECLARE(20)
#undef OZ_DECLARE

// Which shape, if any (GEMM phases in us, s = 11 / 13 / 16 / 18).
// Up to one tile of 32 x 32 per compute unit, and up to 1.75 where the products repay a second round: these, k in eighths
// (402^3 before 25.7 / 33.9 / 44.7 / 62.8, now 16.1 / 18.8 / 23.0 / 26.0; 1.64 tiles: 600 x 700 x 384 21.8 / 28.0 / 36.1 / 49.1, 23.6 / 28.1 / 34.6 / 40.4,
// 600 x 700 x 188 17.6 / 21.8 / 27.1 / 36.5, 20.8 / 23.9 / 28.5 / 33.0; 800^3, 2.4 tiles, 40.6 / 54.8 / 75.1 / 102, 53.1 / 66.2 / 84.7 / 100;
// 10 slices have a kernel of one pass there).
// Then, up to one 64 x 64 tile per compute unit, the one-pass kernels on that tile with 512 registers to a wavefront up to 16
// slices (800^3: against 49.8 / 65.2 / 83.2 in passes; 18: 95.0).
// Up to 12 slices the fixed costs of two passes are only repaid by several rounds or a longer k (s = 11, one-pass kernel against
// passes: 1000 x 1100 x 500 39.7 / 46.3, 1038 x 2512 x 66 33.5 / 36.3, but 1300^3 119 / 114, 3000 x 3000 x 500 234 / 219).
// 128 x 64 or 64 x 64 by rounds of the chip: two 64 x 64 tiles at a time cost a compute unit 1.04 of a 128 x 64 one (pair_rounds);
// at short k the 128 x 64 tile also pays for copies and epilogues that nothing hides (2085 x 4740 x 1000, 4.98 against 4.83
// rounds, s = 13 580 / 584, 18 953 / 940; 3000 x 3000 x 500, 4.41 against 4.31, s = 13 306 / 280; 2207^3, 2.46 against 2.39, 693 / 627).
PassShape gemm_passes_shape(int s, int m, int n, int kp, int Q)
{
    if (s < 10 || s > 20 || m <= 0 || n <= 0) return kNoPasses;
    const int cus = device_cus();
    auto tiles = [&](int tm, int tn) { return (long long)((m + tm - 1) / tm) * ((n + tn - 1) / tn); };
    const long long tiny = tiles(32, 32);
    if (4 * tiny <= 7LL * cus && s == 10) return kNoPasses;
    if (tiny <= cus || (4 * tiny <= 7LL * cus && (s >= 17 ? kp >= 256 : s * kp >= 6144))) return kPassEighths;
    const PassPlan P = pass_plan(s);
    for (int p = 0, d = 0; p + 1 < P.n; ++p)
        if ((d += P.w[p]) % Q != 0) return kNoPasses;                // a level of Q diagonals straddles two passes
    const long long small = tiles(64, 64), wide = tiles(128, 64);
    if (small <= cus) return s <= 16 ? kNoPasses : kPassSmall;
    if (s <= 12 && !(kp >= 1024 || (kp >= 384 && wide > cus))) return kNoPasses;
    const double rounds = (double)wide / cus, whole = (double)((wide + cus - 1) / cus);
    return 1.04 * pair_rounds(small, cus) < (0.8 * whole + 0.2 * rounds) * (1.0 + 40.0 / kp) ? kPassSmall : kPassWide;
}

hipError_t launch_gemm_passes(PassShape shape, int s, int m, int n, int kp, int stride, const int8_t *pA, const int8_t *pB,
                              const int32_t *eA, const int32_t *eB, double *C, int ldc, int Q, hipStream_t st)
{
    if (m <= 0 || n <= 0) return hipSuccess;
    if (shape == kNoPasses || stride < s) return hipErrorInvalidValue;
    if (shape == kPassEighths) return launch_gemm_eighths_passes(s, m, n, kp, stride, pA, pB, eA, eB, C, ldc, Q, st);
    const bool small = shape == kPassSmall;
    switch (s) {
#define OZ_CASE(S_) case S_: return launch_gemm_passes_##S_(small, m, n, kp, stride, pA, pB, eA, eB, C, ldc, Q, st);
        OZ_CASE(4) OZ_CASE(5) OZ_CASE(6) OZ_CASE(7) OZ_CASE(8) OZ_CASE(9)
        OZ_CASE(10) OZ_CASE(11) OZ_CASE(12) OZ_CASE(13) OZ_CASE(14) OZ_CASE(15) OZ_CASE(16) OZ_CASE(17) OZ_CASE(18) OZ_CASE(19)
        OZ_CASE(20)
#undef OZ_CASE
    }
    return hipErrorInvalidValue;
}

}  // namespace oz
