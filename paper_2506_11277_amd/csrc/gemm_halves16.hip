// 64 x 64 tiles, one to a compute unit, the contraction in halves, on the 16x16x64 instruction: two groups of four
// wavefronts take the even and the odd 64-deep k-steps of the tile, each with a ring of LDS slots of its own (gemm_passes_dev.h,
// one pass), and hand each other half of their int32 sums through LDS at the end.
//
// Against the 32x32x32 form of gemm_small.hip: operands are read from LDS once per slice by each wavefront in both, but the
// instruction costs less energy per product and the ring runs further ahead.  GEMM, us, s = 7 / 8 / 9: 1024 x 1024 x 4096 96.0 / 118 /
// 144 -> 84.2 / 105 / 125, 1024^3 31.0 / 36.7 / 43.3 -> 28.3 / 34.1 / 39.4, 800 x 800 x 3000 57.9 / 68.8 / 83.0 -> 52.9 / 66.6 / 79.1, 1024 x 1024 x 128
// 12.5 / 13.2 / 14.4 -> 12.3 / 13.0 / 13.8.  4 ... 6 slices are ahead in the 32x32x32 form except at very long k (800 x 800 x 1000 s = 4 / 6 14.1 /
// 20.8 against 16.0 / 23.1), 2 and 3 from k = 1000 on behind it (1024 x 1024 x 4096 24.2 / 31.7 -> 21.4 / 28.4, 1024^3 11.9 / 13.7 -> 11.5 / 13.4).
// What bounds it at 1024^3: 10 us of launch, first copies, exchange and epilogue around a loop of 3.2 POP/s.
#include "gemm_passes_dev.h"

namespace oz {

namespace {

using PassTileHalves = PassTile<2, 2, 10, 2>;       // 160 KiB

template <int S>
__global__ __launch_bounds__(PassTileHalves::THREADS, 2) void gemm_halves16_kernel(
    const int8_t *__restrict__ pA, const int8_t *__restrict__ pB, const int32_t *__restrict__ eA,
    const int32_t *__restrict__ eB, double *__restrict__ C, int ldc, int m, int n, int KB, int tiles_m, int tiles_n, int Q)
{
    passes_of_a_tile<PassTileHalves, S>(pA, pB, eA, eB, C, ldc, m, n, KB, S, tiles_m, tiles_n, Q);
}

template <int S>
hipError_t launch_halves16(int m, int n, int kp, const int8_t *pA, const int8_t *pB, const int32_t *eA, const int32_t *eB,
                           double *C, int ldc, int Q, hipStream_t st)
{
    auto kern = gemm_halves16_kernel<S>;
    static std::atomic<unsigned long long> configured{0};
    if (hipError_t e = allow_dynamic_lds((const void *)kern, PassTileHalves::LDS, configured); e != hipSuccess) return e;
    const int tiles_m = (m + 63) / 64, tiles_n = (n + 63) / 64;
    note_gemm_kernel("gemm_halves16_kernel<%d> tile 64x64, 8 wavefronts, k in halves", S);
    kern<<<(unsigned)tile_order_blocks(tiles_m, tiles_n, false), PassTileHalves::THREADS, PassTileHalves::LDS, st>>>(
        pA, pB, eA, eB, C, ldc, m, n, kp / kFrag, tiles_m, tiles_n, Q);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_halves16(int s, int m, int n, int kp, const int8_t *pA, const int8_t *pB, const int32_t *eA,
                                const int32_t *eB, double *C, int ldc, int Q, hipStream_t st)
{
    if (m <= 0 || n <= 0) return hipSuccess;
    switch (s) {
#define OZ_CASE(S_) case S_: return launch_halves16<S_>(m, n, kp, pA, pB, eA, eB, C, ldc, Q, st);
        OZ_CASE(2) OZ_CASE(3) OZ_CASE(7) OZ_CASE(8) OZ_CASE(9)
#undef OZ_CASE
    }
    return hipErrorInvalidValue;
}

}  // namespace oz
