// Slice products in passes over groups of diagonals: which shape runs, and the launch (kernels: gemm_passes_dev.h, instantiated
// in gemm_passes_4.hip ... gemm_passes_19.hip; 32 x 32 tiles: gemm_small.hip).
#include "gemm_dev.h"

namespace oz {

#define OZ_DECLARE(S_)                                                                                                      \
    hipError_t launch_gemm_passes_##S_(PassShape shape, int m, int n, int kp, int stride, const int8_t *pA, const int8_t *pB, \
                                       const int32_t *eA, const int32_t *eB, double *C, int ldc, int Q, hipStream_t st);
OZ_DECLARE(4) OZ_DECLARE(5) OZ_DECLARE(6) OZ_DECLARE(7) OZ_DECLARE(8) OZ_DECLARE(9)
OZ_DECLARE(10) OZ_DECLARE(11) OZ_DECLARE(12) OZ_DECLARE(13) OZ_DECLARE(14) OZ_DECLARE(15) OZ_DECLARE(16) OZ_DECLARE(17)
OZ_DECLARE(18) OZ_DECLARE(19) OZ_DECLARE(20)
#undef OZ_DECLARE

// ---- Time of a launch, us: rounds * (product * x + round) + once ----
// x: slice products per entry times kp, in thousands.  `round` is what a round adds whatever its length (first copies, epilogue, the
// sums parked between passes), `once` what a launch adds.  Fitted to the GEMM phases of 1800 random calls of 4 ... 9 slices and 680 of
// 10 ... 12, up to 4 ms, k > 128; the fits leave 3 ... 6 percent.  Where the epilogues of one work-group run beside the products of another
// (64 x 64 tiles in pairs, runs of 128 x 64 tiles), a round adds 0.7 ... 2.7 us instead of 4 ... 5, but the last of them hides behind nothing:
// `once` is 6 ... 7 us instead of 4.5.  So a launch of a single round gains nothing by them.
struct LaunchTime {
    double product, round, once;
    double us(double rounds, double x) const { return rounds * (product * x + round) + once; }
};

// Rounds count the work-groups of the XCD that gets most: a grid in the two-dimensional order has up to 4 % more of them than tiles,
// and an XCD with one tile too many needs a round more (3200 x 613 x 1152, s = 9: 500 tiles of 64 x 64, 65 of them on two XCDs
// with room for 64: 85 us instead of 62 in 128 x 64 tiles).
static long long order_blocks(int m, int n, int tm, int tn) { return tile_order_blocks((m + tm - 1) / tm, (n + tn - 1) / tn, false); }

// One work-group to a compute unit: a partly filled last round counts 0.7 of a full one plus 0.3 of its share (0.8 and 0.2 from 10 slices on,
// where passes and fuller registers leave less to the power cap).
static double single_rounds(int s, long long blocks, int cus)
{
    const double share = s > 9 ? 0.2 : 0.3;
    return (1.0 - share) * (double)((blocks + cus - 1) / cus) + share * (double)blocks / cus;
}

// 64 x 64 tiles, two work-groups to a compute unit, in units of the time two of them take together: one alone takes 0.65 of it;
// behind whole rounds work-groups start as others end, and the last ones count about half a unit, or most of one where some
// compute units get two of them (s = 7: 1500^3, 576 tiles, 1.53; 2304 x 2000 x 2560, 1152 tiles, 2.48; 3328 x 1562 x 817,
// 1300 tiles, 2.95; s = 9: 4455 x 700 x 2660, 770 tiles, 1.99); more with few slices, whose compute units are furthest from the power cap
// (s = 4: 1592^3, 640 work-groups: 48 us, 45 in 128 x 128 tiles).
static double pair_rounds(int s, long long blocks, int cus)
{
    const long long whole = blocks / (2 * cus), rest = blocks % (2 * cus);
    const double part = (double)rest / (2 * cus);
    if (rest == 0) return (double)whole;
    if (s > 9) return whole == 0 ? (rest <= cus ? 0.65 : 1.0) : whole + (rest <= cus ? 0.5 : part < 0.95 ? 0.95 : part);
    if (rest > cus) return whole + 0.7 + 0.3 * part;
    return whole == 0 ? 0.65 : whole + (s == 4 ? 0.6 : s <= 6 ? 0.45 : 0.35) + 0.2 * part;
}

// 96 x 64 tiles: one round of them where 64 x 64 tiles are more than the compute units, so that the other shapes leave a quarter of the chip, or of a second
// round, empty.  A round takes 0.78 of one of 128 x 64 tiles.  Calls, us, best of the others and this, s = 4 ... 9, 13 ... 18: 940 x 1398 x 156 s = 4 13.7 / 13.4 (even with
// the others at kp = 256), 545 x 1984 x 3279 s = 4 65.9 / 60.9, 873 x 1163 x 927 s = 5 29.2 / 25.3, 2240 x 568 x 294 s = 6 19.0 / 17.0, 5312 x 212 x 136 s = 7 17.5 / 15.9, 1531 x 777 x 1001
// s = 8 53.3 / 46.4, 370 x 2691 x 1378 s = 16 212 / 170, 686 x 1920 x 3766 s = 18 693 / 567; over 82 such sizes 1.05 (4 ... 6), 1.11 (7 ... 9) and 1.23 (13 ... 18) in the mean,
// slowest 0.997 (0.985 at kp = 256, s = 4).  k up to 128: 40 sizes of 13 ... 18 slices 1.17 in the mean, slowest 1.06 (1168 x 994 x 30 s = 17 34.1 / 28.6), 40 of 4 ... 9 1.17, slowest 1.05 (364 x 3520 x 27 s = 8 16.8 / 16.0).
// With more rounds, 13 ... 18 slices: even with the others at best.  10 ... 12, 19 and 20 run in passes of which the first, three diagonals, is too short for this tile's
// copies.  (256 tiles, and s kp of what one int32 block holds, keep the planes below 2^32 bytes, the offsets that this tile takes.)
static bool one_round_of_96(int s, int m, int n)
{
    const int cus = device_cus();
    const long long blocks = order_blocks(m, n, 96, 64), small = (long long)((m + 63) / 64) * ((n + 63) / 64);
    return (s <= 9 || (s >= 13 && s <= 18)) && blocks <= cus && small > cus;
}

// 4 ... 9 slices: the other kernels by their tile (128 x 64 outputs count one round, larger tiles as many more).  What is taken where the
// figures are even is what stood there before up to 6 slices, whose fits are the looser ones.  Calls, operands that change from one to
// the next, against the other kernels alone and against the best of the three: geometric means over 900 random sizes 1.085 and 0.997, slowest
// 0.92 (5440 x 384 x 1216, s = 4; else 0.975).
PassShape gemm_one_pass_shape(int s, int m, int n, int kp, int tm, int tn)
{
    if (s < 4 || s > 9 || m <= 0 || n <= 0) return kNoPasses;
    static constexpr LaunchTime kPairs[6] = {{1.454, 2.7, 5.1}, {1.389, 2.1, 5.8}, {1.368, 1.65, 6.0}, {1.284, 1.35, 5.95}, {1.242, 1.2, 6.3}, {1.203, 0.85, 6.85}};
    static constexpr LaunchTime kRuns[6] = {{1.344, 2.0, 6.3}, {1.363, 1.7, 6.0}, {1.272, 1.7, 6.1}, {1.245, 1.8, 6.1}, {1.169, 2.3, 5.7}, {1.136, 2.25, 6.15}};
    static constexpr LaunchTime k64[6] = {{1.844, 3.0, 5.4}, {1.62, 4.9, 4.0}, {1.64, 3.7, 6.0}, {1.484, 2.25, 7.3}, {1.57, 7.2, 4.6}, {1.417, 6.8, 4.5}};
    static constexpr LaunchTime k128x64[6] = {{1.4, 4.5, 4.9}, {1.387, 4.5, 4.9}, {1.241, 4.8, 4.7}, {1.193, 4.75, 4.5}, {1.153, 5.75, 4.05}, {1.126, 5.4, 4.5}};
    static constexpr LaunchTime k128x128[3] = {{1.226, 3.85, 5.85}, {1.147, 4.6, 4.35}, {1.109, 4.05, 5.95}}, k192x128{1.188, 3.95, 4.65};
    static constexpr double kAhead[6] = {0.98, 0.985, 0.99, 1.0, 1.0, 1.0};
    if (one_round_of_96(s, m, n)) return kPassMiddle;
    if (kp <= 128) return kNoPasses;                                 // (the fits are of longer contractions)
    const int cus = device_cus();
    const double x = 1e-3 * kp * (s * (s + 1) / 2);
    const double pairs = kPairs[s - 4].us(pair_rounds(s, order_blocks(m, n, 64, 64), cus), x);
    const double runs = kRuns[s - 4].us(single_rounds(s, order_blocks(m, n, 128, 64), cus), x);
    const LaunchTime &t = tm == 64 ? k64[s - 4] : tm == 192 ? k192x128 : tn == 64 || s > 6 ? k128x64[s - 4] : k128x128[s - 4];
    const double others = t.us(single_rounds(s, order_blocks(m, n, tm, tn), cus) * (tm * tn / 8192.0), x);
    // several rounds of 96 x 64 tiles, 7 ... 9 slices (its round is not scaled by the area).  Per product 0.92 ... 0.97 of a work-group's rate in 128 x 64 tiles away from the power cap,
    // so it pays where its rounds fit better: calls 2304 x 2000 x 2560, s = 7, three whole rounds, 281 -> 268.  260 random
    // sizes of more than 256 tiles of 64 x 64: taken by 67 of them, 11.7 percent faster there, none slower; with 1.0 for 0.98 by 78, the slowest 2 percent behind.
    // (kp > 256: shorter ones gain little, 1600 x 1536 x 230, s = 9 31.5 / 32.4; 32-bit offsets into the planes)
    if (s >= 7 && kp > 256 && (long long)(m > n ? round_up(m, kPad) : round_up(n, kPad)) * kp * s < (1LL << 32)) {
        static constexpr LaunchTime kMiddle[3] = {{0.935, 1.64, 6.15}, {0.896, 1.85, 6.3}, {0.898, 1.75, 6.5}};
        const double middle = kMiddle[s - 7].us(single_rounds(s, order_blocks(m, n, 96, 64), cus), x), rest = pairs < runs ? pairs : runs;
        if (middle < 0.98 * (rest < others ? rest : others)) return kPassMiddle;
    }
    if ((pairs < runs ? pairs : runs) >= kAhead[s - 4] * others) return kNoPasses;
    return pairs < runs ? kPassSmall : kPassWide;
}

// 10 ... 20 slices (phases in us, s = 11 / 13 / 16 / 18; lognormal operands up to here and in the last paragraph).
// Up to one tile of 32 x 32 per compute unit, and up to 1.75 where the products repay a second round: these, k in eighths
// (402^3 before 25.7 / 33.9 / 44.7 / 62.8, now 16.1 / 18.8 / 23.0 / 26.0; 1.64 tiles: 600 x 700 x 384 21.8 / 28.0 / 36.1 / 49.1, 23.6 / 28.1 / 34.6 / 40.4,
// 600 x 700 x 188 17.6 / 21.8 / 27.1 / 36.5, 20.8 / 23.9 / 28.5 / 33.0; 800^3, 2.4 tiles, 40.6 / 54.8 / 75.1 / 102, 53.1 / 66.2 / 84.7 / 100;
// 10 slices have a kernel of one pass there).
// Then, up to one 64 x 64 tile per compute unit, the one-pass kernels on that tile with 512 registers to a wavefront up to 16
// slices (800^3: against 49.8 / 65.2 / 83.2 in passes; 18: 95.0), beyond at short k (calls, one-pass kernel against passes: s = 19 896 x 832 x 113
// 31.2 / 34.2, 704 x 1240 x 167 45.8 / 49.8; s = 17 908 x 717 x 103 26.9 / 27.9, 640 x 1253 x 448 60.9 / 60.6; s = 18 978 x 768 x 86 30.1 / 29.4, 896 x 418 x 118
// 28.3 / 28.7).
// 10 ... 12 slices by the time of the launches; the one-pass kernel, 128 x 64 or 64 x 64 tiles, stays where the figures are even, and at the
// shortest contractions (s = 11 768 x 3372 x 116 34.9 against 37.4).  What decides is rounds: it is 5 to 10 percent ahead in whole ones (s = 10, calls: 1280^3 91.2 against 100, 1872^3
// 253 / 274, 384 x 3066 x 2801 207 / 239; s = 11 604 x 1811 x 5512 426 / 460), behind where its last one is nearly empty and pairs of
// 64 x 64 tiles fit (s = 12 2688 x 2368 x 286 161 / 139, s = 11 1614 x 2688 x 423 128 / 117, s = 10 4537 x 599 x 576 93.4 / 87.9).
// Launches long enough to sit at the power cap run 5 percent faster in passes of 128 x 64 tiles than the fit has them (4073^3, s = 11 2622 / 2465; 3746^3,
// s = 12 2483 / 2326).  Operands badly scaled
// along k, which is what asks for so many slices, digits in all of them; under the power cap the figures depend on the digits (lognormal entries
// have none from the 9th slice on: with them passes of 10 slices measured ahead at 4096^3, 3070 -> 3210 TOP/s).
// Beyond, 128 x 64 or 64 x 64 by rounds of the chip: two 64 x 64 tiles at a time cost a compute unit 1.04 of a 128 x 64 one;
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
    if (one_round_of_96(s, m, n)) return kPassMiddle;
    if (tiles(64, 64) <= cus) return s <= 16 || kp < (s == 18 ? 256 : 512) ? kNoPasses : kPassSmall;
    const double small = pair_rounds(s, order_blocks(m, n, 64, 64), cus);
    const long long blocks = order_blocks(m, n, 128, 64);
    const double wide = single_rounds(s, blocks, cus);
    if (s > 12) return 1.04 * small < wide * (1.0 + 40.0 / kp) ? kPassSmall : kPassWide;
    static constexpr LaunchTime kPairs[3] = {{1.034, 7.3, 8.0}, {1.0, 7.3, 8.0}, {0.97, 7.3, 8.0}}, kLone{1.0, 10.3, 6.7};
    static constexpr LaunchTime kOne{1.01, 5.2, 4.6}, kOne64[3] = {{1.178, 9.2, 5.5}, {1.12, 9.2, 5.5}, {1.168, 9.2, 5.5}};
    const double x = 1e-3 * kp * (s * (s + 1) / 2);
    const double pairs = kPairs[s - 10].us(small, x);
    double lone = s == 10 ? 1e30 : kLone.us(wide, x);              // (no 128 x 64 tile in passes for 10 slices: nowhere ahead)
    if (lone > 400.0) lone *= 0.95;
    const double one = fused_small_tile(s, m, n) ? kOne64[s - 10].us(0.5 * single_rounds(s, tiles(64, 64), cus), x) : kOne.us(wide, x);
    if (kp <= 128 || (pairs < lone ? pairs : lone) >= 0.985 * one) return kNoPasses;
    return pairs < lone ? kPassSmall : kPassWide;
}

hipError_t launch_gemm_passes(PassShape shape, int s, int m, int n, int kp, int stride, const int8_t *pA, const int8_t *pB,
                              const int32_t *eA, const int32_t *eB, double *C, int ldc, int Q, hipStream_t st)
{
    if (m <= 0 || n <= 0) return hipSuccess;
    if (shape == kNoPasses || stride < s) return hipErrorInvalidValue;
    if (shape == kPassEighths) return launch_gemm_eighths_passes(s, m, n, kp, stride, pA, pB, eA, eB, C, ldc, Q, st);
    switch (s) {
#define OZ_CASE(S_) case S_: return launch_gemm_passes_##S_(shape, m, n, kp, stride, pA, pB, eA, eB, C, ldc, Q, st);
        OZ_CASE(4) OZ_CASE(5) OZ_CASE(6) OZ_CASE(7) OZ_CASE(8) OZ_CASE(9)
        OZ_CASE(10) OZ_CASE(11) OZ_CASE(12) OZ_CASE(13) OZ_CASE(14) OZ_CASE(15) OZ_CASE(16) OZ_CASE(17) OZ_CASE(18) OZ_CASE(19)
        OZ_CASE(20)
#undef OZ_CASE
    }
    return hipErrorInvalidValue;
}

}  // namespace oz
