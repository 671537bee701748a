// Fused slice-product kernels for problems whose tiles do not fill the chip: equal slice counts, whole contraction
// in int32.  Same computation, plane layout and order of the binary64 additions as gemm_fused_kernel (gemm.hip); what
// differs is that the wavefronts of a work-group also divide the CONTRACTION among each other.
//
// A problem of a thousand rows and columns has about one 64 x 64 tile per compute unit.  Four wavefronts of 32 x 32
// outputs are then all a compute unit gets, one per SIMD, and nobody covers a wavefront that waits for a barrier or
// an operand.  Here a 64 x 64 tile is worked on by eight wavefronts, two per SIMD: four take the even 32-deep
// k-blocks, four the odd ones, and the two int32 halves of every diagonal sum are added in LDS at the end (exact, so
// the result is the same bit for bit).  Smaller problems still use 32 x 32 tiles, each wavefront a k-block in eight.
#include "gemm_dev.h"
#include "slice_dev.h"

namespace oz {

namespace {

// ---- tile 64 x 64, 2 x 2 x 2 wavefronts (m, n, k), operands staged through LDS (2 ... 6 slices) -----------------------------------
// A stage is two 32-deep k-blocks of the four fragment rows; ring of three stages.
// The loop is the hand-pipelined one of gemm_fused_kernel: slices of A from the last to the first, operands of slice
// l - 1 read while the products of slice l run, the end-of-stage barrier before the products of slice 0, copies of a
// later stage issued one at a time behind single matrix instructions.
template <int S>
struct CfgHalves {
    static constexpr int STAGE = 4 * 2 * S * kFragBytes;
    static constexpr int LDS = 3 * STAGE;                   // also holds the exchange of the sums: 16 S KiB
    static_assert(LDS <= kLdsBytes, "stages do not fit LDS");
};

template <int S>
__global__ __launch_bounds__(512) void gemm_halves_kernel(const int8_t *__restrict__ pA, const int8_t *__restrict__ pB,
                                                          const int32_t *__restrict__ eA, const int32_t *__restrict__ eB,
                                                          double *__restrict__ C, int ldc, int m, int n, int KB,
                                                          int tiles_m, int tiles_n, int Q)
{
    using G = CfgHalves<S>;
    constexpr int STAGE = G::STAGE, CHUNK = 2 * S * kFragBytes, NW = 8, NU = S;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
    int tm, tn;
    if (!tile_of_block_xcd(blockIdx.x, tiles_m, tiles_n, false, tm, tn)) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave & 1, wn = (wave >> 1) & 1, kg = wave >> 2;
    const size_t row_bytes = (size_t)KB * (S * kFragBytes);
    // copy unit u = wave + 8 i of a stage: fragment row u / (2 S) (two of A, two of B), 1 KiB (k-block, slice) u % (2 S)
    const int8_t *src[NU];
#pragma unroll
    for (int i = 0; i < NU; ++i) {
        const int u = wave + i * NW, c = u / (2 * S), o = u % (2 * S);
        src[i] = (c < 2 ? pA + (size_t)(2 * tm + c) * row_bytes : pB + (size_t)(2 * tn + c - 2) * row_bytes) + (size_t)o * kFragBytes;
    }
    const unsigned ldsw = lds0 + wave * kFragBytes;
    auto issue = [&](auto I, unsigned voff, unsigned ldsbuf) {
        constexpr int i = decltype(I)::value;
        lds_dma16_at<i * NW * kFragBytes>(src[i], voff, ldsbuf);
    };
    const int nst = KB / 2;
    static_for<0, 2>([&](auto P) {
        constexpr int p = decltype(P)::value;
        const unsigned v = lane * 16 + (unsigned)(p < nst ? p : nst - 1) * (unsigned)CHUNK;
        static_for<0, NU>([&](auto I) { issue(I, v, ldsw + p * STAGE); });
    });
    wait_vmcnt<NU>();
    __syncthreads();

    v16i acc[S];
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][r] = 0;
    auto readA = [&](int l, const unsigned char *stage) -> v4i {
        return *(const v4i *)(stage + wm * CHUNK + (kg * S + l) * kFragBytes + lane * 16);
    };
    auto readB = [&](int h, const unsigned char *stage) -> v4i {
        return *(const v4i *)(stage + (2 + wn) * CHUNK + (kg * S + h) * kFragBytes + lane * 16);
    };
    v4i bf[S], af = readA(S - 1, lds);
    bf[0] = readB(0, lds);
    constexpr int NSLOT = S * (S - 1) / 2;
    int buf = 0;
    for (int st = 0; st < nst; ++st) {
        // (towards the end the copies and the reads ahead go on, of the last stage again: nobody uses them)
        const int ahead = st + 2 < nst ? st + 2 : nst - 1;
        const unsigned vnext = lane * 16 + (unsigned)ahead * (unsigned)CHUNK;
        const int buf1 = buf + 1 == 3 ? 0 : buf + 1, bufc = buf1 + 1 == 3 ? 0 : buf1 + 1;
        const unsigned ldsnext = ldsw + bufc * STAGE;
        const unsigned char *cur = lds + buf * STAGE, *nxt = lds + buf1 * STAGE;
        if constexpr (NU > NSLOT) static_for<0, NU>([&](auto I) { issue(I, vnext, ldsnext); });
        v4i afn, bfn;
        static_for<0, S>([&](auto L) {
            constexpr int l = S - 1 - decltype(L)::value;
            if constexpr (l > 0) {
                afn = readA(l - 1, cur);
                bf[S - l] = readB(S - l, cur);
                __builtin_amdgcn_sched_barrier(0);          // (the reads stay ahead of the products they hide behind)
            }
            static_for<0, S - l>([&](auto HH) {
                constexpr int hh = decltype(HH)::value, h = l == 0 ? S - 1 - hh : hh;
                if constexpr (l == 0 && hh == 0) {
                    // nothing of this stage is left to read, and the next one must have landed
                    wait_vmcnt<NU>();
                    __syncthreads();
                    afn = readA(S - 1, nxt);
                    bfn = readB(0, nxt);
                }
                acc[l + h] = __builtin_amdgcn_mfma_i32_32x32x32_i8(bf[h], af, acc[l + h], 0, 0, 0);
                constexpr int e = (S - 1 - l) * (S - l) / 2 + hh;
                if constexpr (NU <= NSLOT && e < NU) issue(std::integral_constant<int, (e < NU ? e : 0)>{}, vnext, ldsnext);
            });
            __builtin_amdgcn_sched_barrier(0);              // (and no product of the next slice moves up to wait for them)
            af = afn;
        });
        bf[0] = bfn;
        buf = buf1;
    }

    // The wavefronts kg = 0 and 1 of an output block hold the sums over the even and the odd k-blocks.  Each hands
    // over half of its accumulator registers (kg = 0 finishes r < 8, kg = 1 the others): 16 bytes per lane and
    // group of four registers, in LDS nobody else uses any more.
    wait_vmcnt<0>();
    __syncthreads();
    v4i *xch = (v4i *)lds + (size_t)(wave & 3) * (2 * S * 2 * 64) + lane;
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int q0 = 8 + 4 * g, q1 = 4 * g;       // registers handed over by kg = 0 / kg = 1
            v4i v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = kg ? acc[a][q1 + r] : acc[a][q0 + r];
            xch[((kg * S + a) * 2 + g) * 64] = v;
        }
    __syncthreads();
    int D[S][8];
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const v4i v = xch[(((kg ^ 1) * S + a) * 2 + g) * 64];
#pragma unroll
            for (int r = 0; r < 4; ++r) D[a][g * 4 + r] = v[r] + (kg ? acc[a][8 + 4 * g + r] : acc[a][4 * g + r]);
        }
    const int mi = (tm * 2 + wm) * 32 + (lane & 31);
    if (mi >= m) return;
    const bool stream = stream_c(C, ldc);
    const int ea = eA[mi];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int rr = kg * 8 + r;
        const int nj = (tn * 2 + wn) * 32 + 8 * (rr >> 2) + 4 * (lane >> 5) + (rr & 3);
        if (nj >= n) continue;
        int d[S];
#pragma unroll
        for (int a = 0; a < S; ++a) d[a] = D[a][r];
        store_c(&C[mi + (size_t)nj * ldc], ldexp(diagonal_sum<S>(d, Q), ea + eB[nj]), stream);
    }
}

// ---- tile 32 x 32, eight wavefronts along k, operands straight from memory into registers --------------------------
// Nothing of a tile is shared between wavefronts, so nothing goes through LDS and the loop has no barrier: wavefront w
// takes the k-blocks w, w + 8, ...; row l of the products frees slice l of A and slice S - 1 - l of B, which are
// loaded again for its next k-block at once.  The eight sums per output meet in LDS, kRound diagonals at a time;
// wavefront w finishes accumulator registers 2 w and 2 w + 1.
// Tile of a work-group: equal runs of tiles to the XCDs, in strips of four tile rows -- of all tile rows where there are twice as many tile
// columns or more.  (Four tiles of a 64 x 64 one after the
// other, with nothing to do for those beyond the edge, gave some XCDs half as many tiles again where a side has an odd number of
// them: 130 x 1500 x 3000, s = 3 / 7 20.2 / 44.1 us, now 12.9 / 25.1; 32 x 6000 x 200, s = 7 14.2, now 9.0.  What the order costs beyond the product
// shows in the NEXT call's set-up, which writes planes that L2s of other XCDs hold: whole columns leave most slices of B with
// the XCD that wrote them, rows and columns of strips do not.  Calls, 160 random sizes, against the groups of four, strips / whole columns: twice as many
// columns or more 0.970 / 0.960, slowest 1.05 / 1.01, and 256 x 1100 x 410, s = 7 20.7, 22.0 / 20.4; about square 0.995 / 1.001; more rows 0.963 / 1.004.  One
// in thirty stays 2 to 4 percent behind the groups of four, 384^3 s = 7 11.9 against 12.2 among them.)
// The tile's place is on the way to the first load: one multiplication with magic = ceil(2^32 / d), d = 4 tiles_n or tiles_m, in place of the three
// divisions of tile_of_block(), which take 0.2 us of 12 (exact while the number of tiles times d is below 2^32: some thousand tiles at most come
// here).
__device__ __forceinline__ void tile_in_strips(unsigned b, int tiles_m, int tiles_n, unsigned magic, int whole, int &tm, int &tn)
{
    const unsigned nb = (unsigned)(tiles_m * tiles_n), xcd = b & 7, rem = nb & 7;
    const unsigned lin = xcd * (nb >> 3) + (xcd < rem ? xcd : rem) + (b >> 3);
    const unsigned q = __umulhi(lin, magic);
    if (whole) {
        tn = (int)q;
        tm = (int)(lin - q * (unsigned)tiles_m);
        return;
    }
    const unsigned in = lin - q * (4u * tiles_n);
    const unsigned left = tiles_m - 4 * q;                    // rows of this strip, if fewer than four
    const unsigned c = left >= 4 ? in >> 2 : left == 3 ? in / 3u : left == 2 ? in >> 1 : in;
    tn = (int)c;
    tm = (int)(4 * q + in - c * (left >= 4 ? 4u : left));
}
// (up to four tile rows the two are the same)
inline int strip_whole(int tiles_m, int tiles_n) { return tiles_m > 4 && tiles_n >= 2 * tiles_m; }
inline unsigned strip_magic(int tiles_m, int tiles_n)
{
    const unsigned long long d = strip_whole(tiles_m, tiles_n) ? tiles_m : 4ULL * tiles_n;
    return (unsigned)(((1ULL << 32) + d - 1) / d);
}

template <int S>
struct CfgEighths {
    static constexpr int ROUND = S == 1 ? 1 : S <= 5 ? 2 : 4;             // diagonals per round: 32 KiB of LDS each
    static constexpr int LDS = ROUND * 8 * 8 * 64 * 8;
};

template <int S>
__global__ __launch_bounds__(512) void gemm_eighths_kernel(const int8_t *__restrict__ pA, const int8_t *__restrict__ pB,
                                                           const int32_t *__restrict__ eA, const int32_t *__restrict__ eB,
                                                           double *__restrict__ C, int ldc, int m, int n, int KB,
                                                           int tiles_m, int tiles_n, unsigned magic, int whole, int Q)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    int tm, tn;
    tile_in_strips(blockIdx.x, tiles_m, tiles_n, magic, whole, tm, tn);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t row_bytes = (size_t)KB * (S * kFragBytes);
    v16i acc[S];
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][r] = 0;
    if (wave < KB) {
        const v4i *a = (const v4i *)(pA + (size_t)tm * row_bytes + (size_t)wave * (S * kFragBytes)) + lane;
        const v4i *b = (const v4i *)(pB + (size_t)tn * row_bytes + (size_t)wave * (S * kFragBytes)) + lane;
        v4i af[S], bf[S];
#pragma unroll
        for (int q = 0; q < S; ++q) {
            af[q] = a[q * 64];
            bf[S - 1 - q] = b[(S - 1 - q) * 64];
        }
        for (int kb = wave; kb < KB; kb += 8) {
            // (the last k-block of a wavefront is loaded once more: nobody uses it)
            const size_t step = kb + 8 < KB ? (size_t)8 * S * 64 : 0;
            a += step;
            b += step;
            static_for<0, S>([&](auto L) {
                constexpr int l = decltype(L)::value;
                static_for<0, S - l>([&](auto HH) {
                    constexpr int h = S - 1 - l - decltype(HH)::value;
                    acc[l + h] = __builtin_amdgcn_mfma_i32_32x32x32_i8(bf[h], af[l], acc[l + h], 0, 0, 0);
                });
                af[l] = a[l * 64];
                bf[S - 1 - l] = b[(S - 1 - l) * 64];
                __builtin_amdgcn_sched_barrier(0);
            });
        }
    }
    // the sums of the eight wavefronts meet in LDS, ROUND diagonals at a time; D: those of accumulator registers 2 wave and 2 wave + 1
    typedef int v2i __attribute__((ext_vector_type(2)));
    v2i *x = (v2i *)lds;
    int D[2][S];
    constexpr int ROUND = CfgEighths<S>::ROUND;
    static_for<0, (S + ROUND - 1) / ROUND>([&](auto P) {
        constexpr int a0 = decltype(P)::value * ROUND, a1 = a0 + ROUND < S ? a0 + ROUND : S;
        if constexpr (a0 > 0) __syncthreads();
#pragma unroll
        for (int a = a0; a < a1; ++a)
#pragma unroll
            for (int r = 0; r < 8; ++r) x[(((a - a0) * 8 + r) * 8 + wave) * 64 + lane] = v2i{acc[a][2 * r], acc[a][2 * r + 1]};
        __syncthreads();
#pragma unroll
        for (int a = a0; a < a1; ++a) {
            v2i s{0, 0};
#pragma unroll
            for (int w = 0; w < 8; ++w) s += x[(((a - a0) * 8 + wave) * 8 + w) * 64 + lane];
            D[0][a] = s[0];
            D[1][a] = s[1];
        }
    });
    const int mi = tm * 32 + (lane & 31);
    if (mi >= m) return;
    const bool stream = stream_c(C, ldc);
    const int ea = eA[mi];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int rr = 2 * wave + r;
        const int nj = tn * 32 + 8 * (rr >> 2) + 4 * (lane >> 5) + (rr & 3);
        if (nj < n) store_c(&C[mi + (size_t)nj * ldc], ldexp(diagonal_sum<S>(D[r], Q), ea + eB[nj]), stream);
    }
}

// ---- the same tile, scales and slices in the same launch: contractions of up to 256, few tiles ----------------------------------
// A wavefront reads and slices one k-block of the tile, 32 deep (EPL = 16 entries of either operand to a lane), or half of one up to k = 128 (EPL = 8); the
// maxima of the rows and columns meet in LDS, then the slices do, and four wavefronts multiply them, 16 x 16 outputs each. (Every wavefront multiplying what it has
// sliced, the eight sums meeting in LDS, moves 2.7 times the bytes through LDS: launch and kernel 8.1 / 10.5 us at
// 128^3 s = 3 / 7, now 7.6 / 9.2.)  Every row is read and sliced once for each tile of its row, which few tiles make up for by the launch and the
// gap between the two (128^3, s = 3: 3.4 + 4.1 us on the device and as much again of launches).  The planes, exponents and non-finite words that a call
// leaves in the workspace are written by the tiles of the first column (A) and row (B).
// What bounds it: the host up to seven slices, then slicing, eight entries of either operand to a lane and two wavefronts to a SIMD.
constexpr int kWholeMost = 10, kWholeNearest = 8, kWholeLong = 4;      // slices: k up to 128, nearest ones, k up to 256
template <int S, int EPL>
struct CfgWhole {
    static constexpr int HEAD = 2 * 8 * 32 * 8 + 64 * 4;     // maxima and exponents
    static constexpr int LDS = HEAD + 2 * (EPL / 2) * S * kFragBytes;
};
template <int S, bool NEAREST, int EPL>
__global__ __launch_bounds__(512) void gemm_eighths_whole_kernel(
    const unsigned long long *__restrict__ A, int lda, const unsigned long long *__restrict__ B, int ldb, int32_t *__restrict__ eA,
    int32_t *__restrict__ eB, int8_t *__restrict__ pA, int8_t *__restrict__ pB, double *__restrict__ C, int ldc, int m, int n, int K, int KB, int tiles_m,
    unsigned long long *__restrict__ header, long long bad_offset, int Q)
{
    constexpr int NQ = EPL / 4, KBL = EPL / 2;               // quads of a lane, k-blocks of the tile
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tm = blockIdx.x % (unsigned)tiles_m, tn = blockIdx.x / (unsigned)tiles_m, tiles_n = gridDim.x / (unsigned)tiles_m;
    const int lane = threadIdx.x & 63, r = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int k0 = wave * 2 * EPL, kl = k0 + hh * EPL;       // of the wavefront and of the lane
    const int ra = tm * 32 + r, rb = tn * 32 + r;
    // (rows beyond the operand repeat its last one, at a scale that makes every slice zero)
    const unsigned long long *a = A + (ra < m ? ra : m - 1), *b = B + (size_t)(rb < n ? rb : n - 1) * ldb;
    unsigned long long xa[NQ][4], xb[NQ][4];
    if (k0 + 2 * EPL <= K) {
        typedef unsigned long long pair __attribute__((ext_vector_type(2), aligned(8)));
#pragma unroll
        for (int t = 0; t < EPL; ++t) xa[t >> 2][t & 3] = a[(size_t)(kl + t) * lda];
#pragma unroll
        for (int t = 0; t < EPL; t += 2) {
            const pair v = *(const pair *)(b + kl + t);
            xb[t >> 2][t & 3] = v[0];
            xb[t >> 2][(t & 3) + 1] = v[1];
        }
    } else {
#pragma unroll
        for (int t = 0; t < EPL; ++t) {
            const int k = kl + t < K ? kl + t : K - 1;
            xa[t >> 2][t & 3] = a[(size_t)k * lda];
            xb[t >> 2][t & 3] = b[k];
        }
#pragma unroll
        for (int t = 0; t < EPL; ++t) {
            xa[t >> 2][t & 3] = kl + t < K ? xa[t >> 2][t & 3] : 0ULL;
            xb[t >> 2][t & 3] = kl + t < K ? xb[t >> 2][t & 3] : 0ULL;
        }
    }
    auto *const smx = (unsigned long long *)lds;             // [operand][wavefront][row]
    unsigned long long mx[2] = {0, 0};
#pragma unroll
    for (int t = 0; t < EPL; ++t) {
        const unsigned long long u = xa[t >> 2][t & 3] & 0x7fffffffffffffffULL, v = xb[t >> 2][t & 3] & 0x7fffffffffffffffULL;
        mx[0] = u > mx[0] ? u : mx[0];
        mx[1] = v > mx[1] ? v : mx[1];
    }
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        const unsigned long long u = __shfl_xor(mx[o], 32);
        mx[o] = u > mx[o] ? u : mx[o];
        if (hh == 0) smx[(o * 8 + wave) * 32 + r] = mx[o];
    }
    __syncthreads();
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const unsigned long long u = smx[(o * 8 + w) * 32 + r];
            mx[o] = u > mx[o] ? u : mx[o];
        }
    const int ea = exponent_above(mx[0]) + (NEAREST ? 1 : 0), eb = exponent_above(mx[1]) + (NEAREST ? 1 : 0);
    if (wave == 0) {
        unsigned *const bad = (unsigned *)((char *)header + bad_offset);
        const unsigned long long anyA = __ballot(mx[0] >= 0x7ff0000000000000ULL), anyB = __ballot(mx[1] >= 0x7ff0000000000000ULL);
        if (tn == 0) {
            if (hh == 0) eA[ra] = ra < m ? ea : 0;
            if (lane == 0) bad[tm] = anyA ? 1u : 0u;
        }
        if (tm == 0) {
            if (hh == 0) eB[rb] = rb < n ? eb : 0;
            if (lane == 0) bad[tiles_m + tn] = anyB ? 1u : 0u;
        }
        if (blockIdx.x == 0 && lane < 6) {                   // the header, as scale_split_kernel writes it
            const unsigned long long v[6] = {0ULL, (unsigned long long)(tiles_m + tiles_n), (unsigned long long)bad_offset, kBadWordsMagic,
                                             (unsigned long long)(uintptr_t)header, 0ULL};
            header[lane == 0 ? 0 : kHeaderBadWords + lane - 1] = v[lane];
        }
    }
    typedef int vec __attribute__((ext_vector_type(NQ)));
    vec af[S], bf[S];
    auto slice = [&](const unsigned long long (&x)[NQ][4], int e, vec (&to)[S]) __attribute__((always_inline)) {
        Quad<NEAREST> q[NQ];
#pragma unroll
        for (int t = 0; t < NQ; ++t) q[t].load(x[t], e);
        static_for<0, S>([&](auto LC) __attribute__((always_inline)) {
            constexpr int l = decltype(LC)::value, WIN = Quad<NEAREST>::WIN;
#pragma unroll
            for (int t = 0; t < NQ; ++t) {
                if constexpr (l % WIN == 0) q[t].window();
                to[l][t] = (int)q[t].template word<l % WIN + 1>();
            }
        });
    };
    constexpr int kZeroScale = 4096;                         // exponent at which every finite number has zero slices only
    slice(xa, ra < m ? ea : kZeroScale, af);
    slice(xb, rb < n ? eb : kZeroScale, bf);
    // entry (r, k) of a k-block at 16 (r + 32 (k / 16)) + k % 16, in LDS as in the planes
    const int place = EPL == 16 ? lane * 16 : (r + 32 * (wave & 1)) * 16 + 8 * hh;
    unsigned char *const sliced = lds + CfgWhole<S, EPL>::HEAD;
#pragma unroll
    for (int l = 0; l < S; ++l) {
        *(vec *)(sliced + ((k0 / 32) * S + l) * kFragBytes + place) = af[l];
        *(vec *)(sliced + ((KBL + k0 / 32) * S + l) * kFragBytes + place) = bf[l];
    }
    auto *const sexp = (int *)(smx + 2 * 8 * 32);            // exponents of rows and columns
    if (wave == 0) sexp[lane] = hh ? eb : ea;
    auto store = [&](int8_t *planes, int tile, const vec (&from)[S]) __attribute__((always_inline)) {
        int8_t *to = planes + ((size_t)tile * KB + k0 / 32) * (S * kFragBytes) + place;
#pragma unroll
        for (int l = 0; l < S; ++l) *(vec *)(to + l * kFragBytes) = from[l];
    };
    if (tn == 0) store(pA, tm, af);
    if (tm == 0) store(pB, tn, bf);
    __syncthreads();
    if (wave >= 4) return;
    // 16 rows x 16 columns to each of four wavefronts; this lane's part of an operand as in gemm_fused16_kernel
    const int i2 = wave & 1, j2 = wave >> 1;
    const unsigned char *const mine = sliced + ((lane >> 4) >> 1) * (S * kFragBytes) + ((lane & 15) + 32 * ((lane >> 4) & 1)) * 16;
    v4i acc[S];
#pragma unroll
    for (int d = 0; d < S; ++d) acc[d] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KBL / 2; ++ks) {
        v4i a16[S], b16[S];
#pragma unroll
        for (int l = 0; l < S; ++l) {
            a16[l] = *(const v4i *)(mine + (2 * ks * S + l) * kFragBytes + i2 * 256);
            b16[l] = *(const v4i *)(mine + ((KBL + 2 * ks) * S + l) * kFragBytes + j2 * 256);
        }
#pragma unroll
        for (int l = 0; l < S; ++l)
#pragma unroll
            for (int h = 0; h < S - l; ++h) acc[l + h] = __builtin_amdgcn_mfma_i32_16x16x64_i8(b16[h], a16[l], acc[l + h], 0, 0, 0);
    }
    const int mi = tm * 32 + i2 * 16 + (lane & 15);
    if (mi >= m) return;
    const bool stream = stream_c(C, ldc);
    const int er = sexp[i2 * 16 + (lane & 15)];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int c = j2 * 16 + 4 * (lane >> 4) + q, nj = tn * 32 + c;
        if (nj >= n) continue;
        int d[S];
#pragma unroll
        for (int a = 0; a < S; ++a) d[a] = acc[a][q];
        store_c(&C[mi + (size_t)nj * ldc], ldexp(diagonal_sum<S>(d, Q), er + sexp[32 + c]), stream);
    }
}

// ---- the same tile for 11 ... 20 slices, whose diagonal sums do not fit the registers together: passes over groups of Ws
// diagonals, in ascending order, as in gemm_passes_dev.h --------------------------------------------------------------------
// A pass over the diagonals up to SN + 1 takes the slices 1 ... SN; step i of a k-block brings slice SN - i of A and slice
// i + 1 of B, and meets the last W slices of B: product j of it belongs to the pass's j-th diagonal from the end.  Operands
// are loaded AHEAD steps before their use.  The sums of a pass meet in LDS as above, and every wavefront adds them to
// its two entries, in registers, before the next pass.  What bounds it: operands out of the L2s, 36 to 50 bytes per clock and compute
// unit where all are busy.  GEMM, us, s = 11 / 13 / 18, one-pass 64 x 64 tiles before -> now: 500 x 384 x 512 25.3 / 34.0 / 62.0 -> 15.9 /
// 19.0 / 26.9, 300 x 500 x 1000 41.9 / 58.4 / 114 -> 22.4 / 27.2 / 40.4, 130 x 1500 x 3000 109 / 159 / 320 -> 50.7 / 63.6 / 103.
template <int... Ws>
__global__ __launch_bounds__(512) void gemm_eighths_passes_kernel(
    const int8_t *__restrict__ pA, const int8_t *__restrict__ pB, const int32_t *__restrict__ eA, const int32_t *__restrict__ eB,
    double *__restrict__ C, int ldc, int m, int n, int KB, int stride, int tiles_m, int tiles_n, unsigned magic,
    int whole, int Q)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    int tm, tn;
    tile_in_strips(blockIdx.x, tiles_m, tiles_n, magic, whole, tm, tn);
    const unsigned lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t kb_bytes = (size_t)stride * kFragBytes, row_bytes = (size_t)KB * kb_bytes;
    constexpr int NP = sizeof...(Ws), ROUND = 4, AHEAD = 4;
    constexpr int WS[NP] = {Ws...};
    LevelSum sum[2];
    static_for<0, NP>([&](auto PP) {
        constexpr int p = decltype(PP)::value, W = WS[p], BEFORE = diagonals_before<NP>(WS, p), SN = BEFORE + W;
        constexpr int AH = AHEAD < SN ? AHEAD : SN;
        v16i acc[W];
#pragma unroll
        for (int a = 0; a < W; ++a)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][r] = 0;
        if (wave < KB) {
            const v4i *a = (const v4i *)(pA + (size_t)tm * row_bytes + (size_t)wave * kb_bytes);
            const v4i *b = (const v4i *)(pB + (size_t)tn * row_bytes + (size_t)wave * kb_bytes);
            v4i af[SN], bf[SN];
            static_for<0, AH>([&](auto I) {
                constexpr int i = decltype(I)::value;
                af[i] = (a + (SN - 1 - i) * 64)[lane];
                bf[i] = (b + i * 64)[lane];
            });
            for (int kb = wave; kb < KB; kb += 8) {
                // (the first steps of the last k-block of a wavefront are loaded once more: nobody uses them)
                const size_t step = kb + 8 < KB ? (size_t)8 * stride * 64 : 0;
                const v4i *an = a + step, *bn = b + step;
                v4i an_[AH], bn_[AH];
                static_for<0, SN>([&](auto I) {
                    constexpr int i = decltype(I)::value, used = i + 1 < W ? i + 1 : W;
                    if constexpr (i + AH < SN) {
                        af[i + AH] = (a + (SN - 1 - i - AH) * 64)[lane];
                        bf[i + AH] = (b + (i + AH) * 64)[lane];
                    } else {
                        an_[i + AH - SN] = (an + (SN - 1 - (i + AH - SN)) * 64)[lane];
                        bn_[i + AH - SN] = (bn + (i + AH - SN) * 64)[lane];
                    }
                    static_for<0, used>([&](auto J) {
                        constexpr int j = used - 1 - decltype(J)::value;
                        acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(bf[i - j], af[i], acc[j], 0, 0, 0);
                    });
                    __builtin_amdgcn_sched_barrier(0);
                });
                a = an;
                b = bn;
#pragma unroll
                for (int i = 0; i < AH; ++i) {
                    af[i] = an_[i];
                    bf[i] = bn_[i];
                }
            }
        }
        typedef int v2i __attribute__((ext_vector_type(2)));
        v2i *x = (v2i *)lds;
        static_for<0, (W + ROUND - 1) / ROUND>([&](auto P) {
            constexpr int a0 = decltype(P)::value * ROUND, a1 = a0 + ROUND < W ? a0 + ROUND : W;
            if constexpr (a0 > 0 || p > 0) __syncthreads();
#pragma unroll
            for (int a = a0; a < a1; ++a)
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    x[(((a - a0) * 8 + r) * 8 + wave) * 64 + lane] = v2i{acc[W - 1 - a][2 * r], acc[W - 1 - a][2 * r + 1]};
            __syncthreads();
#pragma unroll
            for (int a = a0; a < a1; ++a) {
                v2i s{0, 0};
#pragma unroll
                for (int w = 0; w < 8; ++w) s += x[(((a - a0) * 8 + wave) * 8 + w) * 64 + lane];
                const double unit = __builtin_ldexp(1.0, -kSliceBits * (BEFORE + a + 2));
#pragma unroll
                for (int r = 0; r < 2; ++r) sum[r].add((double)s[r] * unit, Q, p + 1 == NP && a == W - 1);
            }
        });
        // (the sums are formed before the next pass: left to itself the compiler keeps their terms until after it)
#pragma unroll
        for (int r = 0; r < 2; ++r) asm volatile("" : "+v"(sum[r].S), "+v"(sum[r].L));
    });
    const int mi = tm * 32 + (lane & 31);
    if (mi >= m) return;
    const bool stream = stream_c(C, ldc);
    const int ea = eA[mi];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int rr = 2 * wave + r;
        const int nj = tn * 32 + 8 * (rr >> 2) + 4 * (lane >> 5) + (rr & 3);
        if (nj < n) store_c(&C[mi + (size_t)nj * ldc], ldexp(sum[r].S, ea + eB[nj]), stream);
    }
}

template <int S>
hipError_t launch_halves(int m, int n, int kp, const int8_t *pA, const int8_t *pB, const int32_t *eA, const int32_t *eB,
                         double *C, int ldc, int Q, hipStream_t st)
{
    auto kern = gemm_halves_kernel<S>;
    static std::atomic<unsigned long long> configured{0};
    if (hipError_t e = allow_dynamic_lds((const void *)kern, CfgHalves<S>::LDS, configured); e != hipSuccess) return e;
    const int tiles_m = (m + 63) / 64, tiles_n = (n + 63) / 64;
    note_gemm_kernel("gemm_halves_kernel<%d> tile 64x64, 8 wavefronts, k in halves", S);
    kern<<<(unsigned)tile_order_blocks(tiles_m, tiles_n, false), 512, CfgHalves<S>::LDS, st>>>(pA, pB, eA, eB, C, ldc, m, n, kp / kFrag,
                                                                                           tiles_m, tiles_n, Q);
    return hipGetLastError();
}

template <int S>
hipError_t launch_eighths(int m, int n, int kp, const int8_t *pA, const int8_t *pB, const int32_t *eA, const int32_t *eB,
                          double *C, int ldc, int Q, hipStream_t st)
{
    auto kern = gemm_eighths_kernel<S>;
    static std::atomic<unsigned long long> configured{0};
    if (hipError_t e = allow_dynamic_lds((const void *)kern, CfgEighths<S>::LDS, configured); e != hipSuccess) return e;
    const int tiles_m = (m + 31) / 32, tiles_n = (n + 31) / 32;
    note_gemm_kernel("gemm_eighths_kernel<%d> tile 32x32, 8 wavefronts, k in eighths", S);
    kern<<<(unsigned)(tiles_m * tiles_n), 512, CfgEighths<S>::LDS, st>>>(pA, pB, eA, eB, C, ldc, m, n, kp / kFrag, tiles_m, tiles_n, strip_magic(tiles_m, tiles_n), strip_whole(tiles_m, tiles_n), Q);
    return hipGetLastError();
}

template <int... Ws>
hipError_t launch_eighths_passes(int m, int n, int kp, int stride, const int8_t *pA, const int8_t *pB, const int32_t *eA, const int32_t *eB,
                                 double *C, int ldc, int Q, hipStream_t st)
{
    auto kern = gemm_eighths_passes_kernel<Ws...>;
    static std::atomic<unsigned long long> configured{0};
    constexpr int LDS = 4 * 8 * 8 * 64 * 8;
    if (hipError_t e = allow_dynamic_lds((const void *)kern, LDS, configured); e != hipSuccess) return e;
    const int tiles_m = (m + 31) / 32, tiles_n = (n + 31) / 32;
    note_gemm_kernel("gemm_eighths_passes_kernel<%d> tile 32x32, 8 wavefronts, k in eighths", (Ws + ...));
    kern<<<(unsigned)(tiles_m * tiles_n), 512, LDS, st>>>(pA, pB, eA, eB, C, ldc, m, n, kp / kFrag, stride, tiles_m, tiles_n,
                                                    strip_magic(tiles_m, tiles_n), strip_whole(tiles_m, tiles_n), Q);
    return hipGetLastError();
}

template <int S>
hipError_t launch_eighths_plan(int m, int n, int kp, int stride, const int8_t *pA, const int8_t *pB, const int32_t *eA,
                               const int32_t *eB, double *C, int ldc, int Q, hipStream_t st)
{
    constexpr PassPlan P = pass_plan(S);
    if constexpr (P.n == 2) return launch_eighths_passes<P.w[0], P.w[1]>(m, n, kp, stride, pA, pB, eA, eB, C, ldc, Q, st);
    else return launch_eighths_passes<P.w[0], P.w[1], P.w[2]>(m, n, kp, stride, pA, pB, eA, eB, C, ldc, Q, st);
}

template <int S, bool NEAREST>
hipError_t launch_eighths_whole(int m, int n, int k, const double *A, int lda, const double *B, int ldb, int32_t *eA, int32_t *eB, int8_t *pA, int8_t *pB,
                                unsigned long long *header, size_t bad_offset, double *C, int ldc, int Q, hipStream_t st)
{
    const int kp = round_up(k, kPad), tiles_m = (m + 31) / 32, tiles_n = (n + 31) / 32;
    note_gemm_kernel("gemm_eighths_whole_kernel<%d> tile 32x32, 8 wavefronts slice, 4 multiply", S);
    auto launch = [&](auto EC) -> hipError_t {
        auto kern = gemm_eighths_whole_kernel<S, NEAREST, decltype(EC)::value>;
        static std::atomic<unsigned long long> configured{0};
        constexpr int LDS = CfgWhole<S, decltype(EC)::value>::LDS;
        if (hipError_t e = allow_dynamic_lds((const void *)kern, LDS, configured); e != hipSuccess) return e;
        kern<<<(unsigned)(tiles_m * tiles_n), 512, LDS, st>>>((const unsigned long long *)A, lda, (const unsigned long long *)B, ldb, eA, eB, pA, pB,
                                                                             C, ldc, m, n, k, kp / kFrag, tiles_m, header, (long long)bad_offset, Q);
        return hipGetLastError();
    };
    if (kp <= 128) return launch(std::integral_constant<int, 8>{});
    if constexpr (S <= kWholeLong && !NEAREST) return launch(std::integral_constant<int, 16>{});
    return hipErrorInvalidValue;
}

}  // namespace

// Where it pays (calls, us, two launches and this; 9 us is what the host takes for two of them, 6.8 for one): up to one tile to a compute unit and k = 128
// throughout (128^3 s = 1 / 3 / 5 / 7 / 9 / 10 8.7 / 9.6 / 8.8 / 9.6 / 9.4 / 10.4 and 6.8 / 6.8 / 7.0 / 6.8 / 7.4 / 8.1, 500 x 500 x 128 s = 3 / 7 / 10 9.7 / 9.9 / 11.3 and
// 6.9 / 7.3 / 8.8; 700 x 700 x 128, 484 tiles, s = 7 12.6 against 15.6 then); up to 256, where a wavefront slices twice as much, with four slices (128 x 128 x 256 s = 2 / 3 /
// 4 / 5 / 7 8.7 / 9.5 / 9.1 / 9.1 / 9.7 and 7.5 / 7.4 / 8.0 / 9.0 / 10.3, 500 x 500 x 256 s = 4 / 5 9.4 / 9.6 and 9.0 / 9.9); nearest slices, which cost half as much again, up to
// eight (128^3 s = 3 / 6 / 8 8.9 / 9.4 / 9.6 and 7.1 / 8.4 / 9.4). Eleven and more: passes.
bool gemm_eighths_whole_handles(int m, int n, int k, int s, bool nearest)
{
    if (m < 1 || n < 1 || k < 1 || (long long)((m + 31) / 32) * ((n + 31) / 32) > device_cus()) return false;
    return k <= 128 ? s <= (nearest ? kWholeNearest : kWholeMost) : k <= 256 && s <= kWholeLong && !nearest;
}

hipError_t launch_gemm_eighths_whole(int m, int n, int k, const double *A, int lda, const double *B, int ldb, int s, bool nearest, int32_t *eA,
                                     int32_t *eB, int8_t *pA, int8_t *pB, unsigned long long *header, size_t bad_offset, double *C, int ldc, int Q,
                                     hipStream_t st)
{
    if (!gemm_eighths_whole_handles(m, n, k, s, nearest)) return hipErrorInvalidValue;
    auto launch = [&](auto SC) -> hipError_t {
        constexpr int S = decltype(SC)::value;
        if constexpr (S <= kWholeNearest)
            if (nearest) return launch_eighths_whole<S, true>(m, n, k, A, lda, B, ldb, eA, eB, pA, pB, header, bad_offset, C, ldc, Q, st);
        return launch_eighths_whole<S, false>(m, n, k, A, lda, B, ldb, eA, eB, pA, pB, header, bad_offset, C, ldc, Q, st);
    };
    static_assert(kWholeMost == 10, "cases");
    switch (s) {
#define OZ_CASE(S_) case S_: return launch(std::integral_constant<int, S_>{});
        OZ_CASE(1) OZ_CASE(2) OZ_CASE(3) OZ_CASE(4) OZ_CASE(5) OZ_CASE(6) OZ_CASE(7) OZ_CASE(8) OZ_CASE(9) OZ_CASE(10)
#undef OZ_CASE
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gemm_eighths_passes(int s, int m, int n, int kp, int stride, const int8_t *pA, const int8_t *pB, const int32_t *eA,
                                      const int32_t *eB, double *C, int ldc, int Q, hipStream_t st)
{
    if (m <= 0 || n <= 0) return hipSuccess;
    switch (s) {
#define OZ_CASE(S_) case S_: return launch_eighths_plan<S_>(m, n, kp, stride, pA, pB, eA, eB, C, ldc, Q, st);
        OZ_CASE(11) OZ_CASE(12) OZ_CASE(13) OZ_CASE(14) OZ_CASE(15) OZ_CASE(16) OZ_CASE(17) OZ_CASE(18) OZ_CASE(19) OZ_CASE(20)
#undef OZ_CASE
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gemm_halves(int s, int m, int n, int kp, const int8_t *pA, const int8_t *pB, const int32_t *eA,
                              const int32_t *eB, double *C, int ldc, int Q, hipStream_t st)
{
    if (m <= 0 || n <= 0) return hipSuccess;
    switch (s) {
#define OZ_CASE(S_) case S_: return launch_halves<S_>(m, n, kp, pA, pB, eA, eB, C, ldc, Q, st);
        OZ_CASE(2) OZ_CASE(3) OZ_CASE(4) OZ_CASE(5) OZ_CASE(6)
#undef OZ_CASE
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gemm_eighths(int s, int m, int n, int kp, const int8_t *pA, const int8_t *pB, const int32_t *eA,
                               const int32_t *eB, double *C, int ldc, int Q, hipStream_t st)
{
    if (m <= 0 || n <= 0) return hipSuccess;
    switch (s) {
#define OZ_CASE(S_) case S_: return launch_eighths<S_>(m, n, kp, pA, pB, eA, eB, C, ldc, Q, st);
        OZ_CASE(1) OZ_CASE(2) OZ_CASE(3) OZ_CASE(4) OZ_CASE(5) OZ_CASE(6) OZ_CASE(7) OZ_CASE(8) OZ_CASE(9) OZ_CASE(10)
#undef OZ_CASE
    }
    return hipErrorInvalidValue;
}

}  // namespace oz
