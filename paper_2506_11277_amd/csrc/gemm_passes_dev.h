// Slice products in passes over groups of diagonals (device code and launcher; the slice counts are instantiated in
// gemm_passes_*.hip, the choice between shapes is in gemm_passes.hip).
//
// From 10 slices on the int32 diagonal sums of a 32 x 32 output block no longer fit the registers of two wavefronts per SIMD
// beside the operands, and a lone wavefront per SIMD leaves its matrix pipe idle at every wait (13 slices, 64 x 64 tile, four
// wavefronts of 512 registers: 2.85-3.0 POP/s), while blocks of slice groups write their int32 sums to memory and read them
// back (18 slices at 4096^3: 0.65 of 7.0 ms).  Here a work-group takes its diagonals in passes, W at a time and in ascending order, over the
// same tile: a pass over diagonals up to SN + 1 runs through the whole contraction with the first SN slices and W accumulator
// sets, adds its W sums to the binary64 result, and leaves that in the work-group's own part of C for the next pass.
// Every pair of slices is multiplied once, all sums stay int32 (s k <= 133144), the order of the binary64 additions is the usual one.
//
// A pass is a convolution: step i of a 64-deep k-step brings slice SN - i of A and slice i + 1 of B (1-based), and product j of the
// step, slice i + 1 - j of B times that of A, belongs to diagonal SN + 1 - j whatever i is.  So A is held for one step, B
// for W steps, each read from LDS once, and each slice of the tile is copied to LDS once per pass.  The slices go through a
// ring of LDS slots, one step (slice of A, slice of B) to a slot, filled by LDS-DMA several steps ahead; a barrier stands about
// every 24 products, when the slots of the steps before it become free.  Small first passes cost least, as the last
// pass moves all s slices whatever its width: (3, 9) rather than (6, 6) for 12 slices (4150 against 4020 TOP/s at 4096^3), but no wider than nine
// diagonals, 144 accumulator registers and 72 of B (two or three registers spill in 128 x 64 tiles with 12, 15, 19 and 20 slices, two in 64 x 64 with 20).  The first pass is a multiple of three where that costs less than two
// percent, so that levels of three diagonals end with it.
//
// 16x16x64 instruction, 32 x 32 outputs per wavefront.  Two shapes: 128 x 64 tile, eight wavefronts, 156 KiB ring, one work-group to a compute
// unit; 64 x 64 tile, four wavefronts, 80 KiB ring, two work-groups to a compute unit, whose first copies and epilogues
// hide behind each other's products: within 4 % of each other in whole rounds of the chip, ahead where the tiles of 128 x 64 leave a round partly filled.
// Int8 TOP/s of the products, before -> 128 x 64 / 64 x 64 (what ran before: gemm_fused_kernel, 18 at 4096^3: blocks; operands badly scaled along k,
// digits in all slices; lognormal ones, none from the 9th slice on, had measured 10 to 15 % lower throughout):
//   4096^3                s = 10 3750 -> - / 3580, 13 3560 -> 4150 / 4070, 16 3810 -> 4240 / 4340, 18 3550 -> 4460 / 4480, 20 3150 -> 4420 / 4360
//   2500 x 2400 x 2500    s = 10 3520 -> - / 3480, 13 3330 -> 3850 / 3840, 16 3590 -> 3970 / 4060, 18 3080 -> 4110 / 4170
//   2207^3                s = 10 3040 -> - / 3290, 13 3210 -> 3090 / 3670, 16 3450 -> 3170 / 3880, 18 2670 -> 3290 / 3990
// 4 ... 9 slices fit one pass; the 64 x 64 tile serves them too where whole rounds of the larger tiles of gemm_fused16_kernel fit
// badly or k is short (s = 7: 2304 x 2000 x 2560 264 -> 228 us, 3000 x 3000 x 500 107 -> 94; s = 9: 6001 x 5200 x 256 299 -> 251).  The
// 128 x 64 tile is then worked on in runs: a work-group takes the tiles b, b + grid, ..., the copies of the next tile's first
// steps follow those of the last stage, and the epilogue stands between them (4096 x 4096 x 1024, s = 8 / 9 387 / 469 us as 64 x 64 tiles, 373 /
// 447 in runs; 64 x 64 tiles gain nothing by runs).
// 96 x 64 tiles, twelve wavefronts of 32 x 16 outputs, three to a SIMD: for 4 ... 9 slices (in runs) and 13 ... 18 where 128 x 64 tiles leave a round partly filled and
// pairs of 64 x 64 ones do too.  A wavefront reads three 16-row operands for two blocks where 32 x 32 reads four for four, so LDS is read
// half as often again (about 0.85 of its cycles with the copies), which costs nothing under the power cap (1536 x 1024 x 8000, s = 7, one whole
// round: 3.13 POP/s) and 10 to 15 percent away from it.  Eight wavefronts of 48 x 16, which read less, were behind: two to a SIMD (1531 x 777 x 1001,
// s = 8: calls 50.6 against 46.4).
// What bounds it: the board's power cap, as the other large products (register-only loop of the same instruction: 4200 TOP/s).
#pragma once
#include "gemm_dev.h"

namespace oz {

namespace {

// Compile-time schedule of one 64-deep k-step ("stage") of a pass: SN slices, the last W diagonals of their reduced set.
// A stage is V >= SN positions of the stream (those from SN on are empty), the ring has N slots, N a divisor or a multiple of V
// so that every slot is a compile-time constant within a stage.
// MF: matrix instructions of a product (16 x 16 blocks of a wavefront).
enum Copies { kCopyBoth, kCopyPair, kCopyOne };
template <int SN, int W, int V, int N, int D, int DB, int TARGET, int COPIES, int MF>
struct PassBase {
    static_assert(V >= SN && (V % N == 0 || N % V == 0));
    static constexpr int used(int i) { return i >= SN ? 0 : i + 1 < W ? i + 1 : W; }      // products of step i
    static constexpr int start(int i)                                       // first matrix instruction of step i
    {
        int e = 0;
        for (int q = 0; q < i; ++q) e += MF * used(q);
        return e;
    }
    static constexpr int NM = start(SN);
    static constexpr int step_of(int e)
    {
        int i = 0;
        while (i + 1 < SN && start(i + 1) <= e) ++i;
        return i;
    }
    // product number p of step i meets B slice of step i - j, j = used - 1 - p
    static constexpr int j_of(int e) { return used(step_of(e)) - 1 - (e - start(step_of(e))) / MF; }
    static constexpr int readA(int i) { return start(i) - D; }
    static constexpr int readB(int i)
    {
        const int need = start(i) + MF * (used(i) - 1);
        return need - DB < start(i) - D ? start(i) - D : need - DB;
    }
    // synchronisations: boundary k = first step that may be read only after it; about TARGET products apart
    struct Bounds {
        int n = 0, b[SN + 1] = {};
    };
    static constexpr int at(const Bounds &r, int k)        // k in -1 ... n: those of the stages before and after included
    {
        return k < 0 ? r.b[k + r.n] - V : k >= r.n ? r.b[k - r.n] + V : r.b[k];
    }
    // copies a wavefront of class c has issued for the steps below q: one of A per step; of B one per step (kCopyBoth), or (kCopyPair: 4 units
    // of B, 8 wavefronts) the even steps by class 0 and the odd ones by class 1, both behind the odd step's copy of A; or one per
    // step, of either operand (kCopyOne)
    static constexpr int count(int q)
    {
        const int st = q >= 0 ? q / V : -((-q + V - 1) / V);
        int i = q - st * V;
        if (i > SN) i = SN;
        const int per = COPIES == kCopyPair ? SN + (SN + 1) / 2 : COPIES == kCopyOne ? SN : 2 * SN;
        if (i == SN) return (st + 1) * per;
        return st * per + (COPIES == kCopyPair ? i + i / 2 : COPIES == kCopyOne ? i : 2 * i);
    }
    static constexpr int flying(const Bounds &r, int k)       // copies that may still be in flight at synchronisation k
    {
        int b = at(r, k + 1);
        const int i = (b + 4 * V) % V, iss = at(r, k - 1) + N;
        if (COPIES == kCopyPair && i % 2 == 1 && i < SN) ++b;         // the even step's B comes with the odd step after it
        return b > iss ? -1 : count(iss) - count(b);
    }
    static constexpr Bounds make()
    {
        for (int most = N / 2; most > 0; --most) {
            Bounds r;
            int sum = 0;
            for (int i = 0; i < SN; ++i) {
                const int c = r.n ? i - r.b[r.n - 1] : 0;
                if (r.n == 0 || sum >= TARGET || c >= most) { r.b[r.n++] = i; sum = 0; }
                sum += used(i);
            }
            bool ok = true;
            for (int k = 0; k < r.n; ++k) ok = ok && flying(r, k) >= 0;
            if (ok) return r;
        }
        return Bounds();
    }
};

template <int SN, int W, int V, int N, int D, int DB, int TARGET, int COPIES, int MF>
struct PassSched : PassBase<SN, W, V, N, D, DB, TARGET, COPIES, MF> {
    using P = PassBase<SN, W, V, N, D, DB, TARGET, COPIES, MF>;
    static constexpr int PARTS = COPIES == kCopyOne ? 1 : 2;
    using P::start, P::used, P::readA, P::readB, P::NM, P::at;
    static constexpr typename P::Bounds BS = P::make();
    static constexpr int NSYNC = BS.n;
    static_assert(NSYNC > 0, "ring too short");
    static constexpr int bound(int k) { return at(BS, k); }
    static constexpr int flying(int k) { return P::flying(BS, k); }
    static constexpr int sync_at(int k) { return readA(bound(k)); }          // k = 0: negative, in the stage before
    static constexpr bool is_sync(int e)
    {
        for (int k = 1; k < NSYNC; ++k) if (sync_at(k) == e) return true;
        return sync_at(0) + NM == e;
    }
    static constexpr int sync_of(int e)      // which one stands before e (0: that of the next stage)
    {
        for (int k = 1; k < NSYNC; ++k) if (sync_at(k) == e) return k;
        return 0;
    }
    static constexpr int issued(int k) { return bound(k - 1) + N; }          // copies issued before synchronisation k: steps below
    static constexpr bool any_event(int e)
    {
        if (is_sync(e)) return true;
        for (int i = 0; i < SN; ++i)
            if (readA(i) == e || readB(i) == e || readA(i) + NM == e || readB(i) + NM == e) return true;
        return false;
    }
    // copy issued behind matrix instruction e: PARTS * step + part, or -1.  The copies of interval k
    // (steps issued(k) ... issued(k + 1) - 1) go one behind each matrix instruction from the start of the interval on.
    static constexpr int from(int k) { return k == 0 ? 0 : sync_at(k); }
    static constexpr int copy_at(int e)
    {
        for (int k = 0; k < NSYNC; ++k) {
            const int n = PARTS * (issued(k + 1) - issued(k)), f = from(k);
            if (e >= f && e < f + n) return PARTS * issued(k) + (e - f);
        }
        return -1;
    }
    static constexpr bool fits()
    {
        for (int k = 0; k < NSYNC; ++k) {
            const int n = PARTS * (issued(k + 1) - issued(k));
            const int end = k + 1 < NSYNC ? sync_at(k + 1) : sync_at(0) + NM;
            if (from(k) + n > end) return false;
        }
        return true;
    }
    static constexpr bool ordered()
    {
        for (int k = 0; k < NSYNC; ++k) {
            if (k > 0 && sync_at(k) < 0) return false;
            for (int i = 0; i < SN; ++i) {
                // every read of a step below the boundary stands before the synchronisation, the others not before it
                const int read = P::readB(i), first = readA(i);
                if (k > 0 && (i < bound(k) ? read >= sync_at(k) : first < sync_at(k))) return false;
                if (k == 0 && (read >= sync_at(0) + NM || first < sync_at(0))) return false;
            }
        }
        return true;
    }
    static_assert(fits(), "too few matrix instructions to issue the copies behind");
    static_assert(ordered(), "a read on the wrong side of a synchronisation");
};

// KG groups of WVM x WVN wavefronts of 32 x 32 outputs (NI = 1: 32 x 16), a ring of at most SLOTS slots to each group; the groups take every
// KG-th 64-deep k-step of the same tile
template <int WVM_, int WVN_, int SLOTS_, int KG_ = 1, bool PERSIST_ = false, int NI_ = 2>
struct PassTile {
    static constexpr bool PERSIST = PERSIST_;
    static constexpr int WVM = WVM_, WVN = WVN_, NI = NI_, NW = WVM * WVN, SLOTS = SLOTS_, KG = KG_, THREADS = 64 * NW * KG;
    static constexpr int FM = WVM, FN = WVN * NI / 2, TM = 32 * FM, TN = 32 * FN;        // fragment rows of A and B, outputs
    static constexpr int COPIES = NW == 4 ? kCopyBoth : NW == 8 ? kCopyPair : kCopyOne;
    static constexpr int UNITS = 2 * (FM + FN), SLOT = UNITS * kFragBytes, GROUP = SLOTS * SLOT, LDS = KG * GROUP;
    static_assert(LDS <= kLdsBytes, "rings do not fit LDS");
};
using PassTileWide = PassTile<4, 2, 13>;       // 128 x 64, 156 KiB
using PassTileRuns = PassTile<4, 2, 13, 1, true>;      // the same for one pass, several tiles to a work-group
using PassTileSmall = PassTile<2, 2, 10>;      // 64 x 64, 80 KiB: two work-groups to a compute unit
using PassTileMiddle = PassTile<3, 4, 16, 1, true, 1>;     // 96 x 64 in runs, twelve wavefronts of 32 x 16, 160 KiB
using PassTileMiddleLone = PassTile<3, 4, 16, 1, false, 1>;        // the same, a work-group to a tile: several passes
// operands are read from LDS this many matrix instructions ahead; products between synchronisations (16 ... 40 products and
// 6 ... 16 instructions are within 1 % of each other at 13 and 18 slices,
// one pass of 8 slices, 64 x 64 tile, 1024 x 1024 x 4096: 104 us with 16, 111 with 24)
// 96 x 64, three wavefronts to a SIMD, 1536 x 1024 x 8000 s = 7: GEMM 240 us with 16 products and 8 instructions, 229 with 24 and 8, 227 with 32 and 10)
constexpr int kPassAhead = 8, kPassProducts = 24, kPassProductsOne = 16, kPassAheadMiddle = 10, kPassProductsMiddle = 32;

// positions of a stage and slots of the ring: whole stages in the ring or two rings in a stage
template <int SN, int SLOTS>
struct PassRing {
    static constexpr int V = SN <= SLOTS ? SN : SN + SN % 2;
    static constexpr int N = SN <= SLOTS ? SLOTS / SN * SN : V / 2;
    static_assert(N <= SLOTS, "ring too large");
};

template <int NP>
constexpr int widest(const int (&w)[NP])
{
    int r = 0;
    for (int q = 0; q < NP; ++q) r = w[q] > r ? w[q] : r;
    return r;
}

template <class T, int... Ws>
__device__ __forceinline__ void passes_of_a_tile(const int8_t *__restrict__ pA, const int8_t *__restrict__ pB,
                                                 const int32_t *__restrict__ eA, const int32_t *__restrict__ eB,
                                                 double *__restrict__ C, int ldc, int m, int n, int KB, int stride,
                                                 int tiles_m, int tiles_n, int Q)
{
    constexpr int WVM = T::WVM, NW = T::NW, NI = T::NI, MF = 2 * NI, FM = T::FM, FN = T::FN, SLOT = T::SLOT, KG = T::KG;
    constexpr bool PERSIST = T::PERSIST;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_all[];
    // (several tiles to a work-group: those of the blocks b, b + gridDim.x, ...)
    unsigned b = blockIdx.x;
    const unsigned blocks = PERSIST ? (unsigned)tile_order_blocks(tiles_m, tiles_n, false) : 0;
    int tm, tn;
    auto next_tile = [&]() {
        for (; b < blocks; b += gridDim.x)
            if (tile_of_block_xcd(b, tiles_m, tiles_n, false, tm, tn)) return true;
        return false;
    };
    if (PERSIST ? !next_tile() : !tile_of_block_xcd(b, tiles_m, tiles_n, false, tm, tn)) return;
    const int lane = threadIdx.x & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = KG == 1 ? 0 : wave_all / NW, wave = wave_all - kg * NW;
    unsigned char *const lds = lds_all + kg * T::GROUP;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
    const int wm = wave % WVM, wn = wave / WVM;
    const size_t row_bytes = (size_t)KB * ((size_t)stride * kFragBytes);
    const unsigned STG = 2u * stride * kFragBytes;       // bytes of a stage in a fragment row of the planes
    const int nst = KB / 2 / KG;                         // stages of a group (KB is a multiple of four)
    // Copies of a step: its slice of the WVM fragment rows of A, two k-halves each, one 1 KiB unit to a wavefront; of the
    // two fragment rows of B likewise, four units, so eight wavefronts (PAIR) copy two steps at a time, wavefronts of
    // class 0 the even step's and of class 1 the odd one's (the last step of an odd number: both the same).
    // 96 x 64: six units of A and four of B for twelve wavefronts, one each (ONE); two have none and copy with no lane active.
    constexpr bool PAIR = T::COPIES == kCopyPair, ONE = T::COPIES == kCopyOne;
    static_assert((NW == 8 && FM == 4 && FN == 2) || (NW == 4 && FM == 2 && FN == 2) || (ONE && T::UNITS <= NW), "units per wavefront");
    const int cls = wave >> 2, ub = wave & 3;            // (four wavefronts: class 0)
    const bool unitA = !ONE || wave < 2 * FM;            // (ONE: this wavefront's unit is one of A)
    const unsigned lanes = (unsigned)((wave - T::UNITS) >> 31);     // (ONE: all ones where there is one)
    // (the last tile of 96 rows may reach beyond the planes, which end at a multiple of 128: its rows there repeat the last ones)
    const int rowsA = (m + kPad - 1) / kPad * (kPad / kFrag);
    auto unit_row = [&](int tm_, int tn_) -> unsigned {   // ONE: fragment row of this wavefront's unit
        const int a = tm_ * FM + (wave >> 1), b = tn_ * FN + ((wave - 2 * FM) >> 1 & (FN - 1));
        return unitA ? (a < rowsA ? a : rowsA - 1) : b;
    };
    const int8_t *srcA = pA + (size_t)((PERSIST ? 0 : tm * FM) + (wave >> 1)) * row_bytes + (size_t)((wave & 1) * stride) * kFragBytes;
    const int8_t *srcB = pB + (size_t)((PERSIST ? 0 : tn * FN) + (ub >> 1)) * row_bytes + (size_t)((ub & 1) * stride + cls) * kFragBytes;
    const unsigned dstA = lds0 + wave * kFragBytes, dstB = lds0 + (2 * FM + ub) * kFragBytes;
    const unsigned dstB2 = dstB + cls * SLOT;            // (from the even step's slot to this class's)
    if constexpr (ONE) srcA = (unitA ? pA : pB) + (size_t)((wave & 1) * stride) * kFragBytes;
    const unsigned lane16 = lane * 16;
    // (PERSIST: the tile is in the lane offset, 32 bits; behind the last stage come the first ones of the next tile)
    unsigned tileA = ONE ? unit_row(tm, tn) * (unsigned)row_bytes : PERSIST ? (unsigned)(tm * FM) * (unsigned)row_bytes : 0;
    unsigned tileB = PERSIST ? (unsigned)(tn * FN) * (unsigned)row_bytes : 0;
    unsigned nextA = 0, nextB = 0;
    bool more = false;
    auto stage_off = [&](int st, unsigned tile, unsigned next) {
        if (PERSIST && more && st >= nst) return lane16 + next + (unsigned)(st - nst) * STG;
        return lane16 + tile + (unsigned)((st < nst ? st : nst - 1) * KG + kg) * STG;
    };
    // this lane's part of a 16 x 64 operand in a pair of 32 x 32 fragments, as in gemm_fused16_kernel
    const int lofs = ((lane >> 4) >> 1) * kFragBytes + ((lane & 15) + 32 * ((lane >> 4) & 1)) * 16;
    const unsigned char *ldsA = lds + wm * 2 * kFragBytes + lofs, *ldsB = lds + (FM + wn * NI / 2) * 2 * kFragBytes + (NI == 1 ? (wn & 1) * 256 : 0) + lofs;

    constexpr int NP = sizeof...(Ws);
    constexpr int WS[NP] = {Ws...};
    v4i acc[widest<NP>(WS)][MF];                         // [diagonal of the pass, the last one first][16 x 16 block (i2, j2)]

    static_assert(KG == 1 || (KG == 2 && NP == 1), "k in halves: one pass");
    static_assert(!PERSIST || (KG == 1 && NP == 1), "several tiles: one pass");
    // k in halves: a group finishes the blocks of i2 = kg and hands the others over, through LDS nobody else uses any more
    auto exchange = [&]() {
        constexpr int W = WS[0];
        static_assert(KG == 1 || W * NW * 2 * 2 * 1024 <= T::LDS, "exchange does not fit LDS");
        v4i *x = (v4i *)lds_all + wave * (W * 2 * 2 * 64) + lane;          // [diagonal][i2][j2]
#pragma unroll
        for (int a = 0; a < W; ++a)
#pragma unroll
            for (int j2 = 0; j2 < 2; ++j2) x[((a * 2 + (kg ^ 1)) * 2 + j2) * 64] = kg ? acc[a][j2] : acc[a][2 + j2];
        __syncthreads();
#pragma unroll
        for (int a = 0; a < W; ++a)
#pragma unroll
            for (int j2 = 0; j2 < 2; ++j2) acc[a][j2] = (kg ? acc[a][2 + j2] : acc[a][j2]) + x[((a * 2 + kg) * 2 + j2) * 64];
    };
    int m0 = (tm * FM + wm) * 32, n0 = tn * T::TN + wn * 16 * NI;
    // (one pass: the exponents of the 32 rows and columns are asked for here, a value per lane, and not where a lone tile
    // would wait for them)
    constexpr bool EARLY = NP == 1;
    int early = 0;
    auto ask = [&]() {                                   // (padded like the planes)
        const int ma = FM % 4 == 0 || FM == 2 || m0 + lane < rowsA * kFrag ? m0 + lane : 0;
        early = lane < 32 ? eA[ma] : eB[n0 + ((lane - 32) & (16 * NI - 1))];
    };
    if constexpr (EARLY) ask();
    // Adds the sums of pass p to the entries, in C as they are so far (not yet scaled) between passes.
    const bool stream = stream_c(C, ldc);
    auto finish = [&](auto PP) {
        constexpr int p = decltype(PP)::value, W = WS[p], BEFORE = diagonals_before<NP>(WS, p);
        auto entries = [&](auto ORDER, auto STREAM) {
#pragma unroll
            for (int i2 = 0; i2 < 2 / KG; ++i2) {
                const int mi = m0 + (KG == 1 ? i2 : kg) * 16 + (lane & 15);
                int ea = 0, eb[2][4];
                if constexpr (EARLY) {                   // (before lanes beyond the edge leave)
                    ea = __shfl(early, (KG == 1 ? i2 : kg) * 16 + (lane & 15));
#pragma unroll
                    for (int q = 0; q < 4 * NI; ++q) eb[q >> 2][q & 3] = __shfl(early, 32 + (q >> 2) * 16 + 4 * (lane >> 4) + (q & 3));
                }
                if (mi >= m) continue;
                if constexpr (!EARLY && p + 1 == NP) ea = eA[mi];
#pragma unroll
                for (int j2 = 0; j2 < NI; ++j2)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int nj = n0 + j2 * 16 + 4 * (lane >> 4) + r;
                        if (nj >= n) continue;
                        double *c = &C[mi + (size_t)nj * ldc];
                        LevelSum sum;                    // (a pass ends with a level: launch_passes)
                        if constexpr (p > 0) sum.S = *c;
#pragma unroll
                        for (int a = 0; a < W; ++a) {
                            const double unit = __builtin_ldexp(1.0, -kSliceBits * (BEFORE + a + 2));
                            const int d = acc[W - 1 - a][i2 * NI + j2][r];
                            if constexpr (ORDER.value == kPlainOrder) sum.S = __builtin_fma((double)d, unit, sum.S);
                            else sum.add((double)d * unit, Q, a == W - 1);
                        }
                        if constexpr (p + 1 < NP) *c = sum.S;
                        else store_c(c, ldexp(sum.S, ea + (EARLY ? eb[j2][r] : eB[nj])), STREAM);
                    }
            }
        };
        if constexpr (p + 1 == NP) epilogue_variant<W>(Q, stream, entries);
        else if (Q == 1) entries(std::integral_constant<int, kPlainOrder>{}, false);
        else entries(std::integral_constant<int, kLevels>{}, false);
    };

    static_for<0, NP>([&](auto PP) {
        constexpr int p = decltype(PP)::value, W = WS[p], SN = diagonals_before<NP>(WS, p) + W;
        using G = PassRing<SN, T::SLOTS>;
        constexpr int V = G::V, N = G::N, R = N > V ? N / V : 1;         // (R: stages in the ring)
        constexpr int AHEAD = ONE ? kPassAheadMiddle : kPassAhead;
        using S = PassSched<SN, W, V, N, AHEAD, AHEAD, ONE ? kPassProductsMiddle : NP == 1 ? kPassProductsOne : kPassProducts, T::COPIES, MF>;
        constexpr int NM = S::NM;
        const int8_t *sA[SN], *sB[SN], *sBlast = srcB + (SN - 1 - cls) * kFragBytes;
#pragma unroll
        for (int i = 0; i < SN; ++i) {
            sA[i] = srcA + (SN - 1 - i) * kFragBytes;
            sB[i] = srcB + (PAIR && i % 2 ? i - 1 : i) * kFragBytes;
            if constexpr (ONE) sA[i] = srcA + (unitA ? SN - 1 - i : i) * kFragBytes;
        }
        // Copies of position q of the stream, counted from the start of a stage whose slots begin at `ring`; voff: lane and stage.
        auto copyA = [&](auto QQ, unsigned voff, unsigned ring) {
            constexpr int q = decltype(QQ)::value, i = q % V;
            constexpr int to = (q % (R > 1 ? V : N)) * SLOT;
            if constexpr (i < SN && ONE) lds_dma16_masked_at<to>(sA[i], voff, dstA + ring, lanes);
            else if constexpr (i < SN) lds_dma16_at<to>(sA[i], voff, dstA + ring);
        };
        auto copyB = [&](auto QQ, unsigned voff, unsigned ring) {
            constexpr int q = decltype(QQ)::value, i = q % V, slot = q % (R > 1 ? V : N);
            if constexpr (i >= SN || ONE) return;
            else if constexpr (!PAIR) lds_dma16_at<slot * SLOT>(sB[i], voff, dstB + ring);
            else if constexpr (i % 2 == 1) {
                static_assert(slot > 0 || R == 1, "pair across the end of the ring");
                if constexpr (slot > 0) lds_dma16_at<(slot - 1) * SLOT>(sB[i], voff, dstB2 + ring);
                else lds_dma16_at<0>(sB[i], voff, cls ? dstB : dstB + (N - 1) * SLOT);
            } else if constexpr (i == SN - 1) lds_dma16_at<slot * SLOT>(sBlast, voff, dstB + ring);
        };
        static_assert(S::issued(0) > 0 && S::issued(0) <= N, "first copies");
        static_for<0, S::issued(0)>([&](auto QQ) {
            constexpr int q = decltype(QQ)::value;
            copyA(QQ, stage_off(q / V, tileA, 0), q / V * (V * SLOT));
            copyB(QQ, stage_off(q / V, tileB, 0), q / V * (V * SLOT));
        });
        if constexpr (p > 0) finish(std::integral_constant<int, p - 1>{});         // (the copies land meanwhile)
        auto clear = [&]() {
#pragma unroll
            for (int a = 0; a < W; ++a)
#pragma unroll
                for (int q = 0; q < MF; ++q) acc[a][q] = v4i{0, 0, 0, 0};
        };
        clear();

        v4i A_[SN][2], B_[SN][NI], An[SN][2], Bn[SN][NI];       // (An, Bn: of the next stage)
        auto loadA = [&](v4i (&d)[2], int i, unsigned ring) {
#pragma unroll
            for (int i2 = 0; i2 < 2; ++i2) d[i2] = *(const v4i *)(ldsA + ring + (i % (R > 1 ? V : N)) * SLOT + i2 * 256);
        };
        auto loadB = [&](v4i (&d)[NI], int i, unsigned ring) {
#pragma unroll
            for (int j2 = 0; j2 < NI; ++j2) d[j2] = *(const v4i *)(ldsB + ring + (i % (R > 1 ? V : N)) * SLOT + j2 * 256);
        };
        wait_vmcnt<S::flying(0)>();
        __syncthreads();
        static_for<0, SN>([&](auto I) {
            constexpr int i = decltype(I)::value;
            if constexpr (S::readA(i) < 0) loadA(A_[i], i, 0);
            if constexpr (S::readB(i) < 0) loadB(B_[i], i, 0);
        });
        unsigned ring = 0;                                   // LDS offset of the stage's first slot
        int mn = 0, nn = 0;
        auto look_ahead = [&]() {
            b += gridDim.x;
            if (!(more = next_tile())) return;
            nextA = (ONE ? unit_row(tm, tn) : (unsigned)(tm * FM)) * (unsigned)row_bytes;
            nextB = (unsigned)(tn * FN) * (unsigned)row_bytes;
            mn = (tm * FM + wm) * 32;
            nn = tn * T::TN + wn * 16 * NI;
        };
        if constexpr (PERSIST) look_ahead();
        for (int st = 0; st < nst; ++st) {
            // (towards the end the copies and the reads ahead go on, of the last stage again -- nobody uses them -- or of the
            // first stages of the next tile)
            constexpr int DA = (V - 1 + N) / V + 1;
            unsigned so[DA + 1], sb[DA + 1], rg[DA + 1];
#pragma unroll
            for (int d = 0; d <= DA; ++d) {
                so[d] = stage_off(st + d, tileA, nextA);
                sb[d] = PERSIST ? stage_off(st + d, tileB, nextB) : so[d];
                rg[d] = R == 1 ? 0u : d == 0 ? ring : rg[d - 1] + V * SLOT == N * SLOT ? 0u : rg[d - 1] + V * SLOT;
            }
            static_for<0, NM>([&](auto E) {
                constexpr int e = decltype(E)::value;
                constexpr int i = S::step_of(e), j = S::j_of(e), b = e % MF, i2 = b / NI, j2 = b % NI;
                if constexpr (S::any_event(e)) {
                    __builtin_amdgcn_sched_barrier(0);       // (the compiler moves no read or product across)
                    if constexpr (S::is_sync(e)) {
                        wait_vmcnt<S::flying(S::sync_of(e))>();
                        __syncthreads();
                    }
                    static_for<0, SN>([&](auto II) {
                        constexpr int ii = decltype(II)::value;
                        if constexpr (S::readA(ii) == e) loadA(A_[ii], ii, rg[0]);
                        if constexpr (S::readA(ii) + NM == e) loadA(An[ii], ii, rg[1]);
                        if constexpr (S::readB(ii) == e) loadB(B_[ii], ii, rg[0]);
                        if constexpr (S::readB(ii) + NM == e) loadB(Bn[ii], ii, rg[1]);
                    });
                    __builtin_amdgcn_sched_barrier(0);
                }
                acc[j][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(B_[i - j][j2], A_[i][i2], acc[j][b], 0, 0, 0);
                constexpr int cp = S::copy_at(e);
                if constexpr (cp >= 0) {
                    constexpr int q = cp / S::PARTS;
                    if constexpr (cp % S::PARTS == 0) copyA(std::integral_constant<int, q>{}, so[q / V], rg[q / V]);
                    else copyB(std::integral_constant<int, q>{}, sb[q / V], rg[q / V]);
                }
            });
            static_for<0, SN>([&](auto I) {
                constexpr int i = decltype(I)::value;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if constexpr (S::readA(i) < 0) A_[i][h] = An[i][h];
                    if constexpr (S::readB(i) < 0) if (h < NI) B_[i][h] = Bn[i][h];
                }
            });
            ring = rg[1];
            if constexpr (PERSIST)
                if (st + 1 == nst && more) {
                    // the tile is done: its epilogue while the first copies of the next one fly
                    finish(PP);
                    clear();
                    tileA = nextA;
                    tileB = nextB;
                    m0 = mn;
                    n0 = nn;
                    ask();
                    look_ahead();
                    st = -1;
                }
        }
        // no copy is in flight and nobody reads when the next pass begins to fill the ring
        wait_vmcnt<0>();
        if constexpr (p + 1 < NP || KG > 1) __syncthreads();
    });
    if constexpr (KG > 1) exchange();
    finish(std::integral_constant<int, NP - 1>{});
}

template <class T, int... Ws>
__global__ __launch_bounds__(T::THREADS, T::NW == 12 ? 3 : 2) void gemm_passes_kernel(
    const int8_t *__restrict__ pA, const int8_t *__restrict__ pB, const int32_t *__restrict__ eA,
    const int32_t *__restrict__ eB, double *__restrict__ C, int ldc, int m, int n, int KB, int stride, int tiles_m,
    int tiles_n, int Q)
{
    passes_of_a_tile<T, Ws...>(pA, pB, eA, eB, C, ldc, m, n, KB, stride, tiles_m, tiles_n, Q);
}

// hipErrorInvalidValue: a level of Q diagonals would straddle two passes
template <class T, int... Ws>
hipError_t launch_passes(int m, int n, int kp, int stride, const int8_t *pA, const int8_t *pB, const int32_t *eA,
                         const int32_t *eB, double *C, int ldc, int Q, hipStream_t st)
{
    // (32-bit lane offsets to the tile where a work-group takes several: larger planes go to a launch of single tiles; 96 x 64 tiles have no
    // other way and the choice of shape does not ask for them)
    const bool far = (size_t)(m > n ? round_up(m, kPad) : round_up(n, kPad)) * kp * stride >= (1ULL << 32);
    if constexpr (T::COPIES == kCopyOne) {
        if (far) return hipErrorInvalidValue;
    } else if constexpr (T::PERSIST)
        if (far) return launch_passes<PassTile<T::WVM, T::WVN, T::SLOTS>, Ws...>(m, n, kp, stride, pA, pB, eA, eB, C, ldc, Q, st);
    constexpr int TM = T::TM, TN = T::TN, NP = sizeof...(Ws), WS[NP] = {Ws...};
    for (int p = 1; p < NP; ++p)
        if (diagonals_before<NP>(WS, p) % Q != 0) return hipErrorInvalidValue;      // (gemm_passes_shape() does not ask for it)
    auto kern = gemm_passes_kernel<T, Ws...>;
    static std::atomic<unsigned long long> configured{0};
    if (hipError_t e = allow_dynamic_lds((const void *)kern, T::LDS, configured); e != hipSuccess) return e;
    const int tiles_m = (m + TM - 1) / TM, tiles_n = (n + TN - 1) / TN;
    note_gemm_kernel("gemm_passes_kernel<%d> tile %dx%d, %d pass%s", (Ws + ...), TM, TN, NP, NP == 1 ? "" : "es");
    long long blocks = tile_order_blocks(tiles_m, tiles_n, false);
    if (T::PERSIST) {
        const long long slots = (long long)device_cus() * (T::NW == 4 ? 2 : 1);
        // (behind the last stage of a tile the ring is filled with the first ones of the next: a contraction is as long as the ring)
        if (blocks > slots && kp / 64 < PassRing<WS[0], T::SLOTS>::N / PassRing<WS[0], T::SLOTS>::V) return hipErrorInvalidValue;
        blocks = blocks < slots ? blocks : slots;
    }
    kern<<<(unsigned)blocks, T::THREADS, T::LDS, st>>>(pA, pB, eA, eB, C, ldc, m, n, kp / kFrag, stride,
                                                                                    tiles_m, tiles_n, Q);
    return hipGetLastError();
}

}  // namespace

// launch_gemm_passes_<S>: one slice count of the table
template <class T, int S>
hipError_t launch_pass_plan(int m, int n, int kp, int stride, const int8_t *pA, const int8_t *pB, const int32_t *eA,
                            const int32_t *eB, double *C, int ldc, int Q, hipStream_t st)
{
    constexpr PassPlan P = pass_plan(S);
    if constexpr (P.n == 1) return launch_passes<T, S>(m, n, kp, stride, pA, pB, eA, eB, C, ldc, Q, st);
    else if constexpr (P.n == 2) return launch_passes<T, P.w[0], P.w[1]>(m, n, kp, stride, pA, pB, eA, eB, C, ldc, Q, st);
    else return launch_passes<T, P.w[0], P.w[1], P.w[2]>(m, n, kp, stride, pA, pB, eA, eB, C, ldc, Q, st);
}
#define OZ_DEFINE_GEMM_PASSES(S_)                                                                                           \
    hipError_t launch_gemm_passes_##S_(PassShape shape, int m, int n, int kp, int stride, const int8_t *pA, const int8_t *pB,    \
                                       const int32_t *eA, const int32_t *eB, double *C, int ldc, int Q, hipStream_t st)     \
    {                                                                                                                       \
        if (shape == kPassSmall) return launch_pass_plan<PassTileSmall, S_>(m, n, kp, stride, pA, pB, eA, eB, C, ldc, Q, st); \
        if constexpr (S_ <= 9 || (S_ >= 13 && S_ <= 18))                                                                    \
            if (shape == kPassMiddle)                                                                                       \
                return launch_pass_plan<std::conditional_t<(S_ >= 10), PassTileMiddleLone, PassTileMiddle>, S_>(m, n, kp, stride, pA, pB, eA, eB, C, ldc, Q, st); \
        using Wide = std::conditional_t<(S_ >= 10), PassTileWide, PassTileRuns>;                                            \
        if constexpr (S_ == 10) return hipErrorInvalidValue;                   /* (nowhere ahead: gemm_passes_shape) */     \
        else return launch_pass_plan<Wide, S_>(m, n, kp, stride, pA, pB, eA, eB, C, ldc, Q, st);                            \
    }

}  // namespace oz
