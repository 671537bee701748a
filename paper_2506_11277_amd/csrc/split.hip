// Bit-splitting of a binary64 matrix into s signed 7-bit slices (Sect. 3, eq.
// (bit-splitting-alg) in its bit-level reading: slice l holds bits (l-1)t+1 .. lt of
// |x| / 2^e after the binary point, and carries the sign of x).
//
// The kernels of the MFMA layout take four entries at a time through windows of nine (eight) slices formed with exact
// binary64 operations (slice_dev.h).  The plain layout, a utility, is cut entry by entry in integers:
// |x| = I * 2^q with I the integer significand, so  floor(|x| 2^{lt - e}) mod 2^t  is a
// shift of I by (e - q - lt) places and a mask.
//
// Round-to-nearest variant (second tweak of the "Enhanced algorithm" paragraph of Sect. 3): the block
// scale is 2^{e+1}, and with R_l = the integer nearest to |x| 2^{7l - e - 1} (ties to even) slice l is
// sign(x) (R_l - 128 R_{l-1}), a value in [-64, 64].  R_l = floor(.) + c_l with the round-up decision
//     c_l = guard & (sticky | lsb)
// on the bits below the cut, so  slice l = field_l + c_l - 128 c_{l-1};  c_l is carried from one slice to the next.
//
// The MFMA layout written here is the one the GEMM kernel reads (see include/ozimmu.h):
// fragments of 32 (R) x 32 (K) bytes, 16 contiguous K-bytes per wavefront lane.
#include "slice_dev.h"

namespace oz {

namespace {

struct Elem {
    unsigned long long I;   // integer significand
    int base;               // e - q : right shift that would bring bit position 0 (the binary point) to bit 0
    int neg;
};

__device__ __forceinline__ Elem decompose(unsigned long long bits, int e)
{
    Elem el;
    const int E = (int)((bits >> 52) & 0x7ff);
    const unsigned long long f = bits & 0xfffffffffffffULL;
    el.I = E ? (f | (1ULL << 52)) : f;
    el.base = e - ((E ? E : 1) - 1075);
    el.neg = (int)(bits >> 63);
    return el;
}

// slice l (1-based), as an unsigned byte holding the two's complement int8
__device__ __forceinline__ unsigned int slice_byte(const Elem &el, int l)
{
    const int sh = el.base - kSliceBits * l;
    unsigned long long v;
    if (sh >= 64) v = 0;
    else if (sh >= 0) v = el.I >> sh;
    else if (sh <= -kSliceBits) v = 0;
    else v = el.I << (-sh);
    int d = (int)(v & 127ULL);
    d = el.neg ? -d : d;
    return (unsigned int)d & 0xffu;
}

// slice l by round-to-nearest (el.base taken from the biased exponent e + 1).  `carry` is bit `bit` of a
// per-lane mask: on entry c_{l-1}, on exit c_l (the caller walks l = 1, 2, ... with the mask cleared first:
// c_0 = 0 because |x| 2^{-e-1} < 1/2).
template <bool NEAREST>
__device__ __forceinline__ unsigned int slice_of(const Elem &el, int l, unsigned int &carry, int bit)
{
    if (!NEAREST) return slice_byte(el, l);
    const int sh = el.base - kSliceBits * l;      // bits of I below the cut
    int field, c = 0;
    if (sh > 64) field = 0;                       // I < 2^53 lies below half a unit
    else if (sh >= 1) {
        const unsigned long long t = el.I >> (sh - 1);            // guard bit at bit 0, the slice above it
        const unsigned int lo = (unsigned int)t;
        const bool sticky = (t << (sh - 1)) != el.I;
        field = (int)((lo >> 1) & 127u);
        c = (int)(lo & 1u) & ((int)sticky | (int)((lo >> 1) & 1u));
    } else if (sh > -kSliceBits) field = (int)((el.I << (-sh)) & 127ULL);   // nothing below the cut
    else field = 0;
    int d = field + c - 128 * (int)((carry >> bit) & 1u);
    carry = (carry & ~(1u << bit)) | ((unsigned int)c << bit);
    d = el.neg ? -d : d;
    return (unsigned int)d & 0xffu;
}

// ---- side 'A': X is R x K column-major (R contiguous).  lane <-> row, each lane walks 16
//      consecutive k, so the 16 K-bytes of a lane come out of registers: the transposition to
//      K-contiguous fragments costs nothing, reads are 512 B per wavefront load, writes are
//      512 B contiguous per half wavefront.
template <bool NEAREST>
__device__ __forceinline__ void split_rows_block(int bx, int by, const unsigned long long *__restrict__ X, int ldx,
                                                 int R, int K, int s, int cs, const int32_t *__restrict__ exps,
                                                 int8_t *__restrict__ planes, int KB,
                                                 const unsigned long long *__restrict__ maxbits = nullptr,
                                                 int32_t *__restrict__ exps_out = nullptr)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r = bx * 64 + lane;
    const int k0 = by * 64 + w * 16;
    // (maxbits given: the exponent comes from the row's maximum, biased by one for nearest slices, and the
    // work-groups of the first k-block store it, zero for the padding rows)
    const int e = r >= R ? 0 : maxbits ? exponent_above(maxbits[r]) + (NEAREST ? 1 : 0) : exps[r];
    if (exps_out && by == 0 && w == 0) exps_out[r] = e;
    Quad<NEAREST> el[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        unsigned long long bits[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int kk = k0 + 4 * q + i;
            bits[i] = (r < R && kk < K) ? X[r + (size_t)kk * ldx] : 0ULL;
        }
        el[q].load(bits, e);
    }
    const int rb = r >> 5, kb = k0 >> 5, half = (k0 >> 4) & 1;
    // (the planes hold cs >= s slices per entry; those beyond s are zeros)
    uint4 *dst = (uint4 *)(planes + ((size_t)rb * KB + kb) * (size_t)cs * kFragBytes) + ((r & 31) + 32 * half);
    for (int l = s + 1; l <= cs; ++l) dst[(size_t)(l - 1) * (kFragBytes / 16)] = make_uint4(0, 0, 0, 0);
    for_each_slice<NEAREST, 4>(el, s, [&](int l, const unsigned (&wd)[4]) {
        dst[(size_t)(l - 1) * (kFragBytes / 16)] = make_uint4(wd[0], wd[1], wd[2], wd[3]);
    });
}

// ---- side 'B': X is K x R column-major (K contiguous).  A work-group takes 32 columns x 128 k;
//      lanes read along k (coalesced), slice bytes are packed four k at a time into LDS rows,
//      then re-read so that lane <-> column and a wavefront emits whole 1 KiB fragments.
constexpr int kColTileK = 128;
constexpr int kColLdsRow = kColTileK + 16;   // bytes per (slice, column) row in LDS
constexpr int kColGroup = 8;                 // slices per LDS pass

template <bool NEAREST>
__global__ __launch_bounds__(256) void split_rows_kernel(const unsigned long long *__restrict__ X, int ldx, int R,
                                                         int K, int s, const int32_t *__restrict__ exps,
                                                         int8_t *__restrict__ planes, int KB)
{
    split_rows_block<NEAREST>(blockIdx.x, blockIdx.y, X, ldx, R, K, s, s, exps, planes, KB);
}

template <bool NEAREST>
__device__ __forceinline__ void split_cols_block(int bx, int by, const unsigned long long *__restrict__ X, int ldx,
                                                 int R, int K, int s, int cs, const int32_t *__restrict__ exps,
                                                 int8_t *__restrict__ planes, int KB,
                                                 const unsigned long long *__restrict__ maxbits = nullptr,
                                                 int32_t *__restrict__ exps_out = nullptr)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[kColGroup * 32 * kColLdsRow];
    const int t = threadIdx.x;
    const int j0 = bx * 32, k0 = by * kColTileK;
    const int kq = (t & 31) * 4;
    Quad<NEAREST> el[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int jj = p * 8 + (t >> 5);
        const int j = j0 + jj;
        const int e = j >= R ? 0 : maxbits ? exponent_above(maxbits[j]) + (NEAREST ? 1 : 0) : exps[j];
        if (exps_out && by == 0 && (t & 31) == 0) exps_out[j] = e;
        unsigned long long bits[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int kk = k0 + kq + i;
            bits[i] = (j < R && kk < K) ? X[kk + (size_t)j * ldx] : 0ULL;
        }
        el[p].load(bits, e);
    }
    const int jj2 = t & 31, ch = t >> 5;                    // phase 2: column, 16-byte chunk along k
    const int rb = j0 >> 5;
    const int kb = (k0 + ch * 16) >> 5, half = ch & 1;
    uint4 *dst = (uint4 *)(planes + ((size_t)rb * KB + kb) * (size_t)cs * kFragBytes) + (jj2 + 32 * half);
    for (int l = s + 1; l <= cs; ++l) dst[(size_t)(l - 1) * (kFragBytes / 16)] = make_uint4(0, 0, 0, 0);
    // kColGroup slices at a time go through LDS (a window of nine slices is two groups)
    auto drain = [&](int l) {                               // slices l - (l - 1) % kColGroup ... l are in LDS
        const int nl = (l - 1) % kColGroup + 1;
        __syncthreads();
        for (int dl = 0; dl < nl; ++dl) {
            uint4 v = *(const uint4 *)(lds + ((size_t)dl * 32 + jj2) * kColLdsRow + ch * 16);
            dst[(size_t)(l - nl + dl) * (kFragBytes / 16)] = v;
        }
        __syncthreads();
    };
    for_each_slice<NEAREST, 4>(el, s, [&](int l, const unsigned (&wd)[4]) {
        const int dl = (l - 1) % kColGroup;
#pragma unroll
        for (int p = 0; p < 4; ++p) *(unsigned int *)(lds + ((size_t)dl * 32 + p * 8 + (t >> 5)) * kColLdsRow + kq) = wd[p];
        if (dl == kColGroup - 1 || l == s) drain(l);
    });
}

template <bool NEAREST>
__global__ __launch_bounds__(256) void split_cols_kernel(const unsigned long long *__restrict__ X, int ldx, int R,
                                                         int K, int s, const int32_t *__restrict__ exps,
                                                         int8_t *__restrict__ planes, int KB)
{
    split_cols_block<NEAREST>(blockIdx.x, blockIdx.y, X, ldx, R, K, s, s, exps, planes, KB);
}

// Both operands in one launch: the first nblkA work-groups slice A (numbered rows-block fastest), the others B.
template <bool NEAREST>
__global__ __launch_bounds__(256) void split_both_kernel(const unsigned long long *__restrict__ A, int lda, int m,
                                                         const unsigned long long *__restrict__ B, int ldb, int n, int K,
                                                         int sA, int sB, int cA, int cB,
                                                         const unsigned long long *__restrict__ maxA,
                                                         const unsigned long long *__restrict__ maxB,
                                                         int32_t *__restrict__ eA, int32_t *__restrict__ eB,
                                                         int8_t *__restrict__ pA, int8_t *__restrict__ pB, int KB,
                                                         int gxA, int nblkA, int gxB)
{
    const int b = blockIdx.x;
    if (b < nblkA) split_rows_block<NEAREST>(b % gxA, b / gxA, A, lda, m, K, sA, cA, nullptr, pA, KB, maxA, eA);
    else split_cols_block<NEAREST>((b - nblkA) % gxB, (b - nblkA) / gxB, B, ldb, n, K, sB, cB, nullptr, pB, KB, maxB, eB);
}

// ---- scales and slices of both operands in one launch, for contractions short enough that a work-group keeps its
// part of the operand in registers between the two.  A work-group owns PR rows of A (columns of B) over all of k, so
// their maxima need no atomics, nothing has to be cleared beforehand, and the operand is read once: one launch takes the
// place of three (clear, reduce, slice), with their event overhead 30.8 -> 21.5 us at 1024^3, s = 7, 19.7 -> 11.8 us at 128^3.
//
// A lane holds quads, four consecutive k of a row; a wavefront takes PR rows x 16 (16 / PR) k at a time, up to 16
// wavefronts share k.  The work-group's PR rows are a part of the 16 rows of a cache line of A: the work-groups of one
// line run on the same XCD, one after the other in launch order.  The four bytes a lane has of a slice make up PR * 16
// contiguous bytes of the fragment with those of its neighbours.
// bad[b] != 0: work-group b has met a NaN or an infinity (the maximum of the bit patterns shows it).
template <bool NEAREST, int PR, int NV, bool THROUGH>
__global__ __launch_bounds__(1024) void scale_split_kernel(const unsigned long long *__restrict__ A, int lda, int m,
                                                           const unsigned long long *__restrict__ B, int ldb, int n, int K,
                                                           int sA, int sB, int cA, int cB, int32_t *__restrict__ eA,
                                                           int32_t *__restrict__ eB, int8_t *__restrict__ pA,
                                                           int8_t *__restrict__ pB, int KB, int panelsA,
                                                           unsigned long long *__restrict__ header, int panels,
                                                           long long bad_offset, unsigned *__restrict__ bad)
{
    constexpr int CW = 16 / PR;                             // groups of 16 k a wavefront takes at a time
    __shared__ unsigned long long smx[16][PR];
    // (work-groups are dealt round-robin to the 8 XCDs: each XCD takes neighbouring panels, which share cache lines)
    const int panel = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    if (panel >= panels) return;
    const bool isB = panel >= panelsA;
    const int R0 = PR * (panel - (isB ? panelsA : 0));
    const unsigned long long *X = isB ? B : A;
    const int ldx = isB ? ldb : lda, R = isB ? n : m, s = isB ? sB : sA, cs = isB ? cB : cA;
    const int lane = threadIdx.x & 63, r = lane % PR, q = lane / PR % 4, cl = lane / PR / 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int row = R0 + r;
    const size_t rstep = isB ? (size_t)ldx : 1, kstep = isB ? 1 : (size_t)ldx;
    const unsigned long long *p = X + (size_t)(row < R ? row : R - 1) * rstep;
    if (panel == 0 && threadIdx.x < 6) {
        // header for ozimmu_check: no flag yet, how many words bad[] has, where, and two words that make these valid;
        // the planes of both operands will be there
        static_assert(kHeaderPlanes == kHeaderBadWords + 4, "written together");
        const int i = threadIdx.x;
        const unsigned long long v[6] = {0ULL, (unsigned long long)panels, (unsigned long long)bad_offset, kBadWordsMagic,
                                         (unsigned long long)(uintptr_t)header, 0ULL};
        header[i == 0 ? 0 : kHeaderBadWords + i - 1] = v[i];
    }

    unsigned long long x[NV][4], mx = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int kq = 16 * ((wave + nw * v) * CW + cl) + 4 * q;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool in = row < R && kq + i < K;
            x[v][i] = p[(size_t)(kq + i < K ? kq + i : K - 1) * kstep];
            x[v][i] = in ? x[v][i] : 0ULL;
        }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const unsigned long long u = x[v][i] & 0x7fffffffffffffffULL;
            mx = u > mx ? u : mx;
        }
#pragma unroll
    for (int off = PR; off <= 32; off <<= 1) {
        const unsigned long long o = __shfl_xor(mx, off);
        mx = o > mx ? o : mx;
    }
    if (lane < PR) smx[wave][r] = mx;
    __syncthreads();
    mx = 0;
    for (int i = 0; i < nw; ++i) {
        const unsigned long long o = smx[i][r];
        mx = o > mx ? o : mx;
    }
    const int e = row < R ? exponent_above(mx) + (NEAREST ? 1 : 0) : 0;
    if (wave == 0) {
        if (lane < PR) (isB ? eB : eA)[row] = e;
        const unsigned long long any = __ballot(mx >= 0x7ff0000000000000ULL);
        if (lane == 0) bad[panel] = any ? 1u : 0u;
    }

    int8_t *base = (isB ? pB : pA) + (size_t)(row >> 5) * KB * ((size_t)cs * kFragBytes) + (row & 31) * 16 + 4 * q;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int c = (wave + nw * v) * CW + cl;                // 16 k: half c % 2 of fragment c / 2
        if (c >= 2 * KB) continue;
        unsigned *dst = (unsigned *)(base + (size_t)(c >> 1) * ((size_t)cs * kFragBytes) + (c & 1) * (32 * 16));
        Quad<NEAREST> el[1];
        el[0].load(x[v], e);
        for_each_slice<NEAREST, 1>(el, s, [&](int l, const unsigned (&wd)[1]) {
            unsigned *to = dst + (size_t)(l - 1) * (kFragBytes / 4);
            if constexpr (THROUGH) asm volatile("global_store_dword %0, %1, off sc1" ::"v"(to), "v"(wd[0]) : "memory");
            else *to = wd[0];
        });
        // (the planes hold cs >= s slices per entry; those beyond s are zeros)
        for (int l = s + 1; l <= cs; ++l) dst[(size_t)(l - 1) * (kFragBytes / 4)] = 0;
    }
}

// Sets the header's flag where a work-group of scale_split_kernel has met a NaN or an infinity.
__global__ __launch_bounds__(256) void collect_bad_kernel(unsigned long long *header)
{
    const unsigned long long *h = header + kHeaderBadWords;
    if (h[2] != kBadWordsMagic || h[3] != (unsigned long long)(uintptr_t)header) return;
    const unsigned *words = (const unsigned *)((const char *)header + h[1]);
    unsigned any = 0;
    for (unsigned long long i = blockIdx.x * 256 + threadIdx.x; i < h[0]; i += gridDim.x * 256) any |= words[i];
    if (__ballot(any != 0) && (threadIdx.x & 63) == 0) atomicOr((unsigned *)header, 1u);
}

// ---- plain layout: plane l is a matrix shaped like X (utility / test path) ----
template <bool NEAREST>
__global__ __launch_bounds__(256) void split_plain_kernel(const unsigned long long *__restrict__ X, int ldx, int rows,
                                                          int cols, int s, const int32_t *__restrict__ exps,
                                                          int by_row, int8_t *__restrict__ planes)
{
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r >= rows) return;
    const size_t plane = (size_t)rows * cols;
    for (int c = blockIdx.y; c < cols; c += gridDim.y) {
        const int e = by_row ? exps[r] : exps[c];
        const Elem el = decompose(X[r + (size_t)c * ldx], e);
        unsigned int carry = 0;
        for (int l = 1; l <= s; ++l)
            planes[(size_t)(l - 1) * plane + r + (size_t)c * rows] = (int8_t)slice_of<NEAREST>(el, l, carry, 0);
    }
}

}  // namespace

hipError_t launch_split(char side, int rows, int cols, const double *X, int ldx, int s, const int32_t *exps,
                        int8_t *planes, int layout, bool nearest, hipStream_t st)
{
    if (layout == OZIMMU_LAYOUT_PLAIN) {
        if (rows <= 0 || cols <= 0) return hipSuccess;
        dim3 grid((rows + 255) / 256, cols < 65535 ? cols : 65535);
        auto kern = nearest ? split_plain_kernel<true> : split_plain_kernel<false>;
        kern<<<grid, 256, 0, st>>>((const unsigned long long *)X, ldx, rows, cols, s, exps, side == 'A' ? 1 : 0, planes);
        return hipGetLastError();
    }
    const int R = side == 'A' ? rows : cols, K = side == 'A' ? cols : rows;
    const int Rp = round_up(R > 0 ? R : 1, kPad), Kp = round_up(K > 0 ? K : 1, kPad);
    const int KB = Kp / kFrag;
    if (side == 'A') {
        dim3 grid(Rp / 64, Kp / 64);
        if (grid.y > 65535) return hipErrorInvalidValue;
        auto kern = nearest ? split_rows_kernel<true> : split_rows_kernel<false>;
        kern<<<grid, 256, 0, st>>>((const unsigned long long *)X, ldx, R, K, s, exps, planes, KB);
    } else {
        dim3 grid(Rp / 32, Kp / kColTileK);
        if (grid.y > 65535) return hipErrorInvalidValue;
        auto kern = nearest ? split_cols_kernel<true> : split_cols_kernel<false>;
        kern<<<grid, 256, 0, st>>>((const unsigned long long *)X, ldx, R, K, s, exps, planes, KB);
    }
    return hipGetLastError();
}

// Rows to a work-group.  Four put the most compute units to work (a compute unit takes in some 10-25 GB/s whatever
// it asks for: 1024^3 s = 7 27.1 / 21.3 / 21.5 us for 16 / 8 / 4 rows, 256 x 256 x 1024 25.4 / 18.3 / 15.4, 1024 x 1024 x 2048 41.0 /
// 25.9 / 24.4, 2048^3 40.9 / 42.7 / 37.5; two rows: 29.7 in the last but one); eight where there are plenty of rows and the
// pieces of cache lines begin to count.  With few slices, where that is depends on k (one call repeated, eight against four rows, m = n = 4096 / 5120 / 6144 / 8192: k =
// 1024, s = 3 30.1 and 32.4 / 34.9 and 38.2 / 39.8 and 43.2 / 47.8 and 52.0, k = 2048, s = 3 54.5 and 48.2 / 65.6 and 58.0 / 78.2 and 75.3 /
// 103 and 107, s = 7 63.2 and 57.9 / 80.1 and 92.1 / 98.2 and 112); the line is where the longest contractions change over
// at few slices, and what it costs the shorter ones below it is at most 3 % of a call (12000 x 200 x 1000, s = 7: 113 and 117)
//
// More slices write more, and eight rows, whose pieces fill whole lines, are ahead once the planes outgrow the caches: by bytes, a
// row of A counting more than a column of B, which is read in whole lines whichever way (calls, us, four and eight rows, operands that change from one to
// the next: 2600 x 2600 x 3000 s = 7, 140 MB, A alone 55, 459 and 444; 3736 x 129 x 3968 s = 7, 107, 141 and 128; 7040 x 75 x 1152 s = 9, 74, 77 and
// 71; but 35 x 4096 x 1792 s = 9, 67, 57.5 and 65.5; 2112^3 s = 5, 46, 149 and 163; even at 2500 x 2400 x 2500 s = 7, 88; from twelve
// slices on ahead whichever operand they are of, 48 x 5568 x 1367 s = 13, 103, 102 and 98).  k up to 256: from 6000 rows on (6001 x 5200 x 256 26.1 and 23.3, 3000 x 3000 x 256 19.7
// and 19.1; k = 512 23.5 and 27.0).  With fewer than 3000 rows too few work-groups are left.
static int scale_split_rows(int m, int n, int kp, int c)
{
    const long long rows = (long long)m + n;
    const double bytes = (double)c * kp;                  // of a row
    const bool large = rows >= 3000 && (bytes * (m + 0.4 * n) >= 70e6 || (c >= 12 && bytes * rows >= 80e6));
    return (kp <= 2048 && rows >= 12288) || (kp <= 256 && rows >= 6000) || large ? 8 : 4;
}

// Wavefronts: 64 k (four rows) or 32 k (eight) to each, up to sixteen.  With four rows, two work-groups for every compute unit and planes up to
// 100 MB, eight, so that one work-group loads while another stores, where sixteen leave much of a compute unit or of their last sweep over k empty: at 14 ...
// 24 times 64 k (one full work-group to a compute unit, or a second sweep at most half full), at 34 ... 36 and from 50 on; at 26 ... 32 and 38 ... 48 their
// sweeps are full and they are even or ahead, but where columns of B, up to nine slices, are what there is most of, eight keep ahead up to 40.  Calls, sixteen
// and eight, geometric means over 1200 random sizes: kp = 768 0.986, 896 and 1024 1.026, 1152 1.047, 1536 1.021, 1664 ... 2048 1.000, 2176 1.014, 2432 ...
// 3072 0.985, 3328 1.07, 3712 1.03 (1024^3 s = 7 35.2 and 34.5, 1600 x 1600 x 1536 108 and 103, 20 x 5869 x 2368 s = 5 70.2 and 67.6, 2091 x 75 x 1792 s = 5 27.1
// and 27.5, 2432 x 105 x 2812 s = 2 29.6 and 33.9).  Few slices store little: from 640 on where there are 4096 rows.  Against sixteen throughout, with
// the rows above: 1.022 over 1440 sizes, slowest 0.91; operands that the caches still hold, as after the estimator, lose up to 4 percent (1280^3 s = 6 95.8
// and 99).
static int scale_split_waves(int m, int n, int rows, int kp, int c)
{
    const int waves = kp / 16 * rows / 16;
    const long long R = (long long)m + n;
    const bool apart = (kp >= 896 && kp <= 1536) || (kp >= 2176 && kp <= 2304) || kp >= 3200 || (n >= m && c <= 9 && kp >= 1664 && kp <= 2560) ||
                       (R >= 4096 && ((c <= 3 && kp >= 640 && kp <= 2304) || (c <= 7 && kp == 640)));
    const int most = rows == 4 && apart && R / rows >= 2LL * device_cus() && c * R * kp < 100000000LL ? 8 : 16;
    if (waves <= most) return waves < 1 ? 1 : waves;
    const int sweeps = (waves + most - 1) / most;
    return most == 16 ? 16 : (waves + sweeps - 1) / sweeps;       // (of eight, no more than the sweeps over k keep busy)
}

// Whether the slices are written through the L2s as they are formed (device-scope stores) rather than at the end of the launch, when the next one
// waits for it.  While operands and planes stay in the memory-side cache that gains 1 to 4 percent of a call; where the operands come from memory, the planes are
// displaced meanwhile and the stores, halves of lines, go to memory beside the reads.  Calls, us, plain / through, one pair of operands over and over, and
// pairs of 700 MB in turn in one workspace: 1472 x 152 x 1105 s = 7 (14 MB of operands) 24.6 / 23.4 and 26.4 / 27.2, 2432 x 140 x 768 s = 7 (16 MB) 27.8 / 27.8 and 29.6 / 32.2,
// 1024 x 155 x 1797 s = 5 (17 MB) 24.3 / 23.6 and 25.9 / 27.3.  Means over 460 random sizes by the operands' bytes, the same two and pairs with workspaces of their own:
// 2 to 4 MB 1.01, 1.01, 1.00; 4 to 5 MB 1.02, 1.02, 0.99; 5 to 8 MB 1.03, 1.02, 0.98; 8 to 16 MB 1.04, 1.01, 0.97; more 1.02, 0.96, 0.97.  So operands up to 4 MB, where
// no way of having them is behind (planes up to 14 MB measured).
static bool scale_split_through(int m, int n, int k, int kp, int c)
{
    const long long rows = (long long)m + n;
    return 8 * rows * k <= 4000000LL && rows * kp * c <= 16000000LL;
}

static long long scale_split_groups(int m, int n, int rows)
{
    return (((long long)m + rows - 1) / rows + ((long long)n + rows - 1) / rows + 7) / 8 * 8;
}

// Contractions up to 2048 always; up to 4096 while the operands have up to about 18 million entries (both phases of two
// launches against one, us, s = 7: 2048 x 2048 x 4096 81.7 -> 67.4, 1000 x 1000 x 3000 40.0 -> 27.0, 2500 x 2400 x 2500 64.1 -> 46.0, but
// 3000 x 2900 x 4000 106.5 -> 112.1 and 4096^3 147.7 -> 157.5: there a work-group's loads wait for a chip that is busy
// anyway, and the register-resident form has fewer wavefronts)
// A launch holds fewer than 2^32 threads, 8 to 128 per row here: beyond (134 million rows at k <= 128, 33 million from 512 on)
// the two launches of the general way, which take more, serve.
long long scale_split_threads(int m, int n, int k)
{
    if (m <= 0 || n <= 0 || k <= 0) return 0;
    const int kp = round_up(k, kPad);
    if (kp > 2048 && (kp > 4096 || ((long long)m + n) * kp > 18LL << 20)) return 0;
    const int rows = scale_split_rows(m, n, kp, 0);          // (more slices: other shapes, below 12288 rows)
    const long long threads = scale_split_groups(m, n, rows) * 64 * scale_split_waves(m, n, rows, kp, 0);
    return threads < 1LL << 32 ? threads : 0;
}

hipError_t launch_scale_split(int m, int n, int k, const double *A, int lda, const double *B, int ldb, int sA, int sB, int cA,
                              int cB, int32_t *eA, int32_t *eB, int8_t *pA, int8_t *pB, bool nearest,
                              unsigned long long *header, size_t bad_offset, hipStream_t st)
{
    if (!scale_split_threads(m, n, k) || cA < sA || cB < sB) return hipErrorInvalidValue;
    const int kp = round_up(k, kPad), c = cA > cB ? cA : cB;
    auto *bad = (unsigned *)((char *)header + bad_offset);
    auto launch = [&](auto PRC, auto NVC) {
        constexpr int PR = decltype(PRC)::value, NV = decltype(NVC)::value;
        const int panelsA = (m + PR - 1) / PR, panels = panelsA + (n + PR - 1) / PR;
        auto kern = scale_split_through(m, n, k, kp, c) ? (nearest ? scale_split_kernel<true, PR, NV, true> : scale_split_kernel<false, PR, NV, true>)
                                                     : (nearest ? scale_split_kernel<true, PR, NV, false> : scale_split_kernel<false, PR, NV, false>);
        kern<<<(unsigned)scale_split_groups(m, n, PR), 64 * scale_split_waves(m, n, PR, kp, c), 0, st>>>(
            (const unsigned long long *)A, lda, m, (const unsigned long long *)B, ldb, n, k, sA, sB, cA, cB, eA, eB, pA, pB, kp / kFrag,
            panelsA, header, panels, (long long)bad_offset, bad);
    };
    auto by_k = [&](auto PRC) -> hipError_t {
        constexpr int PR = decltype(PRC)::value;
        const int sweep = scale_split_waves(m, n, PR, kp, c) * 16 * (16 / PR);           // k of all wavefronts
        switch ((kp + sweep - 1) / sweep) {
#define OZ_CASE(NV_) case NV_: launch(PRC, std::integral_constant<int, NV_>{}); return hipGetLastError();
            OZ_CASE(1) OZ_CASE(2) OZ_CASE(3) OZ_CASE(4) OZ_CASE(5) OZ_CASE(7) OZ_CASE(8)
            case 6:                                             // (of eight rows only: scale_split_waves)
                if constexpr (PR == 8) {
                    launch(PRC, std::integral_constant<int, 6>{});
                    return hipGetLastError();
                }
#undef OZ_CASE
        }
        return hipErrorInvalidValue;
    };
    return scale_split_rows(m, n, kp, c) == 8 ? by_k(std::integral_constant<int, 8>{}) : by_k(std::integral_constant<int, 4>{});
}

hipError_t launch_collect_bad(unsigned long long *header, hipStream_t st)
{
    collect_bad_kernel<<<32, 256, 0, st>>>(header);
    return hipGetLastError();
}

hipError_t launch_split_both(int m, int n, int k, const double *A, int lda, const double *B, int ldb, int sA, int sB,
                             int cA, int cB, const unsigned long long *maxA, const unsigned long long *maxB, int32_t *eA,
                             int32_t *eB, int8_t *pA, int8_t *pB, bool nearest, hipStream_t st)
{
    if (cA < sA || cB < sB) return hipErrorInvalidValue;
    const int mp = round_up(m > 0 ? m : 1, kPad), np = round_up(n > 0 ? n : 1, kPad), kp = round_up(k > 0 ? k : 1, kPad);
    const int gxA = mp / 64, gxB = np / 32;
    const long long nblkA = pA ? (long long)gxA * (kp / 64) : 0, nblkB = pB ? (long long)gxB * (kp / kColTileK) : 0;
    if (nblkA + nblkB > 0x7fffffffLL) return hipErrorInvalidValue;
    auto kern = nearest ? split_both_kernel<true> : split_both_kernel<false>;
    kern<<<(unsigned)(nblkA + nblkB), 256, 0, st>>>((const unsigned long long *)A, lda, m,
                                                    (const unsigned long long *)B, ldb, n, k, sA, sB, cA, cB, maxA, maxB, eA, eB,
                                                    pA, pB, kp / kFrag, gxA, (int)nblkA, gxB);
    return hipGetLastError();
}

}  // namespace oz
