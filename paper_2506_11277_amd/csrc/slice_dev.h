// Slicing four entries at a time (device code of split.hip and gemm_vectors.hip).
#pragma once
#include <type_traits>

#include "oz_common.h"

namespace oz {

// Slices of four neighbouring entries (consecutive k) at a time, four bytes to a word.  A 64-bit shift by a variable
// amount, a compare and a select per slice and entry made the slicing kernels arithmetic-bound at sizes that fit the
// caches; here y = |x| 2^-e, a binary64 number below 1, is turned into the integer floor(y 2^63) once per nine slices
// (eight when rounding to nearest, whose last slice needs the bit below it), slice j of such a window at bits
// 63 - 7 j ... 69 - 7 j, and carry, sign and two's complement are handled for the four bytes of a word together.  The
// window costs five binary64 operations, all exact (a product with a power of two, or a number minus its leading bits); what
// is left of y is the next window's.  (y itself is exact unless it falls below 2^-1022, where none of the at most 32
// slices reaches.)
constexpr unsigned kOnes = 0x01010101u, kTops = 0x80808080u, kLows = 0x7f7f7f7fu;

template <bool NEAREST>
struct Quad {
    static constexpr int WIN = NEAREST ? 8 : 9;       // slices per window
    double y[4];               // what the windows so far have left, scaled so that the next slice starts below 2^31
    unsigned neg;              // byte mask of the negative entries
    unsigned sticky;           // NEAREST: byte i = last slice of the window below whose guard bit entry i has bits left
    unsigned carry;            // NEAREST: byte i = c_{l-1} of entry i
    unsigned lo[4], hi[4];     // the window

    __device__ __forceinline__ void load(const unsigned long long (&bits)[4], int e)
    {
        neg = carry = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            y[i] = ldexp(__builtin_fabs(__longlong_as_double((long long)bits[i])), 31 - e);
            neg |= (unsigned)((int)(bits[i] >> 32) >> 31) & (0xffu << (8 * i));
        }
    }
    // the next window
    __device__ __forceinline__ void window()
    {
        sticky = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            hi[i] = (unsigned)y[i];
            const double t = (y[i] - (double)hi[i]) * 4294967296.0;
            lo[i] = (unsigned)t;
            y[i] = t - (double)lo[i];
            if (!NEAREST) y[i] *= 2147483648.0;
            else {
                // bits left below the guard bit 62 - 7 j of slice j: always if anything is left beyond the window, else
                // while j <= (61 - (lowest bit of the window)) / 7
                const unsigned long long F = (unsigned long long)hi[i] << 32 | lo[i];
                const int x = y[i] != 0.0 ? 63 : F ? 61 - __builtin_ctzll(F) : 0;
                sticky |= (((unsigned)(x < 0 ? 0 : x) * 9363u) >> 16) << (8 * i);      // x / 7
                y[i] = (y[i] + (double)(lo[i] & 127u)) * 16777216.0;  // (the window's last seven bits belong to the next one)
            }
        }
    }
    template <int P, int N>
    __device__ __forceinline__ unsigned field(int i) const      // bits P ... P + N - 1 of the window of entry i
    {
        if constexpr (P >= 32) return (hi[i] >> (P - 32)) & ((1u << N) - 1);
        else if constexpr (P + N <= 32) return (lo[i] >> P) & ((1u << N) - 1);
        else return __builtin_amdgcn_alignbit(hi[i], lo[i], P) & ((1u << N) - 1);
    }
    template <int P, int N>
    __device__ __forceinline__ unsigned fields() const
    {
        return field<P, N>(0) | (field<P, N>(1) << 8) | (field<P, N>(2) << 16) | (field<P, N>(3) << 24);
    }
    // the four bytes of slice J of the window (slices in ascending order: the carry of the slice before is kept)
    template <int J>
    __device__ __forceinline__ unsigned word()
    {
        unsigned v;
        if constexpr (!NEAREST) {
            // -v, byte by byte, where neg: ((v ^ 7f) + 1) ^ 80, which no byte carries out of (v < 128)
            v = fields<63 - kSliceBits * J, 7>();
            return ((v ^ (neg & kLows)) + (neg & kOnes)) ^ (neg & kTops);
        } else {
            const unsigned g = fields<62 - kSliceBits * J, 8>();         // slice and the guard bit below it
            const unsigned f = (g >> 1) & kLows;
            const unsigned left = (((sticky | kTops) - (unsigned)J * kOnes) >> 7) & kOnes;   // J <= sticky
            const unsigned c = g & kOnes & (left | f);
            v = (f + c) ^ (carry << 7);                                  // + c_l - 128 c_{l-1}, modulo 256
            carry = c;
        }
        const unsigned minus = (kTops - (v & kLows)) ^ (~v & kTops);     // -v, byte by byte
        return (minus & neg) | (v & ~neg);
    }
};

// calls f(l, word of slice l) ... for N quads at once: f(l, words) for l = 1, ..., s
template <bool NEAREST, int N, class F>
__device__ __forceinline__ void for_each_slice(Quad<NEAREST> (&q)[N], int s, F &&f)
{
    for (int w = 0; w < s; w += Quad<NEAREST>::WIN) {
#pragma unroll
        for (int i = 0; i < N; ++i) q[i].window();
        auto one = [&](auto JC) {
            constexpr int J = decltype(JC)::value;
            if (w + J > s) return;
            unsigned wd[N];
#pragma unroll
            for (int i = 0; i < N; ++i) wd[i] = q[i].template word<J>();
            f(w + J, wd);
        };
        one(std::integral_constant<int, 1>{});
        one(std::integral_constant<int, 2>{});
        one(std::integral_constant<int, 3>{});
        one(std::integral_constant<int, 4>{});
        one(std::integral_constant<int, 5>{});
        one(std::integral_constant<int, 6>{});
        one(std::integral_constant<int, 7>{});
        one(std::integral_constant<int, 8>{});
        if constexpr (!NEAREST) one(std::integral_constant<int, 9>{});
    }
}

}  // namespace oz
