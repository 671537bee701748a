// A large matrix times a few vectors: one operand has at most 64 rows (A) or columns (B), the other is long and the
// contraction too.
//
// Every entry of the long operand then meets one tile only.  Writing its slices to memory and reading them back (8 s
// bytes per 8-byte entry of traffic) is most of what the general path does; here the long operand is read as it is and
// sliced on its way into LDS, by the wavefronts that multiply.  The short operand is sliced beforehand as usual; its
// planes stay in the L2s.  Diagonal sums, product set and binary64 order are those of the other kernels.
//
// Work-group: 32 rows (columns) of the long operand x 64 of the short one x a part of k; eight wavefronts, two halves of
// the short side x four groups that take every fourth 32-deep k-block.  The two wavefronts of a group slice a 32 x 32
// block of the long operand together (8 consecutive k per lane), multiply the block of the step before meanwhile, and
// keep the raw entries of the one to three steps after in flight, as many as the registers hold: 32 KiB per compute unit each.
// At 8192 x 64 x 8192, s = 7 the kernel takes 152 us and the maxima before it 77, where reading, slicing, writing and
// multiplying took 567 us.  What bounds it: two chains of about 120 us each that two wavefronts to a SIMD overlap in part.  Kernel alone in a loop of calls, parts
// of it left out: loading both operands, with the barriers and writes to LDS, 120 us (the long one alone 92, 5.8 TB/s; the short one's slices, out of the L2s once per 32 long
// rows, alone 44); slicing and multiplying with the short one's slices loaded 125 (slicing alone 72, products with their LDS reads 85).  Nothing is
// saturated: of the cycles matrix pipes 41 percent, vector ALUs 44, LDS 16; 3.5 TB/s from memory, 9.8 TB/s out of the L2s; the wavefronts wait for a
// third.  The power cap is not it: with pauses of 4 ms between calls 153 us.  A barrier every second step, and the window formed with integer shifts, changed
// nothing.
// Few tiles are compensated by several parts of k; each part leaves its int32 sums in a slot of its own (in the room
// the general path keeps the long operand's planes in) and a second kernel adds them.
#include "gemm_dev.h"
#include "slice_dev.h"

namespace oz {

namespace {

constexpr int kZeroScale = 4096;        // exponent at which every finite number has zero slices only

template <int S, bool NEAREST>
struct CfgVectors {
    static constexpr int ROUND = S < 4 ? S : 4;             // diagonals that are exchanged at a time
    // steps whose raw entries are in flight, as many as the registers hold
    static constexpr int AHEAD = S <= 6 ? 3 : S == 7 ? (NEAREST ? 2 : 3) : S == 8 ? (NEAREST ? 1 : 2) : 1;
    static constexpr int ABYTES = 2 * 4 * S * kFragBytes;   // sliced blocks of four groups, two steps
    static constexpr int XBYTES = ROUND * 8 * 16 * 256;
    static constexpr int LDS = ABYTES > XBYTES ? ABYTES : XBYTES;
};

// SHORT_A: the short operand is A (C has few rows), the long one B; else the other way round.
template <int S, bool NEAREST, bool SHORT_A>
__global__ __launch_bounds__(512) void gemm_vectors_kernel(const unsigned long long *__restrict__ X, int ldx, int L,
                                                           const unsigned long long *__restrict__ maxbits,
                                                           int32_t *__restrict__ exps_out, const int8_t *__restrict__ P,
                                                           const int32_t *__restrict__ exps_short, double *__restrict__ C,
                                                           int ldc, int m, int n, int K, int KB, int kb_per_part,
                                                           int32_t *__restrict__ slots, int Q)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int lane = threadIdx.x & 63, r = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), j = wave & 1, kg = wave >> 1;
    const int tile = blockIdx.x, part = blockIdx.y;
    const int row = tile * 32 + r;
    const int e = row < L ? exponent_above(maxbits[row]) + (NEAREST ? 1 : 0) : kZeroScale;
    if (part == 0 && wave == 0 && hh == 0) exps_out[row] = row < L ? e : 0;

    // k-blocks of this part: whole ones [kb0, kb1), and perhaps the ragged one behind them, which is taken first (step -1)
    const int kbF = K / 32, kb0 = part * kb_per_part, kb1 = kb0 + kb_per_part < kbF ? kb0 + kb_per_part : kbF;
    const int steps = kb1 > kb0 ? (kb1 - kb0 + 3) / 4 : 0;
    const int first = (K & 31) && kb0 <= kbF && kbF < kb0 + kb_per_part ? -1 : 0;
    const size_t kstep = 8 * (SHORT_A ? 1 : (size_t)ldx), rstep = 8 * (SHORT_A ? (size_t)ldx : 1);      // bytes
    // (rows beyond the operand repeat its last one, at a scale that makes every slice zero)
    const char *base = (const char *)X + (size_t)tile * 32 * rstep;
    const unsigned voff = (unsigned)(row < L ? r : L - 1 - tile * 32) * (unsigned)rstep + (unsigned)(16 * j + 8 * hh) * (unsigned)kstep;
    const char *const sp = (const char *)P + (size_t)j * KB * (S * kFragBytes);

    // raw entries of this lane: k = 32 kb + 16 j + 8 hh + 0 ... 7 of row r.  No branch and no test per entry, so that the
    // loads of several steps can be in flight: a step beyond the part loads the last block again, and scale() makes
    // every slice of it zero.
    auto fetch = [&](int i, unsigned long long (&x)[2][4]) {
        const int kb = kb0 + kg + 4 * i, kc = kb < kb1 ? kb : (kb1 > 0 ? kb1 - 1 : 0);
        const char *q = base + (size_t)kc * 32 * kstep;
#pragma unroll
        for (int t = 0; t < 8; ++t) x[t >> 2][t & 3] = *(const unsigned long long *)(q + (size_t)t * kstep + voff);
    };
    auto scale = [&](int i) { return kb0 + kg + 4 * i < kb1 ? e : kZeroScale; };
    auto short_slice = [&](int i, int h) -> v4i {
        const int kb = i < 0 ? kbF : kb0 + kg + 4 * i;
        return *(const v4i *)(sp + ((size_t)(kb < KB ? kb : KB - 1) * S + h) * kFragBytes + (unsigned)lane * 16);
    };
    unsigned char *const abase = lds + kg * (S * kFragBytes);
    constexpr int ABUF = 4 * S * kFragBytes;

    v16i acc[S];
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[a][q] = 0;

    constexpr int AHEAD = CfgVectors<S, NEAREST>::AHEAD;             // steps whose raw entries are in flight
    unsigned long long x[AHEAD][2][4];
    v4i bf[S];
    Quad<NEAREST> el[2];
    auto begin = [&](const unsigned long long (&raw)[2][4], int escale) {
        el[0].load(raw[0], escale);
        el[1].load(raw[1], escale);
    };
    auto put = [&](int l, unsigned char *dst) {             // slice l (from 0) of this lane's eight entries
        constexpr int WIN = Quad<NEAREST>::WIN;
        static_for<0, S>([&](auto LC) {
            constexpr int ll = decltype(LC)::value;
            if (ll != l) return;
            if constexpr (ll % WIN == 0) {
                el[0].window();
                el[1].window();
            }
            typedef unsigned v2u __attribute__((ext_vector_type(2)));
            v2u w;
            w[0] = el[0].template word<ll % WIN + 1>();
            w[1] = el[1].template word<ll % WIN + 1>();
            *(v2u *)(dst + ll * kFragBytes + (r + 32 * j) * 16 + 8 * hh) = w;
        });
    };
    if (first < 0) {
        // ragged block: group 0 takes what there is of it, the others zeros
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int k = kbF * 32 + 16 * j + 8 * hh + t;
            const bool in = kg == 0 && k < K;
            const unsigned long long v =
                *(const unsigned long long *)(base + (size_t)(in ? k : 0) * kstep + (size_t)(row < L ? r : L - 1 - tile * 32) * rstep);
            x[0][t >> 2][t & 3] = in ? v : 0ULL;
        }
    } else fetch(0, x[0]);
#pragma unroll
    for (int h = 0; h < S; ++h) bf[h] = short_slice(first, h);
    begin(x[0], first < 0 ? e : scale(0));
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) fetch(first + 1 + d, x[d]);
#pragma unroll
    for (int l = 0; l < S; ++l) put(l, abase);
    // (from 3 slices on the short operand's first slices have landed before the loop. The compiler moves their loads down to it,
    // behind the raw entries, and as it counts what may be in flight for both ways into the loop at once, it then waited for
    // everything, entries of steps to come included, once per AHEAD steps. Product alone, us, before -> now: 6000 x 64 x 6001,
    // 4 / 6 / 8 slices 75.6 / 93.9 / 114.9 -> 75.4 / 93.3 / 110.7; 8192 x 64 x 8192, 6 slices 141.0 -> 139.3. With 2 slices
    // 64 x 8192 x 8192 lost by it, 124.7 -> 127.5)
    if constexpr (S > 2) {
#pragma unroll
        for (int h = 0; h < S; ++h) asm volatile("" : "+v"(bf[h]));
    }
    __syncthreads();

    // (the loop runs over whole groups of AHEAD steps: those beyond the last one multiply zeros)
    const int count = steps - first;
    for (int c0 = 0; c0 < count; c0 += AHEAD) {
        static_for<0, AHEAD>([&](auto DC) {
            constexpr int d = decltype(DC)::value;
            const int c = c0 + d, i = first + c;
            const unsigned char *cur = abase + (c & 1) * ABUF + lane * 16;
            unsigned char *nxt = abase + ((c & 1) ^ 1) * ABUF;
            v4i af = *(const v4i *)cur, afn;
            begin(x[d], scale(i + 1));
            static_for<0, S>([&](auto LC) {
                constexpr int l = decltype(LC)::value;
                if constexpr (l + 1 < S) afn = *(const v4i *)(cur + (l + 1) * kFragBytes);
                static_for<0, S - l>([&](auto HC) {
                    constexpr int h = S - 1 - l - decltype(HC)::value;
                    acc[l + h] = SHORT_A ? __builtin_amdgcn_mfma_i32_32x32x32_i8(af, bf[h], acc[l + h], 0, 0, 0)
                                         : __builtin_amdgcn_mfma_i32_32x32x32_i8(bf[h], af, acc[l + h], 0, 0, 0);
                });
                bf[S - 1 - l] = short_slice(i + 1, S - 1 - l);
                put(l, nxt);
                af = afn;
            });
            // (loads return in order: behind those of the short operand, or the next step's wait for them would be a wait
            // for these too)
            __builtin_amdgcn_sched_barrier(0);
            fetch(i + 1 + AHEAD, x[d]);
            __syncthreads();
        });
    }

    // the sums of the four groups meet in LDS; wavefront (j, kg) finishes accumulator registers 4 kg ... 4 kg + 3
    v4i *xch = (v4i *)lds;
    v4i D[S];
    constexpr int ROUND = CfgVectors<S, NEAREST>::ROUND;
    static_for<0, (S + ROUND - 1) / ROUND>([&](auto PC) {
        constexpr int a0 = decltype(PC)::value * ROUND, a1 = a0 + ROUND < S ? a0 + ROUND : S;
        if constexpr (a0 > 0) __syncthreads();
#pragma unroll
        for (int a = a0; a < a1; ++a)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                xch[((((a - a0) * 2 + j) * 4 + g) * 4 + kg) * 64 + lane] = v4i{acc[a][4 * g], acc[a][4 * g + 1], acc[a][4 * g + 2], acc[a][4 * g + 3]};
        __syncthreads();
#pragma unroll
        for (int a = a0; a < a1; ++a) {
            v4i s{0, 0, 0, 0};
#pragma unroll
            for (int g = 0; g < 4; ++g) s += xch[((((a - a0) * 2 + j) * 4 + kg) * 4 + g) * 64 + lane];
            D[a] = s;
        }
    });
    if (slots) {
        v4i *slot = (v4i *)slots + ((size_t)part * gridDim.x + tile) * (S * 512) + threadIdx.x;
#pragma unroll
        for (int a = 0; a < S; ++a) slot[a * 512] = D[a];
        return;
    }
    const int mi = (SHORT_A ? j : tile) * 32 + (lane & 31);
    if (mi >= m) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int nj = (SHORT_A ? tile : j) * 32 + 8 * kg + 4 * hh + q;
        if (nj >= n) continue;
        int d[S];
#pragma unroll
        for (int a = 0; a < S; ++a) d[a] = D[a][q];
        // (the long operand's exponents: of this lane's own row, or formed again for the four columns of this lane)
        const int el_ = SHORT_A ? exponent_above(maxbits[nj]) + (NEAREST ? 1 : 0) : e;
        C[mi + (size_t)nj * ldc] = ldexp(diagonal_sum<S>(d, Q), el_ + exps_short[SHORT_A ? mi : nj]);
    }
}

// adds the slots of the parts of k exactly, then the diagonals in ascending order as everywhere
__global__ __launch_bounds__(512) void finish_vectors_kernel(const int32_t *__restrict__ slots, int parts, int S, bool short_a,
                                                             const int32_t *__restrict__ eA, const int32_t *__restrict__ eB,
                                                             double *__restrict__ C, int ldc, int m, int n, int Q)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = wave & 1, kg = wave >> 1, tile = blockIdx.x;
    const int mi = (short_a ? j : tile) * 32 + (lane & 31);
    LevelSum sum[4];
    for (int a = 0; a < S; ++a) {
        long long v[4] = {0, 0, 0, 0};
        const v4i *slot = (const v4i *)slots + ((size_t)tile * S + a) * 512 + threadIdx.x;
        for (int y = 0; y < parts; ++y) {
            const v4i d = slot[(size_t)y * gridDim.x * (S * 512)];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] += d[q];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) sum[q].add(ldexp((double)v[q], -kSliceBits * (a + 2)), Q, a == S - 1);      // exact: |v| < 2^53
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int nj = (short_a ? tile : j) * 32 + 8 * kg + 4 * (lane >> 5) + q;
        if (mi < m && nj < n) C[mi + (size_t)nj * ldc] = ldexp(sum[q].S, eA[mi] + eB[nj]);
    }
}

// Parts of k: enough work-groups for the compute units in whole rounds.  A step of 128 k takes about 1 us; a slot is
// written and read once; no part shorter than 512 k, none of more (whole) steps than int32 sums allow.
int vectors_parts(int s, int tiles, int kp)
{
    const int cus = device_cus();
    const int all = kp / 128, longest = (int)(kMaxInt32K / (128LL * s)), need = (all + longest - 1) / longest;
    int best = 0;
    double best_cost = 0.0;
    for (int parts = need; parts <= kp / 512 && (parts <= 16 || parts == need); ++parts) {
        const int steps = (all + parts - 1) / parts;
        const double rounds = (double)(((long long)tiles * parts + cus - 1) / cus);
        const double cost = rounds * (steps + 3.0) + (parts > 1 ? 4.0 + (double)parts * tiles * s * 8192 * 2 / 4.5e6 : 0.0);
        if (!best || cost < best_cost) {
            best = (all + steps - 1) / steps;       // (as many as get a step)
            best_cost = cost;
        }
    }
    return best;
}

}  // namespace

// Where it pays: the contraction is too long for the launch that reads the operands once (then 16 bytes per long entry
// are moved here against 16 + 2 s), the short side fits the 64 of a work-group, and the long operand has some million
// entries.  Against the 32 x 32 and 64 x 64 tiles with their operands sliced beforehand (whole calls, us, tiles and this):
// below two million entries it loses (400 x 64 x 4200, s = 2 / 7: 27.9 and 34.1 / 48.8 and 59.0), between two and eight it
// depends on k and s (512 x 64 x 4200, s = 7 47.7 and 59.2; 512 x 64 x 8200, s = 2 / 9 38.0 and 42.0 / 95.0 and 81.7; 256 x 64 x 16000,
// s = 2 / 7 52.8 and 52.0 / 114 and 92), beyond it wins (2048 x 64 x 8200, s = 2 / 7 75.0 and 67.1 / 121 and 97.5; 8192 x 64 x 4200,
// s = 7 247 and 140), and where s k passes the int32 range it replaces the split over k-blocks (300 x 10 x 100000, s = 7 845
// and 280).
int gemm_vectors_parts(int m, int n, int k, int s) { return vectors_parts(s, ((m < n ? n : m) + 31) / 32, round_up(k, kPad)); }

bool gemm_vectors_handles(int m, int n, int k, int sA, int sB, int cA, int cB, bool nearest, int lda, int ldb)
{
    const int sh = m < n ? m : n, lg = m < n ? n : m;
    if (sA != sB || cA != sA || cB != sB || sA < 2 || sA > (nearest ? 8 : 9)) return false;
    if (sh < 1 || sh > 64 || lg < 256 || k <= 2048 || scale_split_handles(m, n, k)) return false;
    if ((m < n ? ldb : lda) >= 1 << 24) return false;                // (32-bit lane offsets)
    return (long long)lg * k >= (2LL << 20) && gemm_vectors_parts(m, n, k, sA) > 0;
}

hipError_t launch_gemm_vectors(int m, int n, int k, const double *A, int lda, const double *B, int ldb, int s, bool nearest,
                               const unsigned long long *maxA, const unsigned long long *maxB, int32_t *eA, int32_t *eB,
                               int8_t *pA, int8_t *pB, double *C, int ldc, int Q, hipStream_t st)
{
    const bool short_a = m < n;
    const int L = short_a ? n : m, tiles = (L + 31) / 32, kp = round_up(k, kPad);
    const int parts = vectors_parts(s, tiles, kp);
    if (parts < 1) return hipErrorInvalidValue;
    const int steps = (kp / 128 + parts - 1) / parts;
    // the slots, parts * tiles * s * 8192 bytes, lie in the room for the long operand's planes, tiles * 32 * s * kp bytes or
    // more (parts <= kp / 512)
    int32_t *slots = parts > 1 ? (int32_t *)(short_a ? pB : pA) : nullptr;
    note_gemm_kernel("gemm_vectors_kernel<%d> tile %s, long operand sliced on the way, %d parts of k", s, short_a ? "64x32" : "32x64", parts);
    auto launch = [&](auto SC, auto NC, auto TC) -> hipError_t {
        constexpr int S = decltype(SC)::value;
        constexpr bool NEAREST = decltype(NC)::value, SHORT_A = decltype(TC)::value;
        auto kern = gemm_vectors_kernel<S, NEAREST, SHORT_A>;
        static std::atomic<unsigned long long> configured{0};
        if (hipError_t e = allow_dynamic_lds((const void *)kern, CfgVectors<S, NEAREST>::LDS, configured); e != hipSuccess) return e;
        kern<<<dim3(tiles, parts), 512, CfgVectors<S, NEAREST>::LDS, st>>>((const unsigned long long *)(SHORT_A ? B : A), SHORT_A ? ldb : lda, L,
                                                                 SHORT_A ? maxB : maxA, SHORT_A ? eB : eA, SHORT_A ? pA : pB, SHORT_A ? eA : eB,
                                                                 C, ldc, m, n, k, kp / kFrag, steps * 4, slots, Q);
        return hipGetLastError();
    };
    auto by_side = [&](auto SC, auto NC) { return short_a ? launch(SC, NC, std::true_type{}) : launch(SC, NC, std::false_type{}); };
    auto by_rule = [&](auto SC) -> hipError_t {
        if (!nearest) return by_side(SC, std::false_type{});
        if constexpr (decltype(SC)::value <= 8) return by_side(SC, std::true_type{});      // (nine: a second window, spills)
        return hipErrorInvalidValue;
    };
    hipError_t err = hipErrorInvalidValue;
    switch (s) {
#define OZ_CASE(S_) case S_: err = by_rule(std::integral_constant<int, S_>{}); break;
        OZ_CASE(2) OZ_CASE(3) OZ_CASE(4) OZ_CASE(5) OZ_CASE(6) OZ_CASE(7) OZ_CASE(8) OZ_CASE(9)
#undef OZ_CASE
    }
    if (err != hipSuccess || !slots) return err;
    finish_vectors_kernel<<<tiles, 512, 0, st>>>(slots, parts, s, short_a, eA, eB, C, ldc, m, n, Q);
    return hipGetLastError();
}

}  // namespace oz
