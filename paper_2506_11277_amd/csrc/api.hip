// extern "C" boundary of libozimmu: argument checks, workspace carve-up, kernel sequencing.
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>

#include "oz_common.h"

using namespace oz;

namespace oz {
static thread_local char t_last_kernel[160] = "";
void note_gemm_kernel(const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(t_last_kernel, sizeof(t_last_kernel), fmt, ap);
    va_end(ap);
}
const char *last_gemm_kernel() { return t_last_kernel; }
}  // namespace oz

namespace {

inline bool bad_matrix(int rows, int cols, const void *p, int ld)
{
    if (rows < 0 || cols < 0) return true;
    if (ld < (rows > 1 ? rows : 1)) return true;
    return rows > 0 && cols > 0 && p == nullptr;
}


// whether two column-major matrices share memory (between their first and last entries)
inline bool overlap(const double *X, int rx, int cx, int ldx, const double *Y, int ry, int cy, int ldy)
{
    const auto x0 = (uintptr_t)X, y0 = (uintptr_t)Y;
    return x0 < y0 + 8 * ((uintptr_t)(cy - 1) * ldy + ry) && y0 < x0 + 8 * ((uintptr_t)(cx - 1) * ldx + rx);
}

#define OZ_TRY(expr)                                        \
    do {                                                    \
        hipError_t e__ = (expr);                            \
        if (e__ != hipSuccess) return OZIMMU_HIP_ERROR;     \
    } while (0)

// Optional per-phase timing of ozimmu_dgemm with HIP events recorded on the caller's stream.  One timer per
// process, guarded by a mutex; a call claims its slot of four events when it starts, so calls from several threads
// never share events (their phases then interleave on the device, which is why the header asks for one thread).
struct Profile {
    std::mutex mutex;
    bool on = false;
    int capacity = 0, calls = 0;
    hipEvent_t *ev = nullptr;   // 4 events per call: start, after scales, after split, after gemm
} g_prof;

// slot of this call's events, or null when the timer is off or full
inline hipEvent_t *prof_claim()
{
    std::lock_guard<std::mutex> lock(g_prof.mutex);
    if (!g_prof.on || g_prof.calls >= g_prof.capacity) return nullptr;
    return g_prof.ev + 4 * (size_t)g_prof.calls++;
}

inline void prof_mark(hipEvent_t *slot, int phase, hipStream_t st)
{
    if (slot) (void)hipEventRecord(slot[phase], st);
}

}  // namespace

extern "C" {

const char *ozimmu_status_string(int status)
{
    switch (status) {
        case OZIMMU_OK: return "ok";
        case OZIMMU_BAD_ARG: return "bad argument";
        case OZIMMU_NONFINITE: return "non-finite input";
        case OZIMMU_HIP_ERROR: return "HIP runtime error";
        case OZIMMU_UNREACHABLE: return "tolerance unreachable";
        case OZIMMU_TOO_LARGE: return "problem too large for the static workspace";
    }
    return "unknown status";
}

size_t ozimmu_workspace_bytes(int m, int n, int k, int s)
{
    if (m < 0 || n < 0 || k < 0 || s < 1 || s > OZIMMU_MAX_SLICES) return 0;
    return carve(m, n, k, s, s).total;
}

size_t ozimmu_workspace_bytes2(int m, int n, int k, int sA, int sB, int all_products)
{
    if (m < 0 || n < 0 || k < 0 || sA < 1 || sA > OZIMMU_MAX_SLICES || sB < 1 || sB > OZIMMU_MAX_SLICES) return 0;
    return carve(m, n, k, sA, sB, all_products != 0).total;
}

size_t ozimmu_planes_bytes(char side, int rows, int cols, int s, int layout)
{
    if ((side != 'A' && side != 'B') || rows < 0 || cols < 0 || s < 1 || s > OZIMMU_MAX_SLICES) return 0;
    if (layout == OZIMMU_LAYOUT_PLAIN) return (size_t)s * rows * cols;
    if (layout != OZIMMU_LAYOUT_MFMA) return 0;
    const int R = side == 'A' ? rows : cols, K = side == 'A' ? cols : rows;
    return (size_t)s * round_up(R > 0 ? R : 1, kPad) * round_up(K > 0 ? K : 1, kPad);
}

size_t ozimmu_split_scratch_bytes(char side, int rows, int cols)
{
    if ((side != 'A' && side != 'B') || rows < 0 || cols < 0) return 0;
    const int nblk = side == 'A' ? rows : cols;
    return 256 + 8 * (size_t)(nblk > 0 ? nblk : 1);
}

// Pinned host memory that the last kernel of the estimators writes its three words into: a copy of 24 bytes to pageable memory takes
// 7 us longer (estimate and product, us, copy and kernel: 200 x 300 x 200 s = 6 49.4 and 41.9, 2944 x 704 x 491 s = 8 82.1 and 75.9). One allocation of 64 slots, made by the first call that
// gets it and kept; a call has a slot of its own until it has waited for its stream, and copies if none is free or the allocation fails (the next call tries again).
namespace {
constexpr int kWordSlots = 64, kWordStride = 8;               // 64 bytes each
struct {
    std::mutex mutex;
    std::atomic<unsigned long long *> base{nullptr};
    std::atomic<unsigned long long> free{0};
    std::atomic<bool> refuse{false};                          // test hook: allocations fail
} g_words;

class HostWords {
    int slot = -1;

    static unsigned long long *memory()
    {
        if (unsigned long long *p = g_words.base.load(std::memory_order_acquire)) return p;
        std::lock_guard<std::mutex> lock(g_words.mutex);
        if (unsigned long long *p = g_words.base.load(std::memory_order_acquire)) return p;
        void *p = nullptr;
        if (g_words.refuse) return nullptr;
        // (an allocation spoils a capture that is under way on another stream, unless the thread's mode is the relaxed one)
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        const hipError_t e = hipHostMalloc(&p, kWordSlots * kWordStride * 8, hipHostMallocPortable | hipHostMallocMapped);
        if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_words.free = ~0ULL;
        g_words.base.store((unsigned long long *)p, std::memory_order_release);
        return (unsigned long long *)p;
    }

public:
    volatile unsigned long long *host = nullptr;
    unsigned long long *device = nullptr;                     // null: none to be had
    HostWords()
    {
        unsigned long long *base = memory();
        if (!base) return;
        unsigned long long mask = g_words.free.load(std::memory_order_relaxed);
        while (mask && !g_words.free.compare_exchange_weak(mask, mask & (mask - 1), std::memory_order_acquire)) {}
        if (!mask) return;
        slot = __builtin_ctzll(mask);
        void *d = nullptr;
        if (hipHostGetDevicePointer(&d, base + slot * kWordStride, 0) != hipSuccess || !d) {
            (void)hipGetLastError();
            give_back();
            return;
        }
        host = base + slot * kWordStride;
        device = (unsigned long long *)d;
    }
    // Called once the stream has been waited for: where a launch or the wait failed, a kernel may still write to the slot, so nobody gets it again.
    void give_back()
    {
        if (slot >= 0) g_words.free.fetch_or(1ULL << slot, std::memory_order_release);
        slot = -1;
    }
    HostWords(const HostWords &) = delete;
    HostWords &operator=(const HostWords &) = delete;
};
}  // namespace

static int kappas(int m, int n, int k, const double *A, int lda, const double *B, int ldb, double *kA, double *kB,
                  void *workspace, size_t workspace_bytes, void *stream)
{
    if (bad_matrix(m, k, A, lda) || bad_matrix(k, n, B, ldb)) return OZIMMU_BAD_ARG;
    const Workspace w = carve(m, n, k, 1, 1);
    if (!workspace || workspace_bytes < w.total || ((uintptr_t)workspace & 255)) return OZIMMU_BAD_ARG;
    hipStream_t st = (hipStream_t)stream;
    char *ws = (char *)workspace;
    auto at = [&](size_t off) { return (unsigned long long *)(ws + off); };
    HostWords words;
    OZ_TRY(launch_kappas(m, n, k, A, lda, B, ldb, at(w.off_header), at(w.off_maxA), at(w.off_minA), at(w.off_maxB), at(w.off_minB),
                         (int32_t *)(ws + w.off_expA), w.mp, (int32_t *)(ws + w.off_expB), w.np, words.device, st));
    unsigned long long host[3];
    if (!words.device) OZ_TRY(hipMemcpyAsync(host, ws + w.off_header, sizeof(host), hipMemcpyDeviceToHost, st));
    OZ_TRY(hipStreamSynchronize(st));
    if (words.device)
        for (int i = 0; i < 3; ++i) host[i] = words.host[i];
    words.give_back();
    if (host[0] & 1ULL) return OZIMMU_NONFINITE;
    double ratioA, ratioB;
    std::memcpy(&ratioA, &host[1], 8);
    std::memcpy(&ratioB, &host[2], 8);
    *kA = 2.0 * ratioA;
    *kB = 2.0 * ratioB;
    return OZIMMU_OK;
}

int ozimmu_estimate_slices(int m, int n, int k, const double *A, int lda, const double *B, int ldb, double tol,
                           int *s_out, double *kappa, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!s_out || !(tol > 0.0)) return OZIMMU_BAD_ARG;
    double kA, kB;
    int rc = kappas(m, n, k, A, lda, B, ldb, &kA, &kB, workspace, workspace_bytes, stream);
    if (rc) return rc;
    if (kappa) { kappa[0] = kA; kappa[1] = kB; }
    // left-hand side of eq. (err-bound) with s_A = s_B = s, tried for s = 1, 2, ...
    for (int s = 1; s <= OZIMMU_MAX_SLICES; ++s) {
        const double lhs = std::ldexp(kA, -s * kSliceBits) + std::ldexp(kB, -s * kSliceBits);
        if (lhs <= tol) { *s_out = s; return OZIMMU_OK; }
    }
    *s_out = OZIMMU_MAX_SLICES;
    return OZIMMU_UNREACHABLE;
}

static int chi(int sA, int sB)
{
    const int sM = sA > sB ? sA : sB, sm = sA > sB ? sB : sA;
    return sm * (2 * sM - sm + 1) / 2;
}

int ozimmu_estimate_slices2(int m, int n, int k, const double *A, int lda, const double *B, int ldb, double tol,
                            int *sA_out, int *sB_out, double *kappa, void *workspace, size_t workspace_bytes,
                            void *stream)
{
    if (!sA_out || !sB_out || !(tol > 0.0)) return OZIMMU_BAD_ARG;
    double kA, kB;
    int rc = kappas(m, n, k, A, lda, B, ldb, &kA, &kB, workspace, workspace_bytes, stream);
    if (rc) return rc;
    if (kappa) { kappa[0] = kA; kappa[1] = kB; }
    // every (sA, sB) that meets eq. (err-bound); keep the one with the fewest products chi(sA, sB),
    // then the smaller sA + sB, then the smaller sA
    bool found = false;
    int bA = OZIMMU_MAX_SLICES, bB = OZIMMU_MAX_SLICES;
    for (int sA = 1; sA <= OZIMMU_MAX_SLICES; ++sA)
        for (int sB = 1; sB <= OZIMMU_MAX_SLICES; ++sB) {
            const double lhs = std::ldexp(kA, -sA * kSliceBits) + std::ldexp(kB, -sB * kSliceBits);
            if (!(lhs <= tol)) continue;
            const int c = chi(sA, sB), cb = chi(bA, bB);
            if (!found || c < cb || (c == cb && (sA + sB < bA + bB || (sA + sB == bA + bB && sA < bA)))) {
                found = true;
                bA = sA;
                bB = sB;
            }
        }
    *sA_out = bA;
    *sB_out = bB;
    return found ? OZIMMU_OK : OZIMMU_UNREACHABLE;
}

int ozimmu_split2(char side, int rows, int cols, const double *X, int ldx, int s, int splitting, int8_t *planes,
                  int32_t *exps, int layout, void *scratch, void *stream)
{
    if ((side != 'A' && side != 'B') || bad_matrix(rows, cols, X, ldx) || s < 1 || s > OZIMMU_MAX_SLICES ||
        (splitting != OZIMMU_SPLIT_TRUNCATE && splitting != OZIMMU_SPLIT_NEAREST) ||
        (layout != OZIMMU_LAYOUT_PLAIN && layout != OZIMMU_LAYOUT_MFMA) || !scratch || ((uintptr_t)scratch & 255))
        return OZIMMU_BAD_ARG;
    const int nblk = side == 'A' ? rows : cols;
    if (nblk > 0 && !exps) return OZIMMU_BAD_ARG;
    if (ozimmu_planes_bytes(side, rows, cols, s, layout) > 0 && !planes) return OZIMMU_BAD_ARG;
    hipStream_t st = (hipStream_t)stream;
    auto *hdr = (unsigned long long *)scratch;
    auto *maxbits = hdr + 32;
    OZ_TRY(launch_clear_header(hdr, st));
    OZ_TRY(launch_reduce(side, rows, cols, X, ldx, maxbits, (unsigned int *)hdr, st));
    const bool nearest = splitting == OZIMMU_SPLIT_NEAREST;
    OZ_TRY(launch_finalize(maxbits, exps, nblk, nearest ? 1 : 0, st));
    OZ_TRY(launch_split(side, rows, cols, X, ldx, s, exps, planes, layout, nearest, st));
    return OZIMMU_OK;
}

int ozimmu_split(char side, int rows, int cols, const double *X, int ldx, int s, int8_t *planes, int32_t *exps,
                 int layout, void *scratch, void *stream)
{
    return ozimmu_split2(side, rows, cols, X, ldx, s, OZIMMU_SPLIT_TRUNCATE, planes, exps, layout, scratch, stream);
}

int ozimmu_max_level_diagonals(int k, int sA, int sB)
{
    if (k < 0 || sA < 1 || sA > OZIMMU_MAX_SLICES || sB < 1 || sB > OZIMMU_MAX_SLICES) return 0;
    // A diagonal holds at most min(sA, sB) products of k terms of magnitude at most 127^2.  In units of the
    // last diagonal of a level of Q diagonals, the level and each of its partial sums are integers below
    //     min(sA, sB) k 127^2 (1 + 2^7 + ... + 2^{7(Q-1)});
    // they are binary64 numbers while that stays below 2^53.
    const long long per_diag = (long long)(sA < sB ? sA : sB) * (k > 0 ? k : 1) * 127 * 127;   // < 2^51
    int Q = 0;
    long long geo = 0;                         // 1 + 2^7 + ... + 2^{7(Q-1)}
    while (Q < 8) {
        const long long next = geo * 128 + 1;
        if ((__int128)per_diag * next >= ((__int128)1 << 53)) break;
        geo = next;
        ++Q;
    }
    return Q;
}

static int dgemm_impl(int m, int n, int k, const double *A, int lda, const double *B, int ldb, double *C, int ldc,
                      int sA, int sB, bool all_products, int splitting, int Q, void *workspace,
                      size_t workspace_bytes, void *stream)
{
    if (bad_matrix(m, k, A, lda) || bad_matrix(k, n, B, ldb) || bad_matrix(m, n, C, ldc) || sA < 1 ||
        sA > OZIMMU_MAX_SLICES || sB < 1 || sB > OZIMMU_MAX_SLICES ||
        (splitting != OZIMMU_SPLIT_TRUNCATE && splitting != OZIMMU_SPLIT_NEAREST) || Q < 1 ||
        Q > ozimmu_max_level_diagonals(k, sA, sB))
        return OZIMMU_BAD_ARG;
    const bool nearest = splitting == OZIMMU_SPLIT_NEAREST;
    const Workspace w = carve(m, n, k, sA, sB, all_products);
    if (!workspace || workspace_bytes < w.total || ((uintptr_t)workspace & 255)) return OZIMMU_BAD_ARG;
    // exact conversion of a diagonal sum to binary64 needs s * k * 127^2 < 2^53: true for every int k
    hipStream_t st = (hipStream_t)stream;
    char *ws = (char *)workspace;
    hipEvent_t *prof = (m > 0 && n > 0) ? prof_claim() : nullptr;
    prof_mark(prof, 0, st);
    auto *eA = (int32_t *)(ws + w.off_expA), *eB = (int32_t *)(ws + w.off_expB);
    auto *pA = (int8_t *)(ws + w.off_planesA), *pB = (int8_t *)(ws + w.off_planesB);
    // short contractions: one launch for exponents and slices; else two for the maxima of both operands, one for the rest
    auto *maxA = (unsigned long long *)(ws + w.off_maxA), *maxB = (unsigned long long *)(ws + w.off_maxB);
    auto *hdr = (unsigned long long *)(ws + w.off_header);
    // (w.cA, w.cB: the counts the GEMM runs with -- counts that differ little run as equal ones, zero slices appended)
    // (the long operand is read while C is written: a C that lies in it takes the general way, whose kernels that write C
    // read planes only)
    if (w.path == kPathFused && !all_products && fused_automatic() && gemm_vectors_handles(m, n, k, sA, sB, w.cA, w.cB, nearest, lda, ldb) &&
        !(m < n ? overlap(C, m, n, ldc, B, k, n, ldb) : overlap(C, m, n, ldc, A, m, k, lda))) {
        OZ_TRY(launch_scales_fused(m, n, k, A, lda, B, ldb, hdr, maxA, maxB, eA, w.mp, eB, w.np, nearest ? 1 : 0, false, false, st));
        prof_mark(prof, 1, st);
        OZ_TRY(launch_split_both(m, n, k, A, lda, B, ldb, sA, sB, w.cA, w.cB, maxA, maxB, eA, eB, m < n ? pA : nullptr,
                                 m < n ? nullptr : pB, nearest, st));
        prof_mark(prof, 2, st);
        OZ_TRY(launch_gemm_vectors(m, n, k, A, lda, B, ldb, sA, nearest, maxA, maxB, eA, eB, pA, pB, C, ldc, Q, st));
        prof_mark(prof, 3, st);
        return OZIMMU_OK;
    }
    // the smallest products: one launch for everything (operands are read while C is written)
    if (!all_products && sA == sB && w.path == kPathFused && w.cA == sA && fused_automatic() && gemm_eighths_whole_handles(m, n, k, sA, nearest) &&
        !overlap(C, m, n, ldc, A, m, k, lda) && !overlap(C, m, n, ldc, B, k, n, ldb)) {
        prof_mark(prof, 1, st);
        prof_mark(prof, 2, st);
        OZ_TRY(launch_gemm_eighths_whole(m, n, k, A, lda, B, ldb, sA, nearest, eA, eB, pA, pB, hdr, w.off_minA, C, ldc, Q, st));
        prof_mark(prof, 3, st);
        return OZIMMU_OK;
    }
    if (scale_split_handles(m, n, k)) {
        prof_mark(prof, 1, st);
        OZ_TRY(launch_scale_split(m, n, k, A, lda, B, ldb, sA, sB, w.cA, w.cB, eA, eB, pA, pB, nearest, hdr, w.off_minA, st));
    } else {
        OZ_TRY(launch_scales_fused(m, n, k, A, lda, B, ldb, hdr, maxA, maxB, eA, w.mp, eB, w.np, nearest ? 1 : 0,
                                   m == 0 || n == 0, true, st));
        if (m == 0 || n == 0) return OZIMMU_OK;
        prof_mark(prof, 1, st);
        OZ_TRY(launch_split_both(m, n, k, A, lda, B, ldb, sA, sB, w.cA, w.cB, maxA, maxB, eA, eB, pA, pB, nearest, st));
    }
    prof_mark(prof, 2, st);
    const int cA = w.cA, cB = w.cB;
    // 10 ... 20 slices whose contraction is one int32 block: diagonals in passes, where that is the faster way (blocks, whose
    // planes may hold more slices per entry: equal counts only, different ones have fewer products)
    const bool triangle = cA == cB && !all_products && (w.path == kPathFused || (w.path == kPathBlocks && sA == sB));
    const int S = w.path == kPathBlocks ? sA : cA;
    const PassShape shape = triangle && fused_automatic() && fused_single_block(S, S, k) ? gemm_passes_shape(S, m, n, w.kp, Q) : kNoPasses;
    if (shape != kNoPasses) {
        OZ_TRY(launch_gemm_passes(shape, S, m, n, w.kp, cA, pA, pB, eA, eB, C, ldc, Q, st));
    } else if (w.path == kPathBlocks) {
        OZ_TRY(launch_gemm_blocks(m, n, w.kp, sA, sB, all_products, pA, pB, eA, eB, C, ldc,
                                  (long long *)(ws + w.off_totals), Q, st));
    } else if (w.path == kPathFused) {
        long long *totals = fused_single_block(cA, cB, k) ? nullptr : (long long *)(ws + w.off_totals);
        OZ_TRY(launch_gemm_fused(m, n, w.kp, cA, cB, all_products, pA, pB, eA, eB, C, ldc, nullptr, totals, Q, st));
    } else {
        const int dmax = all_products ? cA + cB : (cA > cB ? cA : cB) + 1;
        long long *totals = banded_totals_bytes(cA, cB, k) ? (long long *)(ws + w.off_totals) : nullptr;
        OZ_TRY(launch_gemm_banded(m, n, w.kp, cA, cB, dmax, pA, pB, eA, eB, C, ldc, totals, Q, st));
    }
    prof_mark(prof, 3, st);
    return OZIMMU_OK;
}

int ozimmu_dgemm(int m, int n, int k, const double *A, int lda, const double *B, int ldb, double *C, int ldc, int s,
                 void *workspace, size_t workspace_bytes, void *stream)
{
    return dgemm_impl(m, n, k, A, lda, B, ldb, C, ldc, s, s, false, OZIMMU_SPLIT_TRUNCATE, 1, workspace,
                      workspace_bytes, stream);
}

int ozimmu_dgemm2(int m, int n, int k, const double *A, int lda, const double *B, int ldb, double *C, int ldc,
                  int sA, int sB, int all_products, void *workspace, size_t workspace_bytes, void *stream)
{
    return dgemm_impl(m, n, k, A, lda, B, ldb, C, ldc, sA, sB, all_products != 0, OZIMMU_SPLIT_TRUNCATE, 1, workspace,
                      workspace_bytes, stream);
}

int ozimmu_dgemm3(int m, int n, int k, const double *A, int lda, const double *B, int ldb, double *C, int ldc,
                  int sA, int sB, int all_products, int splitting, int level_diagonals, void *workspace,
                  size_t workspace_bytes, void *stream)
{
    return dgemm_impl(m, n, k, A, lda, B, ldb, C, ldc, sA, sB, all_products != 0, splitting, level_diagonals,
                      workspace, workspace_bytes, stream);
}

// ---- the entry point that allocates nothing ----------------------------------------------------------------
// Its workspace is this file-scope device array: every GPU the library runs on holds one copy of it, at an address
// of its own, until the process ends.  In host code the array's name is only a handle for hipGetSymbolAddress; the
// address that kernels and copies take is looked up once per device (with that device current) and kept.
static __device__ __align__(256) unsigned char scratch[OZIMMU_STATIC_WORKSPACE_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};

// device address of `scratch` on the current device (null on failure)
void *static_workspace()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}
}  // namespace

int ozimmu_dgemm_static(int m, int n, int k, const double *A, int lda, const double *B, int ldb, double *C, int ldc,
                        int s, void *stream)
{
    if (m < 0 || n < 0 || k < 0 || s < 1 || s > OZIMMU_MAX_SLICES) return OZIMMU_BAD_ARG;
    if (carve(m, n, k, s, s).total > (size_t)OZIMMU_STATIC_WORKSPACE_BYTES) return OZIMMU_TOO_LARGE;
    void *ws = static_workspace();
    if (!ws) return OZIMMU_HIP_ERROR;
    // every kernel of the path clears what it needs to find cleared (header, maxima, split-k totals) with fill
    // kernels of its own, so the contents the last call left behind do not matter
    return dgemm_impl(m, n, k, A, lda, B, ldb, C, ldc, s, s, false, OZIMMU_SPLIT_TRUNCATE, 1, ws,
                      (size_t)OZIMMU_STATIC_WORKSPACE_BYTES, stream);
}

int ozimmu_profile_start(int max_calls)
{
    std::lock_guard<std::mutex> lock(g_prof.mutex);
    if (max_calls < 1 || max_calls > 4096 || g_prof.on) return OZIMMU_BAD_ARG;
    g_prof.ev = new hipEvent_t[4 * (size_t)max_calls];
    for (int i = 0; i < 4 * max_calls; ++i)
        if (hipEventCreate(&g_prof.ev[i]) != hipSuccess) {
            // give back what was created: the timer stays off and empty
            for (int j = 0; j < i; ++j) (void)hipEventDestroy(g_prof.ev[j]);
            delete[] g_prof.ev;
            g_prof.ev = nullptr;
            g_prof.capacity = g_prof.calls = 0;
            return OZIMMU_HIP_ERROR;
        }
    g_prof.capacity = max_calls;
    g_prof.calls = 0;
    g_prof.on = true;
    return OZIMMU_OK;
}

int ozimmu_profile_stop(int *calls, float *phase_ms)
{
    std::lock_guard<std::mutex> lock(g_prof.mutex);
    if (!g_prof.on || !calls || !phase_ms) return OZIMMU_BAD_ARG;
    g_prof.on = false;
    int rc = OZIMMU_OK;
    double sum[3] = {0, 0, 0};
    for (int c = 0; c < g_prof.calls; ++c) {
        hipEvent_t *e = g_prof.ev + 4 * c;
        if (hipEventSynchronize(e[3]) != hipSuccess) rc = OZIMMU_HIP_ERROR;
        for (int p = 0; p < 3 && rc == OZIMMU_OK; ++p) {
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, e[p], e[p + 1]) != hipSuccess) rc = OZIMMU_HIP_ERROR;
            sum[p] += ms;
        }
    }
    for (int i = 0; i < 4 * g_prof.capacity; ++i) (void)hipEventDestroy(g_prof.ev[i]);
    delete[] g_prof.ev;
    g_prof.ev = nullptr;
    *calls = g_prof.calls;
    for (int p = 0; p < 3; ++p) phase_ms[p] = g_prof.calls ? (float)(sum[p] / g_prof.calls) : 0.f;
    g_prof.capacity = g_prof.calls = 0;
    return rc;
}

int ozimmu_check(void *workspace, void *stream)
{
    if (!workspace) return OZIMMU_BAD_ARG;
    unsigned int flags = 0;
    hipStream_t st = (hipStream_t)stream;
    // a call that formed scales and slices in one launch has left a word per work-group instead of the flag: they are
    // brought together on the device, so that one copy and one synchronisation do whatever the size
    OZ_TRY(launch_collect_bad((unsigned long long *)workspace, st));
    OZ_TRY(hipMemcpyAsync(&flags, workspace, sizeof(flags), hipMemcpyDeviceToHost, st));
    OZ_TRY(hipStreamSynchronize(st));
    return (flags & 1u) ? OZIMMU_NONFINITE : OZIMMU_OK;
}

int ozimmu_get_exponents(int m, int n, int k, int s, const void *workspace, int32_t *eA, int32_t *eB, void *stream)
{
    if (m < 0 || n < 0 || k < 0 || s < 1 || s > OZIMMU_MAX_SLICES || !workspace) return OZIMMU_BAD_ARG;
    const Workspace w = carve(m, n, k, s, s);
    hipStream_t st = (hipStream_t)stream;
    const char *ws = (const char *)workspace;
    if (eA && m) OZ_TRY(hipMemcpyAsync(eA, ws + w.off_expA, 4 * (size_t)m, hipMemcpyDeviceToDevice, st));
    if (eB && n) OZ_TRY(hipMemcpyAsync(eB, ws + w.off_expB, 4 * (size_t)n, hipMemcpyDeviceToDevice, st));
    return OZIMMU_OK;
}

const char *ozimmu_last_gemm_kernel(void) { return last_gemm_kernel(); }

long long ozimmu_debug_setup_threads(int m, int n, int k) { return scale_split_threads(m, n, k); }

int ozimmu_debug_vectors_parts(int m, int n, int k, int s)
{
    if (m <= 0 || n <= 0 || k <= 0 || s < 1 || s > OZIMMU_MAX_SLICES || !fused_automatic()) return 0;
    return gemm_vectors_handles(m, n, k, s, s, s, s, false, m, k) ? gemm_vectors_parts(m, n, k, s) : 0;
}

int ozimmu_debug_panel_bytes(long long bytes)
{
    fused_set_panel_bytes(bytes);
    return OZIMMU_OK;
}

int ozimmu_debug_small_tile_limit(long long tiles)
{
    if (tiles < -1) return OZIMMU_BAD_ARG;
    fused_set_small_tile_limit(tiles);
    return OZIMMU_OK;
}

int ozimmu_debug_host_words(int refuse)
{
    std::lock_guard<std::mutex> lock(g_words.mutex);
    g_words.refuse = refuse != 0;
    if (refuse) {
        g_words.base = nullptr;
        g_words.free = 0;
    }
    return __builtin_popcountll(g_words.free.load());
}

int ozimmu_debug_tile_choice(int choice)
{
    if (choice < 0 || choice > 2) return OZIMMU_BAD_ARG;
    fused16_set_tile_choice(choice);
    return OZIMMU_OK;
}

// whether the last product on this workspace left the planes of both operands; waits for the stream
static int planes_of_both(const void *workspace, hipStream_t st)
{
    unsigned long long word = 0;
    OZ_TRY(hipMemcpyAsync(&word, (const unsigned long long *)workspace + kHeaderPlanes, sizeof(word), hipMemcpyDeviceToHost, st));
    OZ_TRY(hipStreamSynchronize(st));
    return word == kNoPlanes ? OZIMMU_BAD_ARG : OZIMMU_OK;
}

int ozimmu_debug_diagonals(int m, int n, int k, int s, const void *workspace, int32_t *D, void *stream)
{
    if (m <= 0 || n <= 0 || k < 0 || !workspace || !D || !fused_single_block(s, s, k)) return OZIMMU_BAD_ARG;
    if (int rc = planes_of_both(workspace, (hipStream_t)stream)) return rc;
    const Workspace w = carve(m, n, k, s, s);
    const char *ws = (const char *)workspace;
    OZ_TRY(launch_gemm_fused(m, n, w.kp, s, s, false, (const int8_t *)(ws + w.off_planesA),
                             (const int8_t *)(ws + w.off_planesB),
                             nullptr, nullptr, nullptr, m, D, nullptr, 1, (hipStream_t)stream));
    return OZIMMU_OK;
}

int ozimmu_debug_slice_product(int m, int n, int k, int s, const void *workspace, int l, int h, int k0, int k1,
                               int32_t *P, void *stream)
{
    if (m <= 0 || n <= 0 || k < 0 || s < 1 || s > OZIMMU_MAX_SLICES || !workspace || !P || l < 1 || l > s || h < 1 ||
        h > s || k0 < 0 || k1 < k0 || k1 > k || (k0 % kFrag) != 0 || (long long)(k1 - k0) > kMaxInt32K)
        return OZIMMU_BAD_ARG;
    const Workspace w = carve(m, n, k, s, s);
    const char *ws = (const char *)workspace;
    // the planes are zero beyond k, so the last (partial) fragment may be read whole
    const int kb_begin = k0 / kFrag, kb_end = (k1 + kFrag - 1) / kFrag;
    if (k1 != k && (k1 % kFrag) != 0) return OZIMMU_BAD_ARG;
    if (int rc = planes_of_both(workspace, (hipStream_t)stream)) return rc;
    OZ_TRY(launch_gemm_generic(m, n, w.kp, s, (const int8_t *)(ws + w.off_planesA),
                               (const int8_t *)(ws + w.off_planesB), nullptr, nullptr, nullptr, m, l, h, kb_begin,
                               kb_end, P, (hipStream_t)stream));
    return OZIMMU_OK;
}

}  // extern "C"
