"""The routes the library takes by itself at sizes that do not fill the chip, against the oracle, bit for bit.

(The other parity tests steer the choice of kernel; nothing is steered here.)  Every row of A and column of B has a
scale of its own, so a sample of rows and columns of C is the oracle's product of these rows and columns."""
import gc
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle
from paper_2506_11277_amd import ozimmu, workloads


def bits(x):
    return np.asarray(x, dtype=np.float64).view(np.int64)


def sample(n):
    """Edges of 16, 32, 64 and 128, the ends and a few between."""
    picks = {0, 1, 15, 16, 31, 32, 63, 64, 127, 128, n // 2, n - 33, n - 2, n - 1} | set(range(3, n, max(1, n // 9)))
    return np.array(sorted(p for p in picks if 0 <= p < n))


def check(C, A, B, sA, sB, **kw):
    rows, cols = sample(C.shape[0]), sample(C.shape[1])
    want = oracle.dgemm3(np.asfortranarray(A[rows]), np.asfortranarray(B[:, cols]), sA, sB, **kw)
    got = C.cpu().numpy()[np.ix_(rows, cols)]
    assert np.array_equal(bits(got), bits(want)), (C.shape, sA, sB, kw, ozimmu.last_gemm_kernel())


def special(A, B):
    """Zero, subnormal, tiny, huge and sign-only entries in a few rows and columns."""
    A[0, :] = 0.0
    A[-1, ::2] = 5e-324
    A[A.shape[0] // 2, :] = -(1.0 - 2.0 ** -53)
    B[:, 0] = -0.0
    B[::3, -1] = -1.0e300
    B[:, B.shape[1] // 2] = 1.0 - 2.0 ** -53


@pytest.mark.parametrize("s", range(1, 11))
@pytest.mark.parametrize("m,n,k,kernel", [
    (1, 1, 1, "whole"), (33, 31, 130, "eighths"), (161, 1300, 70, "whole"), (300, 610, 140, "eighths"), (512, 512, 64, "whole"), (97, 70, 1000, "eighths"), (40, 300, 2100, "eighths"),
    (545, 700, 1, "eighths"), (700, 545, 97, "eighths"), (640, 700, 128, "eighths"),      # (fewer k-blocks than wavefronts)
    (705, 961, 65, "halves"), (1024, 1000, 129, "halves"), (65, 8000, 700, "halves"),
    (705, 961, 2049, "halves"), (1000, 1000, 1100, "halves"),
])
def test_contraction_divided_within_a_work_group(m, n, k, kernel, s):
    # tiles of 32 x 32 (k in eighths) and of 64 x 64 (k in halves): every slice count, k-blocks that do not divide
    # evenly, plain order and levels of two diagonals
    print(f"{m}x{n}x{k} s={s}", flush=True)
    A, B = workloads.lognormal(m, n, k, 1.0, 7 + s)
    if m > 4:
        special(A, B)
    dA, dB = ozimmu.to_colmajor(A), ozimmu.to_colmajor(B)
    C = ozimmu.dgemm(dA, dB, s)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256 and 2 <= s <= 9:
        if kernel == "halves" and (s >= 7 or (s <= 3 and k >= 1024)):
            kernel = "halves16"
        if kernel == "whole" or (kernel == "eighths" and s <= 4 and k <= 256 and m < 512):
            kernel = "eighths_whole"
        assert ozimmu.last_gemm_kernel().startswith(f"gemm_{kernel}_kernel<{s}>"), ozimmu.last_gemm_kernel()
    check(C, A, B, s, s)
    check(ozimmu.dgemm3(dA, dB, s, s, splitting=ozimmu.SPLIT_NEAREST, level_diagonals=2), A, B, s, s, nearest=True, Q=2)


WHOLE = "gemm_eighths_whole_kernel<"


# Scales, slices and product in one launch: edges of tiles, half k-blocks that are whole, ragged and empty, both depths, the ends of the rule; the
# planes, exponents and the non-finite report that it leaves
@pytest.mark.parametrize("s", range(1, 11))
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (33, 31, 15), (64, 32, 128), (100, 130, 113), (512, 500, 97), (31, 65, 129), (200, 190, 255), (480, 512, 256)])
def test_everything_in_one_launch(m, n, k, s):
    A, B = workloads.pow2_scaled(m, n, k, 30, 3 + k)
    if m > 4:
        special(A, B)
    dA, dB = ozimmu.colmajor_empty(m + 1, k)[1:, :], ozimmu.colmajor_empty(k + 3, n)[3:, :]
    dA.copy_(torch.as_tensor(A))
    dB.copy_(torch.as_tensor(B))
    ws = ozimmu.alloc_workspace(m, n, k, s)
    ws.fill_(0x5a)
    big = ozimmu.colmajor_empty(m + 3, n).fill_(7.0)
    C = ozimmu.dgemm(dA, dB, s, C=big[2:m + 2, :], workspace=ws, check_finite=True)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert (WHOLE in ozimmu.last_gemm_kernel()) == (k <= 128 or s <= 4), ozimmu.last_gemm_kernel()
    check(C, A, B, s, s)
    assert (big[:2] == 7).all() and (big[m + 2:] == 7).all()
    other = ozimmu.alloc_workspace(m, n, k, s)
    try:
        ozimmu.debug_small_tile_limit(256)
        want = ozimmu.dgemm(dA, dB, s, workspace=other)
    finally:
        ozimmu.debug_small_tile_limit(-1)
    assert WHOLE not in ozimmu.last_gemm_kernel() and torch.equal(C, want)
    for x, y in zip(ozimmu.get_exponents(m, n, k, s, ws), ozimmu.get_exponents(m, n, k, s, other)):
        assert torch.equal(x, y)
    assert torch.equal(ozimmu.debug_diagonals(m, n, k, s, ws), ozimmu.debug_diagonals(m, n, k, s, other))
    check(ozimmu.dgemm3(dA, dB, s, s, splitting=ozimmu.SPLIT_NEAREST, level_diagonals=2), A, B, s, s, nearest=True, Q=2)
    for X in (dA, dB):                       # the last entry of either operand is looked at
        X[-1, -1] = float("nan")
        with pytest.raises(ozimmu.OzimmuError):
            ozimmu.dgemm(dA, dB, s, workspace=ws, check_finite=True)
        X[-1, -1] = 0.0


def test_a_result_over_an_operand_takes_two_launches():
    m, s = 96, 3
    A, B = workloads.lognormal(m, m, m, 1.0, 8)
    dA, dB = ozimmu.to_colmajor(A), ozimmu.to_colmajor(B)
    want = ozimmu.dgemm(dA, dB, s)
    assert WHOLE in ozimmu.last_gemm_kernel()
    for X, Y, C in ((dA.clone(memory_format=torch.preserve_format), dB, 0), (dA, dB.clone(memory_format=torch.preserve_format), 1)):
        C = (X, Y)[C]
        ozimmu.dgemm(X, Y, s, C=C)
        assert WHOLE not in ozimmu.last_gemm_kernel() and torch.equal(C, want)


@pytest.mark.parametrize("m,n,k", [(5, 3, 1), (4, 9, 127), (64, 6, 128), (17, 33, 129), (70, 50, 1023), (70, 50, 1024), (31, 8, 1025),
                                   (9, 130, 2048), (33, 20, 2049), (65, 40, 4096), (7, 5, 4097), (9000, 3288, 40), (8200, 4100, 513),
                                   (12000, 300, 1100)])
@pytest.mark.parametrize("sA,sB,nearest", [(1, 1, False), (7, 7, True), (9, 9, False), (9, 10, True), (19, 18, False), (24, 32, True)])
def test_scales_and_slices_in_one_launch(m, n, k, sA, sB, nearest):
    # up to four sweeps over k (more: the test below), both panel heights, the limits of the rule, windows of slices that end on and off
    # a whole window, zero slices appended to the short operand, leading dimensions that are odd
    if m > 4000 and sA + sB > 19:
        pytest.skip("large shapes with one pair of windows only")
    A, B = workloads.pow2_scaled(m, n, k, 30, 11 + k)
    if m > 4 and k > 2:
        special(A, B)
    dA, dB = ozimmu.colmajor_empty(m + 1, k)[1:, :], ozimmu.colmajor_empty(k + 3, n)[:k, :]
    dA.copy_(torch.as_tensor(A))
    dB.copy_(torch.as_tensor(B))
    splitting = ozimmu.SPLIT_NEAREST if nearest else ozimmu.SPLIT_TRUNCATE
    check(ozimmu.dgemm3(dA, dB, sA, sB, splitting=splitting), A, B, sA, sB, nearest=nearest)


# operands of 4000000 bytes and planes of 16000000, the most whose slices are written through the caches, and of a little more; four and eight rows to a work-group
@pytest.mark.parametrize("nearest", [False, True])
@pytest.mark.parametrize("m,n,k,s", [(600, 400, 500, 8), (600, 401, 500, 8), (1203, 47, 400, 13), (6000, 250, 60, 20), (6000, 251, 60, 20), (7000, 1000, 60, 15), (7000, 1000, 250, 16), (1300, 1200, 1280, 10)])
def test_planes_written_through(m, n, k, s, nearest):
    A, B = workloads.lognormal(m, n, k, 1.0, 23 + s)
    special(A, B)
    splitting = ozimmu.SPLIT_NEAREST if nearest else ozimmu.SPLIT_TRUNCATE
    check(ozimmu.dgemm3(ozimmu.to_colmajor(A), ozimmu.to_colmajor(B), s, s, splitting=splitting), A, B, s, s, nearest=nearest)


# five to eight sweeps over k: four rows to a work-group (1100 x 1050: five, seven, eight; 4100 x 90: three of eight wavefronts), eight
# rows (2500 x 1700: five to eight; 3003 x 37: six, with a last work-group of three rows), the ends of the rule by bytes (2000 x 2100 x 4000 with 6 and 7
# slices)
@pytest.mark.parametrize("nearest", [False, True])
@pytest.mark.parametrize("m,n,k,s", [(1100, 1050, 2200, 7), (1100, 1050, 3401, 7), (1100, 1050, 4090, 7), (4100, 90, 1099, 3), (2500, 1700, 2490, 13),
                                     (2500, 1700, 2689, 13), (2500, 1700, 3200, 13), (2500, 1700, 4090, 13), (3003, 37, 2565, 13),
                                     (2000, 2100, 4000, 6), (2000, 2100, 4000, 7)])
def test_sweeps_of_the_one_launch_set_up(m, n, k, s, nearest):
    print(f"{m}x{n}x{k} s={s}", flush=True)
    assert ozimmu.lib().ozimmu_debug_setup_threads(m, n, k) > 0
    A, B = workloads.lognormal(m, n, k, 1.0, 17 + s)
    special(A, B)
    dA, dB = ozimmu.colmajor_empty(m + 1, k)[1:, :], ozimmu.colmajor_empty(k + 3, n)[:k, :]
    dA.copy_(torch.as_tensor(A))
    dB.copy_(torch.as_tensor(B))
    splitting = ozimmu.SPLIT_NEAREST if nearest else ozimmu.SPLIT_TRUNCATE
    ws = torch.empty(ozimmu.lib().ozimmu_workspace_bytes2(m, n, k, s, s, 0), dtype=torch.uint8, device="cuda")
    check(ozimmu.dgemm3(dA, dB, s, s, splitting=splitting, workspace=ws, check_finite=True), A, B, s, s, nearest=nearest)
    for X in (dA, dB):                       # the last entry of either operand is looked at
        X[-1, -1] = float("inf")
        with pytest.raises(ozimmu.OzimmuError):
            ozimmu.dgemm3(dA, dB, s, s, splitting=splitting, workspace=ws, check_finite=True)
        X[-1, -1] = 0.0


def test_more_rows_than_the_one_launch_set_up_has_threads_for():
    # 2^27 rows: the launch that forms scales and slices together would have 2^32 threads, the separate ones serve
    m, n, k, s = 2 ** 27 + 5, 1, 1, 1
    free, _ = torch.cuda.mem_get_info()
    if free < 40 << 30:
        pytest.skip("needs 40 GB of device memory")
    A = torch.arange(m, device="cuda", dtype=torch.float64).remainder_(1009).sub_(500).reshape(m, 1)
    B = torch.full((1, 1), 1.5, dtype=torch.float64, device="cuda")
    print(f"{m} rows", flush=True)
    C = ozimmu.dgemm(A, B, s, check_finite=True)
    rows = torch.as_tensor([0, 1, 2, 500, 1009, 2 ** 26, 2 ** 27 - 1, 2 ** 27, m - 1], device="cuda")
    want = oracle.dgemm(np.asfortranarray(A[rows].cpu().numpy()), np.array([[1.5]], order="F"), s)
    assert np.array_equal(bits(C[rows].cpu().numpy()), bits(want))


@pytest.mark.parametrize("k", [100, 3000, 5000])
def test_non_finite_is_reported_and_forgotten(k):
    # the report of a call replaces that of the call before it in the same workspace, whichever way either slices
    m, n, s = 70, 6000 if k == 3000 else 50, 3
    A, B = workloads.uniform(m, n, k, 3)
    ws = torch.empty(max(ozimmu.workspace_bytes(m, n, kk, s) for kk in (k, 100)), dtype=torch.uint8, device="cuda")
    dA, dB = ozimmu.to_colmajor(A), ozimmu.to_colmajor(B)
    small = ozimmu.to_colmajor(A[:, :100]), ozimmu.to_colmajor(B[:100])
    for X, at, value in [(dA, (0, 0), np.nan), (dA, (m - 1, k - 1), -np.inf), (dB, (k - 1, n - 1), np.inf), (dB, (k // 2, 17), np.nan)]:
        old = X[at].item()
        X[at] = value
        with pytest.raises(ozimmu.OzimmuError):
            ozimmu.dgemm(dA, dB, s, workspace=ws, check_finite=True)
        ozimmu.dgemm(*small, s, workspace=ws, check_finite=True)
        X[at] = old
        ozimmu.dgemm(dA, dB, s, workspace=ws, check_finite=True)
        assert ozimmu.estimate_slices(dA, dB, 1e-6, workspace=ws)[1] in (ozimmu.OK, ozimmu.UNREACHABLE)
        ozimmu.check(ws)


def test_check_takes_one_round_trip_whatever_the_size():
    # a million rows are 250 000 work-groups of the launch that forms scales and slices; the first and the last of them
    # report, and asking takes about as long as for a few rows
    def seconds(ws):
        best = 1.0
        for _ in range(7):
            torch.cuda.synchronize()
            t = time.perf_counter()
            ozimmu.check(ws)
            best = min(best, time.perf_counter() - t)
        return best

    took = {}
    for m in (300, 1_000_000):
        n, k, s = 20, 16, 1
        dA, dB = ozimmu.colmajor_empty(m, k).fill_(0.5), ozimmu.colmajor_empty(k, n).fill_(0.25)
        ws = ozimmu.alloc_workspace(m, n, k, s)
        C = ozimmu.colmajor_empty(m, n)
        for X, at in ((dA, (0, 0)), (dA, (m - 1, k - 1)), (dB, (k - 1, n - 1))):
            X[at] = float("nan")
            with pytest.raises(ozimmu.OzimmuError):
                ozimmu.dgemm(dA, dB, s, C=C, workspace=ws, check_finite=True)
            X[at] = 0.5
        ozimmu.dgemm(dA, dB, s, C=C, workspace=ws, check_finite=True)
        took[m] = seconds(ws)
    print(took, flush=True)
    assert took[1_000_000] < 8 * took[300], took


@pytest.mark.parametrize("m,n,k", [(9000, 64, 2100), (2100, 33, 5000), (300, 1, 30001), (64, 5000, 4500), (31, 260, 9000), (257, 40, 140000),
                                   (2, 700, 20000), (33000, 7, 4200), (260, 9, 304256)])
@pytest.mark.parametrize("s,nearest,Q", [(2, False, 1), (3, True, 2), (7, False, 1), (8, True, 1), (9, False, 3)])
def test_long_operand_sliced_on_the_way(m, n, k, s, nearest, Q):
    # either operand short, one part of k and several, ragged ends of every dimension, leading dimensions that are odd
    rng = np.random.default_rng(5)
    A = np.asfortranarray(rng.standard_normal((m, k)) * np.exp2(rng.integers(-20, 20, (m, 1))))
    B = np.asfortranarray(rng.standard_normal((k, n)) * np.exp2(rng.integers(-20, 20, (1, n))))
    special(A, B)
    dA, dB = ozimmu.colmajor_empty(m + 1, k)[1:, :], ozimmu.colmajor_empty(k + 3, n)[:k, :]
    dA.copy_(torch.as_tensor(A))
    dB.copy_(torch.as_tensor(B))
    ws = ozimmu.alloc_workspace(m, n, k, s)
    C = ozimmu.dgemm3(dA, dB, s, s, splitting=ozimmu.SPLIT_NEAREST if nearest else ozimmu.SPLIT_TRUNCATE,
                      level_diagonals=min(Q, ozimmu.max_level_diagonals(k, s, s)), workspace=ws, check_finite=True)
    assert ozimmu.last_gemm_kernel().startswith("gemm_vectors_kernel"), ozimmu.last_gemm_kernel()
    check(C, A, B, s, s, nearest=nearest, Q=min(Q, ozimmu.max_level_diagonals(k, s, s)))
    eA, eB = ozimmu.get_exponents(m, n, k, s, ws)
    assert eA.shape == (m,) and eB.shape == (n,)
    mx = np.abs(A).max(axis=1)
    assert np.array_equal(eA.cpu().numpy(), np.where(mx > 0, np.frexp(mx)[1], 0) + nearest)
    mx = np.abs(B).max(axis=0)
    assert np.array_equal(eB.cpu().numpy(), np.where(mx > 0, np.frexp(mx)[1], 0) + nearest)


@pytest.mark.parametrize("s", [1, 3, 5, 7, 9, 10, 14])
@pytest.mark.parametrize("m,n,offset,extra", [(70, 61, 0, 0), (300, 290, 1, 7), (301, 1025, 0, 0), (1100, 1000, 8, 0), (2048, 130, 3, 5)])
def test_stores_of_c_by_alignment(m, n, offset, extra, s):
    # columns of C on 64-byte boundaries (streaming stores) and off them, nothing written outside the m x n entries
    k = 70
    A, B = workloads.lognormal(m, n, k, 1.0, 5)
    buf = torch.full(((m + extra) * n + offset + 8,), -7.0, dtype=torch.float64, device="cuda")
    C = torch.as_strided(buf, (m, n), (1, m + extra), offset)
    ozimmu.dgemm(ozimmu.to_colmajor(A), ozimmu.to_colmajor(B), s, C=C)
    check(C, A, B, s, s)
    outside = buf.clone()
    torch.as_strided(outside, (m, n), (1, m + extra), offset).fill_(-7.0)
    assert bool((outside == -7.0).all())


@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (256, 257, 3), (300, 5, 1000), (130, 1025, 70), (4, 0, 5), (0, 3, 4), (3, 4, 0)])
def test_kappas_of_both_operands(m, n, k):
    # blocks without a nonzero entry, zeros among the others, subnormal minima; more rows than a work-group finishes
    A, B = workloads.lognormal(m, n, k, 1.5, 21)
    if m > 4 and k > 2:
        A[1, :] = 0.0
        A[2, 1] = 0.0
        A[-1, 0] = 5e-324
        B[0, -1] = -0.0
    dA, dB = ozimmu.to_colmajor(A), ozimmu.to_colmajor(B)
    s, status, kA, kB = ozimmu.estimate_slices(dA, dB, 1e-6)
    want = []
    for X, axis in ((np.abs(A), 1), (np.abs(B), 0)):
        mx, mn = X.max(axis=axis, initial=0.0), np.where(X > 0, X, np.inf).min(axis=axis, initial=np.inf)
        with np.errstate(over="ignore"):
            want.append(2.0 * max((a / b for a, b in zip(mx, mn) if a > 0), default=0.0))
    assert (kA, kB) == tuple(want)
    assert ozimmu.estimate_slices2(dA, dB, 1e-6)[3:] == (kA, kB)


@pytest.mark.parametrize("short_a", [False, True])
def test_result_inside_the_long_operand(short_a):
    # C may lie in the memory of an operand: its entries are written when the operand has been read
    m, n, k, s = (40, 3000, 6000, 3) if short_a else (3000, 40, 6000, 3)
    A, B = workloads.lognormal(m, n, k, 1.0, 33)
    dA, dB = ozimmu.to_colmajor(A), ozimmu.to_colmajor(B)
    want = ozimmu.dgemm(dA, dB, s).clone()
    assert ozimmu.last_gemm_kernel().startswith("gemm_vectors_kernel")
    C = dB[:m, :] if short_a else dA[:, :n]
    ozimmu.dgemm(dA, dB, s, C=C)
    assert not ozimmu.last_gemm_kernel().startswith("gemm_vectors_kernel")
    assert torch.equal(C, want)
    check(C, A, B, s, s)


@pytest.mark.parametrize("n,k,kernel", [(512, 90, "eighths_whole"), (576, 700, "eighths"), (672, 33, "eighths"), (704, 90, "halves")])
def test_six_slices_follow_the_same_rule_as_seven(n, k, kernel):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the expectations are worked out for 256 compute units")
    A, B = workloads.lognormal(n, n, k, 1.0, 23)
    for s in (6, 7):
        C = ozimmu.dgemm(ozimmu.to_colmajor(A), ozimmu.to_colmajor(B), s)
        assert ozimmu.last_gemm_kernel().startswith(f"gemm_{kernel + '16' * (kernel == 'halves' and s == 7)}_kernel<{s}>"), ozimmu.last_gemm_kernel()
        check(C, A, B, s, s)


@pytest.mark.parametrize("m,n,k,name", [(1440, 1440, 512, "gemm_eighths_kernel<1>"), (1440, 1440, 40960, "gemm_eighths_kernel<1>"),
                                        (1440, 1440, 40961, "gemm_fused_kernel<1> equal counts tile 128x128"),
                                        (1408, 1408, 41000, "gemm_eighths_kernel<1>"),
                                        (400, 5600, 41000, "gemm_fused_kernel<1> equal counts tile 128x128")])
def test_one_slice_over_long_contractions(m, n, k, name):
    # where the 128 x 128 tile would be the alternative, 32 x 32 tiles serve one slice up to k = 40960 only
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the expectations are worked out for 256 compute units")
    dA, dB = workloads.lognormal_device(m, n, k, 1.0, 17)
    C = ozimmu.dgemm(dA, dB, 1)
    assert ozimmu.last_gemm_kernel().startswith(name), ozimmu.last_gemm_kernel()
    rows, cols = [0, m // 2, m - 1], [0, n // 2, n - 1]
    A, B = dA[rows].cpu().numpy(), dB[:, cols].cpu().numpy()
    assert np.array_equal(bits(C.cpu().numpy()[np.ix_(rows, cols)]), bits(oracle.dgemm(np.asfortranarray(A), np.asfortranarray(B), 1)))


@pytest.mark.parametrize("m,n", [(700, 40), (40, 700)])
def test_hooks_refuse_planes_that_a_call_has_not_left(m, n):
    # the few-vectors way writes no slices of the long operand: the hooks that read both operands' say so, also when the
    # estimator has used the workspace since, until a call leaves them
    k, s = 5000, 3
    A, B = workloads.lognormal(m, n, k, 1.0, 55)
    dA, dB = ozimmu.to_colmajor(A), ozimmu.to_colmajor(B)
    ws = torch.empty(max(ozimmu.workspace_bytes(m, n, kk, s) for kk in (k, 100)), dtype=torch.uint8, device="cuda")

    def code(hook):              # (no exception is kept: its frames would keep the tensors)
        try:
            hook()
        except ozimmu.OzimmuError as error:
            return error.code
        return ozimmu.OK

    def refused():
        assert code(lambda: ozimmu.debug_diagonals(m, n, k, s, ws)) == ozimmu.BAD_ARG
        assert code(lambda: ozimmu.debug_slice_product(m, n, k, s, ws, 1, 2)) == ozimmu.BAD_ARG

    C = ozimmu.dgemm(dA, dB, s, workspace=ws)
    assert ozimmu.last_gemm_kernel().startswith("gemm_vectors_kernel")
    refused()
    ozimmu.estimate_slices(dA, dB, 1e-6, workspace=ws)
    refused()
    try:
        ozimmu.debug_small_tile_limit(0)
        assert torch.equal(ozimmu.dgemm(dA, dB, s, workspace=ws), C)
    finally:
        ozimmu.debug_small_tile_limit(-1)
    D = ozimmu.debug_diagonals(m, n, k, s, ws)
    assert torch.equal(D[1], ozimmu.debug_slice_product(m, n, k, s, ws, 1, 2) + ozimmu.debug_slice_product(m, n, k, s, ws, 2, 1))
    eA, eB = ozimmu.get_exponents(m, n, k, s, ws)
    S = sum(D[d].cpu().numpy().T * 2.0 ** (-7 * (d + 2)) for d in range(s))
    assert np.array_equal(np.ldexp(S, eA.cpu().numpy()[:, None] + eB.cpu().numpy()[None, :]), C.cpu().numpy())
    # and a call with scales and slices in one launch leaves both again after the few-vectors way
    ozimmu.dgemm(dA, dB, s, workspace=ws)
    small = ozimmu.to_colmajor(A[:, :100]), ozimmu.to_colmajor(B[:100])
    ozimmu.dgemm(*small, s, workspace=ws)
    ozimmu.debug_diagonals(m, n, 100, s, ws)


def test_estimates_from_several_threads():
    # every call has words of its own in host memory while it waits
    import threading
    cases = [workloads.lognormal(40 + 3 * i, 30 + 5 * i, 50 + 7 * i, 0.5 + i, 60 + i) for i in range(8)]
    dev = [(ozimmu.to_colmajor(A), ozimmu.to_colmajor(B)) for A, B in cases]
    want = [oracle.estimate_slices(A, B, 1e-9, s_max=ozimmu.MAX_SLICES) for A, B in cases]
    torch.cuda.synchronize()
    wrong, done = [], []

    def work(i):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            ws = ozimmu.alloc_workspace(*dev[i][0].shape[:1], dev[i][1].shape[1], dev[i][0].shape[1], 1)
            for _ in range(20):
                got = ozimmu.estimate_slices(*dev[i], 1e-9, workspace=ws)
                if got != want[i]:
                    wrong.append((i, got, want[i]))
        done.append(i)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(cases))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=60)
    assert not wrong and sorted(done) == list(range(len(cases)))      # (a thread that raised or hangs is not done)


@pytest.fixture
def host_words():
    yield
    ozimmu.debug_host_words(False)
    gc.collect()                             # (nothing of these tests is freed while another measures the allocator)


def test_estimates_without_pinned_memory(host_words):
    # no pinned words to be had: the result is copied; then they are, though the first attempt has failed
    A, B = workloads.lognormal(123, 77, 95, 1.0, 61)
    dA, dB = ozimmu.to_colmajor(A), ozimmu.to_colmajor(B)
    want = oracle.estimate_slices(A, B, 1e-9, s_max=ozimmu.MAX_SLICES)
    bad = dB.clone(memory_format=torch.preserve_format)
    bad[-1, -1] = float("inf")

    def both():
        assert ozimmu.estimate_slices(dA, dB, 1e-9) == want
        with pytest.raises(ozimmu.OzimmuError, match=f"status {ozimmu.NONFINITE} "):
            ozimmu.estimate_slices(dA, bad, 1e-9)

    assert ozimmu.debug_host_words(True) == 0
    both()
    assert ozimmu.debug_host_words(False) == 0
    both()
    assert ozimmu.debug_host_words(False) == 64


def forget_host_words():
    ozimmu.debug_host_words(True)
    assert ozimmu.debug_host_words(False) == 0


@pytest.mark.parametrize("mode", ["global", "thread_local", "relaxed"])
def test_first_estimate_while_a_stream_is_captured(host_words, mode):
    # on the default stream, which the runtime may wait for meanwhile: the words are allocated then, and the capture is good
    m, n, k, s = 123, 77, 95, 5
    A, B = workloads.lognormal(m, n, k, 1.0, 63)
    dA, dB = ozimmu.to_colmajor(A), ozimmu.to_colmajor(B)
    want = oracle.estimate_slices(A, B, 1e-9, s_max=ozimmu.MAX_SLICES)
    C, ws, other = ozimmu.colmajor_empty(m, n), ozimmu.alloc_workspace(m, n, k, s), ozimmu.alloc_workspace(m, n, k, 1)
    eager = ozimmu.dgemm(dA, dB, s, C=C, workspace=ws).clone()
    forget_host_words()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode=mode):
        ozimmu.dgemm(dA, dB, s, C=C, workspace=ws)
        with torch.cuda.stream(torch.cuda.default_stream()):
            got = [ozimmu.estimate_slices(dA, dB, 1e-9, workspace=other) for _ in range(2)]
    assert got == [want, want] and ozimmu.debug_host_words(False) == 64
    for _ in range(3):
        C.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, eager)
        assert ozimmu.estimate_slices(dA, dB, 1e-9, workspace=other) == want


def test_words_of_an_estimate_that_could_not_wait_are_not_given_to_another(host_words):
    # while a stream is captured in the global mode the runtime refuses to wait for another: the estimate's kernels run on
    import ctypes
    import re
    A, B = workloads.lognormal(64, 60, 70, 1.0, 62)
    dA, dB = ozimmu.to_colmajor(A), ozimmu.to_colmajor(B)
    want = oracle.estimate_slices(A, B, 1e-9, s_max=ozimmu.MAX_SLICES)
    forget_host_words()
    assert ozimmu.estimate_slices(dA, dB, 1e-9) == want and ozimmu.debug_host_words(False) == 64
    hip = ctypes.CDLL(re.search(r"\S*libamdhip64\.so\S*", open("/proc/self/maps").read())[0])
    captured, other, ws = torch.cuda.Stream(), torch.cuda.Stream(), ozimmu.alloc_workspace(64, 60, 70, 1)
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(ctypes.c_void_p(captured.cuda_stream), 0) == 0
    try:
        with torch.cuda.stream(other), pytest.raises(ozimmu.OzimmuError, match=f"status {ozimmu.HIP_ERROR} "):
            ozimmu.estimate_slices(dA, dB, 1e-9, workspace=ws)
    finally:
        graph = ctypes.c_void_p()
        hip.hipStreamEndCapture(ctypes.c_void_p(captured.cuda_stream), ctypes.byref(graph))      # (spoilt by the refused wait)
        hip.hipGetLastError()
    torch.cuda.synchronize()
    assert ozimmu.debug_host_words(False) == 63
    assert ozimmu.estimate_slices(dA, dB, 1e-9) == want and ozimmu.debug_host_words(False) == 63
