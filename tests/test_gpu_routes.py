"""The routes the library takes by itself at sizes that do not fill the chip, against the oracle, bit for bit.

(The other parity tests steer the choice of kernel; nothing is steered here.)  Every row of A and column of B has a
scale of its own, so a sample of rows and columns of C is the oracle's product of these rows and columns."""
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
    (1, 1, 1, "32x32"), (33, 31, 130, "32x32"), (512, 512, 64, "32x32"), (97, 70, 1000, "32x32"), (40, 300, 2100, "32x32"),
    (705, 961, 65, "64x64, 8"), (1024, 1000, 129, "64x64, 8"), (65, 8000, 700, "64x64, 8"),
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
        assert kernel in ozimmu.last_gemm_kernel(), ozimmu.last_gemm_kernel()
    check(C, A, B, s, s)
    check(ozimmu.dgemm3(dA, dB, s, s, splitting=ozimmu.SPLIT_NEAREST, level_diagonals=2), A, B, s, s, nearest=True, Q=2)
