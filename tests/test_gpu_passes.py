"""Slices streamed through a ring of LDS slots (unsteered), bit for bit: 4 ... 9 slices in one pass, 10 ... 20 with the diagonals in
passes; a sample of rows and columns against the oracle,
every entry against the one-pass kernels that the test knob puts in their place."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle
from paper_2506_11277_amd import ozimmu, workloads
from tests.test_gpu_routes import bits, check, special


def steered(f):
    try:
        ozimmu.debug_small_tile_limit(256)
        return f()
    finally:
        ozimmu.debug_small_tile_limit(-1)


def both_ways(A, B, sA, sB, name, **kw):
    dA, dB = ozimmu.to_colmajor(A), ozimmu.to_colmajor(B)
    run = lambda: ozimmu.dgemm3(dA, dB, sA, sB, **kw)
    C = run()
    if name and torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert ozimmu.last_gemm_kernel().startswith(name), ozimmu.last_gemm_kernel()
    want = steered(run)
    assert "passes" not in ozimmu.last_gemm_kernel()
    assert torch.equal(C.view(torch.int64), want.view(torch.int64))
    check(C, A, B, sA, sB, nearest=kw.get("splitting") == ozimmu.SPLIT_NEAREST, Q=kw.get("level_diagonals", 1))


# 64 x 64 tiles, two work-groups to a compute unit: four 64-deep k-steps (what the shortest such contraction is padded to) and many, edges of
# tiles, a last round of few
@pytest.mark.parametrize("s", range(4, 10))
@pytest.mark.parametrize("m,n,k,least", [(1500, 1530, 130, 4), (3000, 2900, 195, 6), (2311, 2003, 1281, 5), (61, 37000, 300, 4), (1409, 2726, 1281, 4)])
def test_one_pass(m, n, k, least, s):
    A, B = workloads.lognormal(m, n, k, 1.0, 50 + s)
    special(A, B)
    both_ways(A, B, s, s, f"gemm_passes_kernel<{s}> tile 64x64" if s >= least else "")
    both_ways(A, B, s, s - 1, "", splitting=ozimmu.SPLIT_NEAREST, level_diagonals=2)


# 128 x 64 tiles, several to a work-group: a second tile for some of them, several for all, four k-steps and more, a grid in the
# two-dimensional order with ten blocks that have no tile (5994 x 631)
@pytest.mark.parametrize("s", range(4, 10))
@pytest.mark.parametrize("m,n,k", [(5994, 631, 500), (3292, 960, 500), (8777, 1360, 250)])
def test_one_pass_in_runs(m, n, k, s):
    A, B = workloads.lognormal(m, n, k, 1.0, 30 + s)
    special(A, B)
    both_ways(A, B, s, s, f"gemm_passes_kernel<{s}> tile 128x64")


# 96 x 64 tiles: one round and several (7 ... 9), a last tile that reaches beyond the planes (1650 rows, padded to 1664), contractions of a single k-block and more, both ends of
# what one round holds and 13/16 of it
ALL_96 = [*range(4, 10), *range(13, 19)]
TILES_OF_96 = [((1531, 777, 1001), ALL_96), ((1531, 841, 300), ALL_96), ((1650, 700, 450), ALL_96), ((1650, 2670, 700), range(7, 10)), ((2304, 2000, 600), range(7, 10)),
               ((1000, 1190, 257), ALL_96), ((4030, 340, 260), ALL_96), ((90, 16380, 131), ALL_96), ((1025, 1153, 1030), ALL_96), ((1030, 1400, 65), ALL_96),
               ((1001, 1250, 1), ALL_96), ((1040, 1450, 128), ALL_96)]


@pytest.mark.parametrize("m,n,k,s", [(*size, s) for size, counts in TILES_OF_96 for s in counts])
def test_tiles_of_96_rows(m, n, k, s):
    A, B = workloads.lognormal(m, n, k, 1.0, 40 + s)
    special(A, B)
    both_ways(A, B, s, s, f"gemm_passes_kernel<{s}> tile 96x64")
    both_ways(A, B, s - 1, s, "", splitting=ozimmu.SPLIT_NEAREST, level_diagonals=2 if s < 10 else 3)


def test_planes_too_large_for_the_offsets_of_a_run():
    # the planes of A take 4.3 GB: beyond 32-bit offsets, so a work-group takes one tile
    m, n, k, s = 340000, 130, 1400, 9
    dA, dB = workloads.lognormal_device(m, n, k, 1.0, 44)
    assert ozimmu.workspace_bytes(m, n, k, s) > 1 << 32
    C = ozimmu.dgemm(dA, dB, s)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert ozimmu.last_gemm_kernel().startswith(f"gemm_passes_kernel<{s}> tile 128x64"), ozimmu.last_gemm_kernel()
    assert torch.equal(C, steered(lambda: ozimmu.dgemm(dA, dB, s)))
    rows, cols = [0, 127, 128, m // 2, 336000, m - 33, m - 1], [0, 63, 64, n - 1]
    want = oracle.dgemm(np.asfortranarray(dA[rows].cpu().numpy()), np.asfortranarray(dB[:, cols].cpu().numpy()), s)
    assert np.array_equal(bits(C[rows][:, cols].cpu().numpy()), bits(want))


# Shapes where tiles in pairs or runs, or passes, are behind: one XCD with a tile more than it has places for, a round and a bit with few
# slices, whole rounds with 10 and 11, a single round of short contractions
@pytest.mark.parametrize("m,n,k,s,name", [
    (3200, 613, 1152, 9, "tile 128x64"), (731, 3573, 3538, 5, "gemm_fused16_kernel<5> tile 128x128"),
    (5120, 512, 5208, 6, "gemm_fused16_kernel<6> tile 128x128"), (1664, 1664, 1664, 4, "gemm_fused16_kernel<4> tile 128x128"),
    (384, 5760, 3648, 6, "gemm_fused16_kernel<6> tile 128x128"),
    (1280, 1280, 1280, 10, "gemm_fused_kernel<10>"), (4005, 960, 257, 10, "gemm_fused_kernel<10>"), (384, 3066, 2801, 10, "gemm_fused_kernel<10>"),
    (604, 1811, 5512, 11, "gemm_fused_kernel<11>"), (1090, 1090, 1090, 11, "gemm_fused_kernel<11>"),
    (896, 832, 113, 19, "gemm_fused_kernel<19>"), (908, 717, 103, 17, "gemm_fused_kernel<17>")])
def test_where_the_larger_tiles_stay(m, n, k, s, name):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the expectations are worked out for 256 compute units")
    dA, dB = workloads.lognormal_device(m, n, k, 1.0, 18)
    C = ozimmu.dgemm(dA, dB, s)
    assert name in ozimmu.last_gemm_kernel(), ozimmu.last_gemm_kernel()
    assert torch.equal(C, steered(lambda: ozimmu.dgemm(dA, dB, s)))


@pytest.mark.parametrize("choice,name", [(1, "gemm_fused16_kernel<5> tile 128x128"), (2, "gemm_fused16_kernel<5> tile 128x64"),
                                         (0, "gemm_passes_kernel<5>")])
def test_a_forced_tile_is_the_one_that_runs(choice, name):
    dA, dB = workloads.lognormal_device(3500, 3500, 300, 1.0, 19)
    try:
        ozimmu.debug_tile_choice(choice)
        ozimmu.dgemm(dA, dB, 5)
    finally:
        ozimmu.debug_tile_choice(0)
    if choice or torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert ozimmu.last_gemm_kernel().startswith(name), ozimmu.last_gemm_kernel()


# 128 x 64 tiles: one partly filled round, ragged edges; 64 x 64 tiles: a second work-group on some compute units, edges; two
# 64-deep k-steps (k = 40 and 65) and many
@pytest.mark.parametrize("s", range(10, 21))
@pytest.mark.parametrize("m,n,k,tile,least", [(1793, 1009, 1030, "128x64", 13), (2050, 2020, 1100, "64x64", 10), (1030, 1700, 65, "64x64", 13),
                                              (2300, 4600, 40, "64x64", 13), (80, 20000, 400, "64x64", 10)])
def test_passes_through_lds(m, n, k, tile, least, s):
    A, B = workloads.lognormal(m, n, k, 1.0, 70 + s)
    special(A, B)
    name = f"gemm_passes_kernel<{s}> tile {tile}" if s >= least else ""
    both_ways(A, B, s, s, name)
    both_ways(A, B, s, s, name, splitting=ozimmu.SPLIT_NEAREST, level_diagonals=3)


# 11 and 12 slices take 128 x 64 tiles where the launch is long
@pytest.mark.parametrize("s", [11, 12])
def test_long_launches_of_few_passes(s):
    m, n, k = 1030, 1000, 11000
    A, B = workloads.lognormal(m, n, k, 1.0, 60 + s)
    special(A, B)
    both_ways(A, B, s, s, f"gemm_passes_kernel<{s}> tile 128x64")


# 32 x 32 tiles, k in eighths: fewer k-blocks than wavefronts, one more than a round of them, edges of tiles, the ends of the rule; any
# level size
@pytest.mark.parametrize("s", range(11, 21))
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (33, 31, 130), (161, 1300, 70), (97, 70, 289), (512, 512, 64), (512, 896, 560), (40, 1000, 1100), (31, 65, 6657)])
def test_passes_of_a_divided_contraction(m, n, k, s):
    A, B = workloads.lognormal(m, n, k, 1.0, 90 + s)
    if m > 4:
        special(A, B)
    name = f"gemm_eighths_passes_kernel<{s}>"
    both_ways(A, B, s, s, name)
    for Q in (2, 3):
        both_ways(A, B, s, s, name, splitting=ozimmu.SPLIT_NEAREST, level_diagonals=Q)


# levels that would straddle two passes take the one-pass kernels, levels that end with a pass do not; counts that differ little run
# as equal ones
@pytest.mark.parametrize("sA,sB,Q,passes", [(13, 13, 4, False), (16, 16, 2, False), (13, 13, 2, True), (12, 13, 1, True), (18, 17, 3, True), (20, 19, 1, True),
                                            (10, 14, 1, True)])
def test_levels_and_different_counts(sA, sB, Q, passes):
    A, B = workloads.lognormal(1100, 1090, 300, 1.0, 5)
    both_ways(A, B, sA, sB, f"gemm_passes_kernel<{max(sA, sB)}>" if passes else "gemm_fused_kernel", level_diagonals=Q)


def test_leading_dimensions_and_odd_alignment():
    m, n, k, s = 1101, 1091, 1100, 14
    A, B = workloads.lognormal(m, n, k, 1.0, 9)
    dA, dB = ozimmu.to_colmajor(A), ozimmu.to_colmajor(B)
    big = ozimmu.colmajor_empty(m + 5, n + 2).fill_(7.0)
    C = big[3:m + 3, 1:n + 1]
    ozimmu.dgemm(dA, dB, s, C=C)
    assert "passes" in ozimmu.last_gemm_kernel()
    assert torch.equal(C, steered(lambda: ozimmu.dgemm(dA, dB, s)))
    assert (big[:3] == 7).all() and (big[m + 3:] == 7).all() and (big[:, 0] == 7).all() and (big[:, -1] == 7).all()
