"""Which pass and variant a product takes: the library's rule, asked on the host."""
import ctypes
import itertools
import random

import pytest

import test_gpu_block_pass

ROUND_WORDS = {1: 256, 2: 192}


@pytest.fixture(scope="module")
def plan():
    import os

    import paper_2309_10285_amd as fls
    from paper_2309_10285_amd import _build

    if not os.path.exists(fls.LIB_PATH):
        _build.build()

    def ask(rounds, version, M, K, N, cus=256, entry="fls_spmm"):
        p = fls.spmm_plan({"max_tile_words": rounds * ROUND_WORDS[version], "format_version": version, "M": M, "K": K}, N, cus, entry)
        return p["pass"], p["share"], p["rounds"], p["slices"]

    return ask


def test_the_block_pass_cases_reach_every_variant(plan):
    """The cases of the GPU test, asked with the rounds that tiles of their sparsity need, and all variants among them."""
    need = {0.9: 2, 0.85: 3, 0.8: 4, 0.7: 6, 0.6: 7, 0.55: 8, 0.5: 9}
    seen = set()
    for M, K, N, sparsity, version, want in test_gpu_block_pass.ROWS:
        p = plan(need[sparsity], version, M, K, N)
        assert (*p[:3], p[3] > 1) == want, (M, K, N)
        if p[0] == "block":
            seen.add((p[1], p[2], version))
    assert seen == {(share, r, v) for v in (1, 2) for share, rounds in ((1, (2, 3, 4, 6)), (2, (2, 4, 6, 8, 10))) for r in rounds}


@pytest.mark.parametrize("version", [1, 2])
def test_columns_and_density_decide(plan, version):
    M, K = 12288, 8192  # bands of 256 K tiles: too short for the 64-column pass at up to 32 columns
    for N in (1, 16, 17, 32):
        assert plan(4, version, M, K, N)[0] == "narrow"
    for N in (33, 64):
        assert plan(4, version, M, K, N)[0] == "wide"
    assert plan(4, version, M, K, 4096)[0] == "block"
    for N in (33, 64, 65, 4096):  # denser tiles than any of the wider passes stages
        assert plan(11, version, M, K, N) == ("narrow", 0, 8, 0)
    long_band = (2, version, 12288, 49152)
    assert plan(*long_band, 32)[0] == "wide" and plan(*long_band, 16)[0] == "narrow"
    assert plan(*long_band, 32, entry="fls_spmm_noalloc")[0] == "narrow"
    for rounds, staged in ((1, 2), (2, 2), (3, 3), (4, 4), (5, 6), (6, 6), (7, 8), (8, 8), (9, 10), (10, 10)):
        assert plan(rounds, version, M, K, 64)[2] == staged


@pytest.mark.parametrize("N", [17, 24, 32])
def test_short_bands_stay_with_the_kernel_that_checks_offsets(plan, N):
    """The 64-column pass trusts TileOffsets: up to 32 columns it takes calls on long bands only, whatever tiles need and the estimate says."""
    rng = random.Random(11)
    for version, rounds in itertools.product((1, 2), range(1, 11)):
        for _ in range(60):
            kt, bands = int((1024 if version == 2 else 288) ** rng.random()), int(400 ** rng.random())
            assert plan(rounds, version, bands * 128, kt * 32, N)[0] == "narrow", (version, rounds, bands, kt)
    for rounds in range(5, 11):  # the pass has no variant with one column block for them in version 2
        assert plan(rounds, 2, 12288, 49152, N)[0] == "narrow"
    # bands of 288 - 383 K tiles: sparse tiles, and K slices that do not come out even
    assert plan(2, 1, 8192, 352 * 32, N)[0] == "narrow" and plan(1, 1, 27648, 9216, N)[0] == "narrow"
    assert plan(9, 1, 128, 300 * 32, N)[0] == "narrow"
    assert plan(9, 1, 1024, 384 * 32, N)[0] == "wide"  # tiles of more than eight rounds, on a long band


@pytest.mark.parametrize("rounds,version,M,K,N,share", [
    # K tiles that fill no body of the 64-column pass (us there / in the block pass with share 1 / 2)
    (4, 1, 12288, 480, 4096, 2),    # 139 / 70 / 67
    (7, 1, 12288, 224, 4096, 2),    # 100 / - / 57
    (4, 1, 46720, 672, 149, 2),     # 48 / 28 / 25
    (5, 1, 39808, 192, 266, 1),     # 26 / 19 / 27
    # so little work that the start of a block pass costs more than it saves
    (2, 1, 12288, 32, 4096, 0),     # 30 / 38 / 38
    (4, 1, 4096, 160, 1000, 0),     # 12.6 / 15.9 / 14.9
    (7, 1, 2176, 384, 1768, 0),     # 17.0 / - / 19.6
    (7, 2, 1280, 1056, 1475, 0),    # 28.9 / - / 32.8
    # sparse tiles, which cost the 64-column pass least
    (2, 1, 12288, 12288, 512, 0),   # 133 / 145 / 140
    (2, 1, 12288, 12288, 2048, 0),  # 437 / 530 / 498
    (2, 1, 9216, 9216, 4096, 0),    # 537 / 607 / 582
    (2, 1, 12288, 12288, 1024, 2),  # 272 / 249 / 242
    # level: the pass with fewer partial sums
    (4, 1, 12288, 12288, 128, 0),   # 57.9 / 60.5 / 70.8
])
def test_the_rule_takes_the_pass_that_measured_faster(plan, rounds, version, M, K, N, share):
    assert plan(rounds, version, M, K, N)[1] == share


@pytest.mark.parametrize("rounds,version,M,K,N,slices", [
    # us, slices of two bodies and more / of one
    (6, 1, 2560, 288, 564, 1),    # 12.1 / 17.7: one slice has no second kernel and no sums
    (6, 1, 4608, 416, 260, 1),    # 14.5 / 18.6
    (6, 2, 4096, 288, 244, 1),    # 12.4 / 15.1
    (3, 1, 3584, 608, 378, 1),    # 14.9 / 17.8
    (4, 1, 2176, 512, 341, 1),    # 13.5 / 15.8
    (6, 2, 4096, 1536, 50, 6),    # 15.6 / 17.6 with twelve
    (3, 1, 2176, 1056, 360, 2),   # 17.4 / 19.0 with three
    (6, 2, 2944, 1088, 58, 8),    # 16.3 with four / 14.2
    (4, 1, 1024, 1024, 64, 4),    # 15.0 with two / 11.5
    (2, 2, 2048, 2880, 54, 11),   # 17.6 with five / 13.7
])
def test_slices_of_one_body_where_they_measured_faster(plan, rounds, version, M, K, N, slices):
    assert plan(rounds, version, M, K, N)[3] == slices


@pytest.mark.parametrize("M,K,N,groups,slices", [
    # us, slices of 16 steps and more / of two
    (7424, 224, 356, 6, 1),     # 16.8 / 30.7: one slice has no second kernel and no sums
    (15744, 352, 240, 4, 1),    # 20.9 / 36.7
    (28928, 384, 78, 2, 1),     # 25.1 / 34.3
    (9088, 352, 202, 4, 1),     # 21.9 / 33.4
    (1408, 1120, 182, 3, 9),    # 37.9 / 18.0
    (5120, 1120, 51, 1, 9),     # 71.2 / 22.8
    (1280, 1888, 97, 2, 15),    # 90.0 / 18.3
    (128, 30848, 52, 1, 128),   # 27.9 with 256
    (30848, 5248, 143, 2, 2),   # with a pass of its own for the rest 217, without 246
])
def test_dense_slices_where_they_measured_faster(plan, M, K, N, groups, slices):
    import paper_2309_10285_amd as fls

    out = (ctypes.c_uint32 * 2)()
    fls.lib().fls_internal_dense_plan(M, K, N, 256, out)
    assert tuple(out) == (groups, slices)


def _shapes(count):
    rng = random.Random(7)
    for _ in range(count):
        M, K = int(128 * 500 ** rng.random()) // 128 * 128, int(32 * 2000 ** rng.random()) // 32 * 32
        N = min(int(33 * 248 ** rng.random()), (2**30 - 1) // max(M, K))
        if N > 32 and M * K < 2**32:
            yield M, K, N


@pytest.mark.parametrize("cus", [8, 64, 256, 304])
def test_partial_sums_fit_their_area(plan, cus):
    """A sliced product leaves slices x bands x groups of 64 columns partial results of 32 KB; the area holds 2048."""
    for (M, K, N), rounds, version in itertools.product(_shapes(400), (2, 4, 6, 10), (1, 2)):
        kind, share, staged, slices = plan(rounds, version, M, K, N, cus)
        assert slices >= 1 and staged >= rounds
        if slices > 1:
            groups = -(-N // 64)
            units = -(-M // 512) * groups if kind == "wide" else -(-M * share // 512) * -(-N // (128 * share))
            assert units * slices <= min(cus, 512) and M // 128 * groups * slices <= 2048


@pytest.mark.parametrize("cus", [8, 64, 256, 304])
def test_what_the_wider_passes_divide_is_small_enough(plan, cus):
    """Unit numbers and slice x K tiles: the kernels' division by multiplication is exact below 2^29."""
    largest = [(128, 2**23, 64), (2**23, 480, 64), (128 * 512, 2**15, 8192), (2**25, 96, 31), (2**17 - 128, 2**14, 8191)]
    for M, K, N in [*_shapes(200), *largest]:
        assert M * K < 2**32 and max(M, K) * N < 2**30  # what a call may have
        bands, groups, kt = M // 128, -(-N // 64), K // 32
        for rounds, version in itertools.product((2, 6, 10), (1, 2)):
            kind, share, _, slices = plan(rounds, version, M, K, N, cus)
            if kind != "narrow":
                units = (-(-bands * share // 4) * -(-N // (128 * share)) if kind == "block" else -(-bands // 4) * groups) * slices
                assert units + 8 * groups < 2**29 and (slices + 1) * kt < 2**29, (M, K, N)
        # the dense product: units of four bands and 64 columns, as many slices as fill the CUs
        assert max(-(-bands // 4) * groups, cus) + 8 * groups < 2**29 and (cus + 1) * kt < 2**29
