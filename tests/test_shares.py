"""How the passes of up to 32 columns share tiles out to workgroups: the library's rule, asked on the host."""
import ctypes
import random

import pytest


@pytest.fixture(scope="module")
def shares():
    import os

    import paper_2309_10285_amd as fls
    from paper_2309_10285_amd import _build

    if not os.path.exists(fls.LIB_PATH):
        _build.build()
    f = fls.lib().fls_internal_shares
    f.argtypes = [ctypes.c_uint32, ctypes.c_uint32, ctypes.c_int, ctypes.c_float, ctypes.c_int, ctypes.POINTER(ctypes.c_uint32)]
    f.restype = None

    def ask(bands, kt, cus=256, tile_us=0.105, wide=False):
        out = (ctypes.c_uint32 * 3)()
        f(bands * 128, kt * 32, cus, tile_us, int(wide), out)
        return tuple(out)

    return ask


def _begin(P, unit, bands, kt, q):
    return q * bands // P * kt if unit == 0 else q * bands * kt // P


def _share(P, unit, block):
    """The share of a workgroup id, None for an idle one."""
    if unit == 0:
        return block if block < P else None
    x, units = block % 8, P // unit
    q = x * units // 8 * unit + block // 8
    return q if q < (x + 1) * units // 8 * unit else None


def _shapes(count):
    rng = random.Random(5)
    for _ in range(count):
        bands, kt = int(400 ** rng.random()), int(2000 ** rng.random())
        yield bands, kt, rng.choice([0.07, 0.105, 0.14, 0.27]), rng.random() < 0.5
    yield from ((2**20 - 1, 1, 0.105, False), (1, 2**18, 0.105, False), (1, 2**18, 0.27, True), (2**10, 2**10 - 1, 0.07, False))


@pytest.mark.parametrize("cus", [1, 8, 20, 64, 256, 304])
def test_every_share_runs_once_and_holds_tiles(shares, cus):
    for bands, kt, tile_us, wide in _shapes(1500):
        P, unit, grid = shares(bands, kt, cus, tile_us, wide)
        assert 1 <= P <= cus and (unit == 0 or P % unit == 0)
        assert P * bands * kt < 2**29  # the kernels' division by multiplication is exact below
        assert sorted(q for q in (_share(P, unit, b) for b in range(grid)) if q is not None) == list(range(P))
        begins = [_begin(P, unit, bands, kt, q) for q in range(P + 1)]
        assert begins[0] == 0 and begins[-1] == bands * kt and all(a < b for a, b in zip(begins, begins[1:]))
        if unit == 0:
            assert all(b % kt == 0 for b in begins)
        elif unit > 1:  # the shares of a band, or of a pair of bands, on one XCD, and at most one workgroup to a CU there
            assert begins[unit] in (kt, 2 * kt) and -(-P // unit // 8) * unit <= max(1, cus // 8)


@pytest.mark.parametrize("cus", [8, 64, 256])
def test_shares_begin_where_the_kernels_division_says(shares, cus):
    """share_begin of the kernels, with the library's own division: no tile is left out or done twice."""
    import paper_2309_10285_amd as fls

    div = fls.lib().fls_internal_divide
    div.argtypes, div.restype = [ctypes.c_uint32] * 2, ctypes.c_uint32
    for bands, kt, tile_us, wide in _shapes(150):
        P, unit, _ = shares(bands, kt, cus, tile_us, wide)
        for q in range(P + 1):
            assert (div(q * bands, P) * kt if unit == 0 else div(q * bands * kt, P)) == _begin(P, unit, bands, kt, q), (bands, kt, q)


@pytest.mark.parametrize("bands,kt,tile_us,wide,want", [
    # us, N = 8 (wide: 32), measured with forced cuts
    (8, 16, 0.105, False, [8]),     # whole 5.6, in 2 shares 6.7
    (8, 32, 0.105, False, [32]),    # whole 7.3, in 2 / 4 shares 7.8 / 6.7
    (8, 64, 0.105, False, [40, 64]),  # whole 10.9, in 4 / 5 / 8 / 10 7.8 / 7.6 / 7.4 / 9.0
    (8, 32, 0.07, False, [8]),      # 90 %: whole 6.1, in 4 6.4
    (8, 512, 0.105, False, range(128, 193)),  # in 12 / 16 / 24 12.2 / 11.5 / 11.7
    (8, 64, 0.125, True, [40]),     # whole 12.8, in 4 / 5 / 8 9.6 / 9.3 / 9.6
    (138, 92, 0.27, False, [256]),  # dense: whole 36.9, cut evenly 26.7
    (191, 63, 0.27, False, [256]),  # 35.6 / 32.4
    (92, 154, 0.27, False, [256]),  # in 2 shares 34.2, cut evenly 29.3
    (25, 474, 0.27, True, [250]),   # in 10 shares 33.7, cut evenly 34.6
    (150, 61, 0.125, True, [150]),  # 90 %: 14.6 / 16.1
    (130, 110, 0.16, True, [256]),  # 21.2 / 18.9
    (384, 8, 0.105, False, [192]),  # two bands to a workgroup 7.3, cut over 256 9.7
    (384, 384, 0.105, False, [256]),
    (224, 224, 0.105, False, [224]),
    (96, 384, 0.105, False, [256]),
    (168, 224, 0.105, False, [252]),
])
def test_the_rule_takes_what_measured_fastest(shares, bands, kt, tile_us, wide, want):
    assert shares(bands, kt, 256, tile_us, wide)[0] in want


def test_division_by_multiplication(shares):
    """Exact below 2^29 for every divisor a launch can have (shares up to 512, K tiles up to 2^18)."""
    import paper_2309_10285_amd as fls

    f = fls.lib().fls_internal_divide
    f.argtypes, f.restype = [ctypes.c_uint32] * 2, ctypes.c_uint32
    rng = random.Random(6)
    for d in [*range(1, 600), *(rng.randrange(600, 2**18 + 1) for _ in range(400)), 2**18, 2**18 - 1]:
        for q in (0, 1, 2**29 // d - 1, *(rng.randrange(2**29 // d) for _ in range(8))):
            for n in (q * d - 1, q * d, q * d + d - 1):
                if 0 <= n < 2**29:
                    assert f(n, d) == n // d, (n, d)


@pytest.mark.parametrize("rounds,version,M,K,N,want", [
    # us, passes of up to 32 columns / 64-column pass
    (4, 1, 1024, 1024, 64, "wide"),       # 16.3 / 15.0
    (4, 1, 32768, 1024, 64, "narrow"),    # 18.3 / 26.5
    (4, 1, 12288, 12288, 64, "wide"),     # 63.7 / 43.8
    (2, 1, 8192, 8192, 33, "narrow"),     # 25.1 / 31.2
    (2, 1, 8832, 48736, 31, "wide"),      # 62.6 / 51.9
    (2, 1, 6272, 13440, 27, "narrow"),    # 16.6 / 25.4
    (4, 1, 16128, 10400, 19, "narrow"),   # 29.6 / 43.5
    (6, 1, 27648, 9216, 32, "wide"),      # 62.5 / 58.4
    (6, 2, 12288, 49152, 32, "narrow"),   # version 2 has variants with one column block for up to four rounds
    (9, 1, 32768, 1024, 64, "wide"),      # the narrow kernel stages eight rounds
    (3, 1, 41216, 160, 35, "wide"),       # 13.2 / 8.7: one slice, no body
    (3, 2, 29952, 192, 50, "wide"),       # 14.8 / 10.3
    (4, 2, 128, 128, 54, "wide"),         # 12.0 / 8.4
    (3, 2, 384, 224, 57, "wide"),         # 14.0 / 9.7: bands of fewer than eight tiles
    (3, 1, 34944, 448, 62, "wide"),       # 19.1 / 15.4: one slice
    (3, 2, 45056, 480, 53, "wide"),       # 19.1 / 16.2
    (8, 1, 26368, 512, 41, "narrow"),     # 14.6 / 20.5
])
def test_the_rule_for_17_to_64_columns(shares, rounds, version, M, K, N, want):
    import paper_2309_10285_amd as fls

    stats = {"max_tile_words": rounds * (256 if version == 1 else 192) - 12, "format_version": version, "M": M, "K": K}
    assert fls.spmm_plan(stats, N)["pass"] == want
    assert fls.spmm_plan(stats, min(N, 32), entry="fls_spmm_noalloc")["pass"] == "narrow"
