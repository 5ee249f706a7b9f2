"""The block pass of fls_spmm (calls of more than 64 columns): every variant of it, at the edges of its tiles, bodies and slices.
Each case says which variant it is there for, and the library's own rule is asked whether it runs that one.  C against the
product in 64 bits of the same fp16 operands.

Tolerance: products of fp16 values are exact in fp32; a sum of K <= 11200 of them in fp32 is off by at most K * 2^-24 of the
sum of their magnitudes (about 7e-4 of it, and far less in effect), fp16 rounding adds 2^-11 of the value: 2e-3 of the
largest value covers both, as in the other parity tests.
"""
import numpy as np
import pytest

import fls_workloads as wl

pytestmark = pytest.mark.gpu

TOL = 2e-3


@pytest.fixture(scope="module")
def fls():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2309_10285_amd as f

    f.lib()
    return f


def _call(fls, blob, X, M, K, N):
    import torch

    C = torch.full((N, M), float("nan"), dtype=torch.float16, device="cuda")
    fls.ensure_workspace(M, K, N)
    fls.fls_spmm(blob, torch.from_numpy(X.view(np.float16)).cuda(), C, M, K, N)
    torch.cuda.synchronize()
    return C.cpu().numpy().astype(np.float64)


def _f64(bits):
    return bits.view(np.float16).astype(np.float64)


def _compress(fls, W, version):
    import torch

    Wd = torch.from_numpy(W.view(np.float16)).cuda()
    return (fls.fls_compress_v2 if version == 2 else fls.fls_compress)(Wd)


def _plan(fls, stats, N):
    import torch

    p = fls.spmm_plan(stats, N, torch.cuda.get_device_properties(0).multi_processor_count)
    return (p["pass"], p["share"], p["rounds"], p["slices"] > 1)


# M, K, N, sparsity, version, and the pass with its share, the rounds of a tile that the variant stages and whether K is sliced
ROWS = [
    # 128 columns x four bands, an incomplete group of bands, K tiles that are no multiple of three, a ragged last column group
    (35968, 160, 257, 0.9, 1, ("block", 1, 2, False)),
    (33664, 160, 271, 0.9, 2, ("block", 1, 2, False)),
    (5376, 800, 1477, 0.85, 1, ("block", 1, 3, False)),
    (5376, 800, 1533, 0.85, 2, ("block", 1, 3, False)),
    (22912, 544, 513, 0.8, 1, ("block", 1, 4, False)),
    (22912, 544, 513, 0.8, 2, ("block", 1, 4, False)),
    (22912, 416, 513, 0.7, 1, ("block", 1, 6, False)),
    (22912, 416, 513, 0.7, 2, ("block", 1, 6, False)),
    # ... K slices of unequal length
    (5504, 8672, 277, 0.8, 1, ("block", 1, 4, True)),
    (12160, 3680, 331, 0.8, 2, ("block", 1, 4, True)),
    # 256 columns x two bands: one band on its own in dozens of K slices; few K tiles
    (128, 11200, 137, 0.9, 1, ("block", 2, 2, True)),
    (21632, 160, 732, 0.9, 2, ("block", 2, 2, False)),
    # ... an odd number of bands, a last column group with one column, or half empty
    (16768, 544, 449, 0.8, 1, ("block", 2, 4, False)),
    (640, 3040, 897, 0.8, 2, ("block", 2, 4, True)),
    (640, 3040, 385, 0.7, 1, ("block", 2, 6, True)),
    (896, 3040, 641, 0.7, 2, ("block", 2, 6, True)),
    (8064, 608, 129, 0.6, 1, ("block", 2, 8, False)),
    (1664, 1696, 513, 0.55, 1, ("block", 2, 8, True)),
    (640, 3040, 384, 0.6, 2, ("block", 2, 8, True)),
    (5760, 736, 257, 0.5, 1, ("block", 2, 10, False)),
    (1664, 3040, 129, 0.5, 2, ("block", 2, 10, True)),
    # shapes like these that the rule gives to the 64-column pass, whose K tiles fill no whole number of bodies
    (3968, 544, 257, 0.7, 1, ("wide", 0, 6, True)),
    (3968, 544, 512, 0.7, 2, ("wide", 0, 6, True)),
    (3968, 544, 512, 0.9, 1, ("wide", 0, 2, False)),
    (15232, 544, 125, 0.7, 1, ("wide", 0, 6, True)),
    (15232, 544, 125, 0.8, 2, ("wide", 0, 4, False)),
    (7296, 1696, 125, 0.7, 1, ("wide", 0, 6, True)),
]


@pytest.mark.parametrize("M,K,N,sparsity,version,plan", ROWS)
def test_edges(fls, M, K, N, sparsity, version, plan):
    W = wl.prune_uniform(wl.gen_weights_f32(M, K, 71), sparsity, 72)
    X = wl.gen_x(N, K, 73)
    ref = _f64(X) @ _f64(W).T
    blob, stats = _compress(fls, W, version)
    assert _plan(fls, stats, N) == plan
    C = _call(fls, blob, X, M, K, N)
    assert np.abs(C - ref).max() / np.abs(ref).max() <= TOL


@pytest.mark.parametrize("M,K,N,sparsity,version,plan", [r for r in ROWS if r[:3] in (
    (22912, 416, 513), (5504, 8672, 277), (8064, 608, 129), (640, 3040, 384), (640, 3040, 385), (1664, 3040, 129))])
def test_denser_blob_behind_the_librarys_back(fls, M, K, N, sparsity, version, plan):
    """The variant is picked for the sparse blob that the library remembers; the denser one that stands there by the
    time of the call does not fit its stages and takes the block pass's plain loop."""
    import torch

    W32 = wl.gen_weights_f32(M, K, 81)
    X = wl.gen_x(N, K, 82)
    W = wl.prune_uniform(W32, 0.3, 83)
    (sparse, stats), (dense, dense_stats) = _compress(fls, wl.prune_uniform(W32, sparsity, 83), version), _compress(fls, W, version)
    assert _plan(fls, stats, N) == plan and dense_stats["max_tile_words"] > plan[2] * (192 if version == 2 else 256)
    ref = _f64(X) @ _f64(W).T
    place = torch.zeros(dense.numel(), dtype=torch.uint8, device="cuda")
    place[:sparse.numel()].copy_(sparse)
    _call(fls, place, X, M, K, N)
    place.copy_(dense)
    C = _call(fls, place, X, M, K, N)
    fls.fls_forget(place)
    assert np.abs(C - ref).max() / np.abs(ref).max() <= TOL


@pytest.mark.parametrize("M,K,N,sparsity,plan", [
    (3968, 544, 300, 0.7, ("wide", 0, 6, True)),
    (8064, 608, 300, 0.7, ("block", 2, 6, False)),
    (896, 3040, 641, 0.7, ("block", 2, 6, True)),
    (22912, 416, 513, 0.7, ("block", 1, 6, False)),
    (5504, 8672, 277, 0.82, ("block", 1, 4, True)),
])
def test_inf_and_nan_stay_in_their_slice(fls, M, K, N, sparsity, plan):
    """An Inf of X at the first k behind a slice or behind the last K tile must not meet the zero tiles that fill a body
    up: against stored weights everywhere it gives Inf, never NaN."""
    W = wl.dense_bits(wl.gen_weights_f32(M, K, 91))
    g = np.random.Generator(np.random.Philox(92))
    W[g.random((M, K)) < sparsity] = 0
    X = wl.gen_x(N, K, 93)
    for i, k in enumerate(range(0, K, 32)):  # one Inf per K tile, in a column of its own
        W[:, k] = 0x2400
        X[i % N, k] = 0x7C00 if i % 2 else 0xFC00
    X[N - 1, 5] = 0x7E00
    with np.errstate(invalid="ignore"):
        ref = _f64(X) @ _f64(W).T
    blob, stats = _compress(fls, W, 1)
    assert _plan(fls, stats, N) == plan
    C = _call(fls, blob, X, M, K, N)
    finite = np.isfinite(ref)
    assert np.isinf(ref).any() and np.isnan(ref).any() and finite.any()
    for test in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(test(C), test(ref))
    assert np.abs(C[finite] - ref[finite]).max() / np.abs(ref[finite]).max() <= TOL
