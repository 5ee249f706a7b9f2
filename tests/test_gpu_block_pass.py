"""The block pass of fls_spmm (calls of more than 64 columns): edges of its tiles, bodies and slices, at shapes that the
estimate behind the dispatch sends to it.  C against the product in 64 bits of the same fp16 operands.

Tolerance: products of fp16 values are exact in fp32; a sum of K <= 3040 of them in fp32 is off by at most K * 2^-24 of the
sum of their magnitudes (about 2e-4 of it, and far less in effect), fp16 rounding adds 2^-11 of the value: 2e-3 of the
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
    return (fls.fls_compress_v2 if version == 2 else fls.fls_compress)(Wd)[0]


@pytest.mark.parametrize("M,K,N,sparsity,version", [
    # 256 columns x two bands, no slices: an odd number of bands, K tiles that are no multiple of three, a last
    # column group with one column
    (3968, 544, 257, 0.7, 1),
    (3968, 544, 512, 0.7, 2),
    (3968, 544, 512, 0.9, 1),
    # ... K slices of unequal length, three column groups, a last one that is half empty
    (896, 3040, 641, 0.7, 2),
    (1664, 3040, 129, 0.5, 2),   # tiles of ten rounds
    (1664, 1696, 513, 0.55, 1),
    # 128 columns x four bands, an incomplete group of bands
    (15232, 544, 125, 0.7, 1),
    (15232, 544, 125, 0.8, 2),
    # ... in four K slices
    (7296, 1696, 125, 0.7, 1),
])
def test_edges(fls, M, K, N, sparsity, version):
    W = wl.prune_uniform(wl.gen_weights_f32(M, K, 71), sparsity, 72)
    X = wl.gen_x(N, K, 73)
    ref = _f64(X) @ _f64(W).T
    C = _call(fls, _compress(fls, W, version), X, M, K, N)
    assert np.abs(C - ref).max() / np.abs(ref).max() <= TOL


@pytest.mark.parametrize("version", [1, 2])
def test_denser_blob_behind_the_librarys_back(fls, version):
    """The variant is picked for the sparse blob that the library remembers; the denser one that stands there by the
    time of the call does not fit its stages and takes the plain loop."""
    import torch

    M, K, N = 3968, 544, 513
    W32 = wl.gen_weights_f32(M, K, 81)
    X = wl.gen_x(N, K, 82)
    sparse, dense = (_compress(fls, wl.prune_uniform(W32, s, 83), version).clone() for s in (0.8, 0.45))
    ref = _f64(X) @ _f64(wl.prune_uniform(W32, 0.45, 83)).T
    place = torch.zeros(dense.numel(), dtype=torch.uint8, device="cuda")
    place[:sparse.numel()].copy_(sparse)
    _call(fls, place, X, M, K, N)
    place.copy_(dense)
    C = _call(fls, place, X, M, K, N)
    fls.fls_forget(place)
    assert np.abs(C - ref).max() / np.abs(ref).max() <= TOL


@pytest.mark.parametrize("M,K,N", [(3968, 544, 300), (896, 3040, 641)])
def test_inf_and_nan_stay_in_their_slice(fls, M, K, N):
    """An Inf of X at the first k behind a slice or behind the last K tile must not meet the zero tiles that fill a body
    up: against stored weights everywhere it gives Inf, never NaN."""
    W = wl.dense_bits(wl.gen_weights_f32(M, K, 91))
    g = np.random.Generator(np.random.Philox(92))
    W[g.random((M, K)) < 0.7] = 0
    X = wl.gen_x(N, K, 93)
    for i, k in enumerate(range(0, K, 32)):  # one Inf per K tile, in a column of its own
        W[:, k] = 0x2400
        X[i % N, k] = 0x7C00 if i % 2 else 0xFC00
    X[N - 1, 5] = 0x7E00
    with np.errstate(invalid="ignore"):
        ref = _f64(X) @ _f64(W).T
    C = _call(fls, _compress(fls, W, 1), X, M, K, N)
    finite = np.isfinite(ref)
    assert np.isinf(ref).any() and np.isnan(ref).any() and finite.any()
    for test in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(test(C), test(ref))
    assert np.abs(C[finite] - ref[finite]).max() / np.abs(ref[finite]).max() <= TOL
