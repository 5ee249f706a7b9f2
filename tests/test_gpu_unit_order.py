"""How the 64-column passes, sparse and dense, spread their units over the XCDs: whole (group of four bands, K slice) pairs in
turn, or an even cut of all units where whole pairs would cost a round more.  Shapes of either kind, every element of C
against the product in 64 bits (a unit that nobody takes leaves its part of C at NaN, one that two take does not show).

Tolerance: products of fp16 values are exact in fp32, sums of K <= 2048 of them are off by far less than the fp16 rounding of
C, 2^-11 of the value: 2e-3 of the largest value, as in the other parity tests.
"""
import ctypes

import numpy as np
import pytest

import fls_workloads as wl

pytestmark = pytest.mark.gpu

TOL = 2e-3


def _whole(M, N, slices, cus):
    """whole_pairs of csrc/fls_launch.h for that many slices."""
    pairs, groups, per_xcd = -(-M // 512) * slices, -(-N // 64), cus // 8
    return -(-(-(-pairs // 8) * groups) // per_xcd) == -(-(-(-pairs * groups // 8)) // per_xcd)


@pytest.mark.parametrize("M,K,N,whole", [
    (4608, 64, 1088, False),   # nine groups of four bands x 17 groups of columns
    (4224, 64, 1061, False),   # ... the last group of bands and the last of columns incomplete
    (2432, 2048, 720, False),  # five groups of bands in four K slices
    (4096, 64, 1088, True),    # eight groups of bands
    (1536, 1024, 128, True),   # three in K slices
])
def test_every_unit_is_taken(M, K, N, whole):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2309_10285_amd as fls

    cus = torch.cuda.get_device_properties(0).multi_processor_count
    W = wl.prune_uniform(wl.gen_weights_f32(M, K, 61), 0.8, 62)
    X = wl.gen_x(N, K, 63)
    ref = X.view(np.float16).astype(np.float64) @ W.view(np.float16).astype(np.float64).T
    Wd, Xd = (torch.from_numpy(a.view(np.float16)).cuda() for a in (W, X))
    fls.ensure_workspace(M, K, N)
    blob, stats = fls.fls_compress(Wd)
    plan = fls.spmm_plan(stats, N, cus)
    dense = (ctypes.c_uint32 * 2)()
    fls.lib().fls_internal_dense_plan(M, K, N, cus, dense)
    assert plan["pass"] == "wide" and dense[0] == -(-N // 64)
    assert _whole(M, N, plan["slices"], cus) == whole and _whole(M, N, dense[1], cus) == whole
    for call, first in ((fls.fls_spmm, blob), (fls.fls_dense_gemm, Wd)):
        C = torch.full((N, M), float("nan"), dtype=torch.float16, device="cuda")
        call(first, Xd, C, M, K, N)
        torch.cuda.synchronize()
        err = np.abs(C.cpu().numpy().astype(np.float64) - ref).max() / np.abs(ref).max()
        assert err <= TOL, (call.__name__, err)
