"""Passes of up to 32 columns (and, at 40 and 64 columns, whichever pass the rule takes) on problems of a few tiles to a few hundred per band: whole bands, bands cut into shares that stay on
one XCD, bands cut across XCDs, owners with many slots to add - against the oracle, on the registered workspace and on the
static one, eager and replayed from a graph."""
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


def _operands(bands, kt, N, sparsity, seed):
    import torch

    W = wl.prune_uniform(wl.gen_weights_f32(bands * 128, kt * 32, seed), sparsity, seed + 1)
    X = wl.gen_x(N, kt * 32, seed + 2)
    return W, X, torch.from_numpy(W.view(np.float16)).cuda(), torch.from_numpy(X.view(np.float16)).cuda()


@pytest.mark.parametrize("N,version", [(8, 1), (8, 2), (24, 1), (32, 2), (40, 1), (64, 2)])
@pytest.mark.parametrize("bands,kt", [
    (1, 1), (8, 2), (8, 3), (5, 7), (8, 8),  # fewer than eight tiles to a band: several bands to a workgroup
    (8, 9), (3, 31), (8, 32), (7, 63),       # whole bands, or cut into shares of at least eight tiles
    (9, 144), (1, 512), (3, 700), (42, 51),  # many shares to a band; bands that lie on two XCDs
    (257, 4), (300, 9), (270, 40),           # more bands than CUs: whole bands, or all tiles cut evenly
    (130, 36), (130, 88),                    # more than half as many: whole bands, or all tiles cut evenly (dense; and 24 columns)
])
def test_products_of_every_cut(fls, oracle_mod, bands, kt, N, version):
    import torch

    M, K = bands * 128, kt * 32
    W, X, Wd, Xd = _operands(bands, kt, N, 0.75, 7000 + 13 * bands + kt)
    blob, stats = (fls.fls_compress_v2 if version == 2 else fls.fls_compress)(Wd)
    ref = oracle_mod.ref_spmm_f64(W, X)
    scale = float(np.abs(ref).max())
    fls.ensure_workspace(M, K, N)
    calls = [lambda C: fls.fls_spmm(blob, Xd, C, M, K, N)]
    if N <= fls.NOALLOC_MAX_N:
        calls.append(lambda C: fls.fls_spmm_noalloc(blob, stats, Xd, C, M, K, N))
    if version == 1:
        calls.append(lambda C: fls.fls_dense_gemm(Wd, Xd, C, M, K, N))
    for call in calls:
        for _ in range(3):  # the flags that a call leaves are the ones the next finds
            C = torch.full((N, M), float("nan"), dtype=torch.float16, device="cuda")
            call(C)
            assert float(np.abs(C.cpu().numpy().astype(np.float64) - ref).max()) / scale <= TOL
    fls.fls_check_workspace()
    fls.fls_forget(blob)


@pytest.mark.parametrize("N", [33, 64, 66, 80, 97, 143, 200])
@pytest.mark.parametrize("bands,kt", [(1, 1), (3, 3), (9, 5), (5, 131), (241, 2)])
def test_dense_products_of_many_columns(fls, oracle_mod, bands, kt, N):
    """K slices down to two steps of 64 k, a half last step, and a rest of up to 32 columns in the launch of the others or in a pass of its own."""
    import torch

    M, K = bands * 128, kt * 32
    W, X, Wd, Xd = _operands(bands, kt, N, 0.3, 7500 + 13 * bands + kt)
    ref = oracle_mod.ref_spmm_f64(W, X)
    fls.ensure_workspace(M, K, N)
    for _ in range(2):
        C = torch.full((N, M), float("nan"), dtype=torch.float16, device="cuda")
        fls.fls_dense_gemm(Wd, Xd, C, M, K, N)
        assert float(np.abs(C.cpu().numpy().astype(np.float64) - ref).max()) / float(np.abs(ref).max()) <= TOL
    fls.fls_check_workspace()


@pytest.mark.parametrize("entry", ["fls_spmm_stats", "fls_spmm_noalloc"])
def test_two_matrices_in_one_graph_with_eager_calls_between_replays(fls, oracle_mod, entry):
    """Slots and flags change hands between two matrices with different cuts, in graph order and out of it."""
    import torch

    N, cases = 16, []
    for bands, kt in ((9, 144), (42, 51)):
        W, X, Wd, Xd = _operands(bands, kt, N, 0.8, 7900 + bands)
        M, K = bands * 128, kt * 32
        blob, stats = fls.fls_compress(Wd)
        fls.ensure_workspace(M, K, N)
        C = torch.zeros((N, M), dtype=torch.float16, device="cuda")
        cases.append((blob, stats, Xd, C, M, K, N, oracle_mod.ref_spmm_f64(W, X)))
    run = getattr(fls, entry)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for c in cases:
            run(*c[:7])
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            for c in (cases + cases[::-1]) * 3:
                run(*c[:7])
        for i in range(20):
            for c in cases:
                c[3].fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            for c in cases:
                assert float(np.abs(c[3].cpu().numpy().astype(np.float64) - c[7]).max()) / float(np.abs(c[7]).max()) <= TOL, i
            run(*cases[i % 2][:7])
    torch.cuda.synchronize()
    fls.fls_check_workspace()


class _Memory:
    """Device memory of the library as something torch can view."""

    def __init__(self, ptr, words, typestr):
        self.__cuda_array_interface__ = {"data": (ptr, False), "shape": (words,), "typestr": typestr, "version": 3}


@pytest.mark.parametrize("recorded", [False, True])
def test_flags_that_a_call_which_gave_up_left_raised(fls, oracle_mod, recorded):
    """A hand-over that was given up leaves its flag raised and its slot filled.  Neither a later call nor a further replay of the same
    recorded call, which bears the same number, may take them for its own: flags and slots are filled as such a call would leave them (every
    one, the slots with NaN), and the error word stays for fls_check_workspace."""
    import ctypes

    import torch

    N, bands, kt = 16, 42, 51
    M, K = bands * 128, kt * 32
    W, X, Wd, Xd = _operands(bands, kt, N, 0.8, 7950)
    ref = oracle_mod.ref_spmm_f64(W, X)
    blob, stats = fls.fls_compress(Wd)
    scratch = fls.lib().fls_internal_noalloc_scratch
    scratch.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.POINTER(ctypes.c_void_p), ctypes.POINTER(ctypes.c_uint32)]
    control, parts, number = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_uint32()
    C = torch.empty((N, M), dtype=torch.float16, device="cuda")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        fls.fls_spmm_noalloc(blob, stats, Xd, C, M, K, N)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            fls.fls_spmm_noalloc(blob, stats, Xd, C, M, K, N)
        assert scratch(ctypes.byref(control), ctypes.byref(parts), ctypes.byref(number)) == fls.OK
        words = torch.as_tensor(_Memory(control.value, 2048, "<i4"), device="cuda")
        slots = torch.as_tensor(_Memory(parts.value, 512 * 2 * 2048, "<f4"), device="cuda")
        assert words.data_ptr() == control.value and slots.data_ptr() == parts.value
        for i in range(4):
            slots.fill_(float("nan"))
            words[:512] = number.value  # of partial sums in memory, of those in an XCD's L2
            words[1536:] = number.value
            words[512] = 1
            C.fill_(float("nan"))
            if recorded:
                graph.replay()
            else:
                fls.fls_spmm_noalloc(blob, stats, Xd, C, M, K, N)
            torch.cuda.synchronize()
            if recorded:  # none that this replay could have taken for its own, none for the next
                assert torch.nonzero(words).flatten().tolist() == [512]
            assert float(np.abs(C.cpu().numpy().astype(np.float64) - ref).max()) / float(np.abs(ref).max()) <= TOL, i
            with pytest.raises(fls.FlsError) as e:
                fls.fls_check_workspace()
            assert e.value.code == fls.EHANDOVER
            torch.cuda.synchronize()
            assert int(words.abs().max()) == 0
        fls.fls_check_workspace()
