"""The calls whose time matters to a user of this library, as one list and as ranges to draw more from.

Four kinds of work, each through the package's public entry points:
  spmm     C = W . X with W compressed: the serving path.  N = 1 ... 64 columns is a decode step (a column per sequence
           of the batch), hundreds to thousands of columns a prefill or a large batch.
  layer    the four weight products of one decoder layer (QKV, attention output, FFN up and down), one after the
           other on fixed buffers, as a decode loop issues them with calls that were prepared once.
  compress dense pruned W -> blob: run once per matrix when a model is loaded.
  dense    C = W . X with W dense: matrices of a model that were not pruned.
Weights are N(0, 0.02) in fp16, pruned by magnitude, uniformly or with row densities ~ Beta(2, 5), activations N(0, 1), as in
the package's benchmark; all of it is drawn on the GPU from the seed alone.
"""
import math
from statistics import NormalDist

import numpy as np
import torch

import paper_2309_10285_amd as fls

SIGMA = 0.02
MOST_WEIGHTS = 12288 * 49152                # the largest matrix of the benchmark's configurations
MOST_PRODUCTS = 12288 * 12288 * 4096        # M * K * N of the largest listed call


def _spmm(name, M, K, N, sparsity, mask, version=1, entry="fls_spmm"):
    return {"name": name, "op": "spmm", "M": M, "K": K, "N": N, "sparsity": sparsity, "mask": mask, "version": version, "entry": entry}


def listed():
    return [
        # a small projection in a decode step: nothing but latency
        _spmm("spmm-1024x1024-n8", 1024, 1024, 8, 0.8, "uniform"),
        # fused QKV of a 66B-shaped model, decode with a batch of 32
        _spmm("spmm-27648x9216-n32", 27648, 9216, 32, 0.7, "magnitude"),
        # FFN down-projection of a 175B-shaped model, decode with a batch of 64: the benchmark's headline
        _spmm("spmm-12288x49152-n64", 12288, 49152, 64, 0.9, "magnitude"),
        # FFN up-projection of a 175B-shaped model, batch of 8, 3-byte format: the longest stream of a decode step
        _spmm("spmm-49152x12288-n8-v2", 49152, 12288, 8, 0.7, "magnitude", version=2),
        # attention output projection with unevenly pruned rows, an odd batch, on the entry that allocates nothing
        _spmm("spmm-12288x12288-n13-noalloc", 12288, 12288, 13, 0.8, "row_skewed", entry="fls_spmm_noalloc"),
        # the same projection, batch of 128
        _spmm("spmm-12288x12288-n128", 12288, 12288, 128, 0.8, "magnitude"),
        # a prefill of 1000 tokens (no multiple of any tile) through an FFN down-projection
        _spmm("spmm-7168x28672-n1000", 7168, 28672, 1000, 0.8, "magnitude"),
        # a long prefill, 3-byte format: the largest call
        _spmm("spmm-12288x12288-n4096-v2", 12288, 12288, 4096, 0.7, "magnitude", version=2),
        # one 30B-shaped decoder layer, decode with a batch of 16
        {"name": "layer-7168-n16", "op": "layer", "hidden": 7168, "N": 16, "sparsity": 0.8, "mask": "magnitude", "version": 1},
        # model loading, both formats
        {"name": "compress-28672x7168", "op": "compress", "M": 28672, "K": 7168, "sparsity": 0.8, "mask": "magnitude", "version": 1},
        {"name": "compress-12288x12288-v2", "op": "compress", "M": 12288, "K": 12288, "sparsity": 0.9, "mask": "row_skewed", "version": 2},
        # a matrix that was left dense, decode with a batch of 16
        {"name": "dense-28672x7168-n16", "op": "dense", "M": 28672, "K": 7168, "N": 16},
    ]


def _log_int(rng, lo, hi, step=1):
    """An integer in [lo, hi], a multiple of `step`, spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))
    return min(hi // step * step, max(-(-lo // step) * step, int(v) // step * step))


def _matrix(rng, most):
    """M (a multiple of 128) and K (of 32), each 1024 ... 49152, of at most `most` weights."""
    M = _log_int(rng, 1024, 49152, 128)
    K = _log_int(rng, 1024, min(49152, most // M), 32)
    return (M, K) if K % 128 or rng.random() < 0.5 or K * M > most else (K, M)


def draw(rng):
    """One more case: the listed kinds over their ranges (sparsity 60 - 90 %, N 1 ... 4096, odd ones among them)."""
    kind = rng.choices(["spmm", "layer", "compress", "dense"], weights=[7, 1, 2, 1])[0]
    s, mask, version = round(rng.uniform(0.6, 0.9), 3), rng.choice(["magnitude", "uniform", "row_skewed"]), rng.choice([1, 1, 2])
    if kind == "spmm":
        M, K = _matrix(rng, MOST_WEIGHTS)
        N = _log_int(rng, 1, min(4096, MOST_PRODUCTS // (M * K)))
        entry = "fls_spmm_noalloc" if N <= 32 and rng.random() < 0.25 else rng.choice(["fls_spmm", "fls_spmm", "fls_spmm_stats"])
        return {"op": "spmm", "M": M, "K": K, "N": N, "sparsity": s, "mask": mask, "version": version, "entry": entry}
    if kind == "layer":
        return {"op": "layer", "hidden": _log_int(rng, 1024, 8192, 128), "N": _log_int(rng, 1, 64), "sparsity": s, "mask": mask, "version": version}
    if kind == "compress":
        M, K = _matrix(rng, 28672 * 7168)
        return {"op": "compress", "M": M, "K": K, "sparsity": s, "mask": mask, "version": version}
    M, K = _matrix(rng, 28672 * 7168)
    return {"op": "dense", "M": M, "K": K, "N": _log_int(rng, 1, 256)}


def _weights(M, K, sparsity, mask, gen, rows):
    """Pruned fp16 weights [M, K]; pruned entries are +0."""
    W = torch.empty((M, K), dtype=torch.float16, device="cuda")
    dens = None
    if mask == "row_skewed":
        dens = torch.from_numpy(np.minimum(1.0, (1.0 - sparsity) * rows.beta(2.0, 5.0, size=M) * 3.5).astype(np.float32)).cuda()
    cut = SIGMA * NormalDist().inv_cdf(0.5 + 0.5 * sparsity)  # magnitude pruning of normal weights keeps those above this
    for r in range(0, M, 2048):
        n = min(2048, M - r)
        w = torch.randn((n, K), generator=gen, device="cuda") * SIGMA
        if mask == "magnitude":
            keep = w.abs() > cut
        else:
            keep = torch.rand((n, K), generator=gen, device="cuda") < (1.0 - sparsity if dens is None else dens[r:r + n, None])
        W[r:r + n] = torch.where(keep, w, torch.zeros_like(w)).half()
    return W


def _compress(W, version, out=None):
    return fls.fls_compress_v2(W, out) if version == 2 else fls.fls_compress(W, out)


def _products(case):
    """(M, K) of the products of a case."""
    if case["op"] == "layer":
        h, f = case["hidden"], 4 * case["hidden"]
        return [(3 * h, h), (h, h), (f, h), (h, f)]
    return [(case["M"], case["K"])]


def _operands(case, gen, rows):
    """M, K, X [N, K] and W [M, K] of each product of a case that multiplies, drawn in this order."""
    dense = case["op"] == "dense"
    for M, K in _products(case):
        X = torch.randn((case["N"], K), generator=gen, device="cuda").half()
        yield M, K, X, _weights(M, K, 0.0 if dense else case["sparsity"], "uniform" if dense else case["mask"], gen, rows)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rows = np.random.default_rng(seed)
    if case["op"] == "compress":
        # one buffer for the blob, as a loader keeps one for all its matrices: what is kept of W and a fifth more
        room = int(work(case)["bytes"] - 2.0 * case["M"] * case["K"]) * 6 // 5 // 16 * 16 + 4096
        out = torch.zeros(room, dtype=torch.uint8, device="cuda")
        return {"case": case, "W": _weights(case["M"], case["K"], case["sparsity"], case["mask"], gen, rows), "out": out}
    N, calls, outs = case["N"], [], []
    for M, K, X, W in _operands(case, gen, rows):
        C = torch.empty((N, M), dtype=torch.float16, device="cuda")
        fls.ensure_workspace(M, K, N)
        if case["op"] == "dense":
            calls.append((fls.fls_dense_gemm, (W, X, C, M, K, N)))
        else:
            blob, stats = _compress(W, case["version"])
            if case["op"] == "layer":
                calls.append((fls.prepare_spmm(blob, X, C, M, K, N), ()))
            elif case["entry"] == "fls_spmm":
                calls.append((fls.fls_spmm, (blob, X, C, M, K, N)))
            else:
                calls.append((getattr(fls, case["entry"]), (blob, stats, X, C, M, K, N)))
        outs.append(C)
    return {"case": case, "calls": calls, "outs": outs}


def run(state):
    case = state["case"]
    if case["op"] == "compress":
        _, stats = _compress(state["W"], case["version"], state["out"])
        return {"buffer": state["out"], "stats": stats}  # the whole buffer: its size does not depend on the seed
    for call, args in state["calls"]:
        call(*args)
    return state["outs"]


def work(case):
    """Bytes: the blob (or dense W), X and C once each.  Operations: every product, zeros of W included - the path is
    defined that way (a zero weight times Inf is NaN)."""
    total = {"bytes": 0.0, "flops": 0.0}
    for M, K in _products(case):
        blob = (4 if case.get("version", 1) == 1 else 3) * (1.0 - case.get("sparsity", 0.0)) * M * K + 4.0 * (M // 128) * (K // 32)
        if case["op"] == "compress":
            total["bytes"] += 2.0 * M * K + blob
        else:
            total["bytes"] += (2.0 * M * K if case["op"] == "dense" else blob) + 2.0 * case["N"] * (M + K)
            total["flops"] += 2.0 * M * K * case["N"]
    return total


def tolerance(case):
    """Blobs are a pure function of W.  C is an fp32 sum rounded once to fp16: against the product in fp64 of the same fp16
    operands it is off by 2.1e-4 (2-norm) and by 4.9e-4 of the larger of a value and the root mean square; about four
    times that."""
    return "exact" if case["op"] == "compress" else {"rel": 8e-4, "max": 2e-3}


def exact(case, seed):
    """C in 64 bits from the same fp16 operands, a few thousand rows of W at a time."""
    if case["op"] == "compress":
        return None
    gen = torch.Generator(device="cuda").manual_seed(seed)
    outs = []
    for M, K, X, W in _operands(case, gen, np.random.default_rng(seed)):
        X, C = X.double(), torch.empty((case["N"], M), dtype=torch.float64, device="cuda")
        for r in range(0, M, 4096):
            C[:, r:r + 4096] = X @ W[r:r + 4096].double().T
        outs.append(C)
    return outs
