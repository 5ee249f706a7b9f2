"""Times of the passes that a product of more than 64 columns can take, beside the estimate that picks one of them
(spmm_pass_share in csrc/fls_spmm_block.hip).

Builds three copies of libfls.so with -DFLS_PASS=<p>, which take pass p (0 the 64-column pass, 1 and 2 the block pass with
that share) for every such call, times them in turn on a list of products and prints one line each: the three times in
us, the pass that the library picks and its time over the shortest.  Weights N(0, 0.02) pruned uniformly, X N(0, 1), drawn on the
GPU; a call's blob is one of several copies of more than 512 MB in all.  Share 1 stages at most six rounds of a tile: no time beyond.

    python -m paper_2309_10285_amd.pass_times --build-only --keep DIR   (no GPU needed)
    python -m paper_2309_10285_amd.pass_times --prebuilt DIR [--only products|ends|small|drawn] [--draw 60] [--seed 5]
"""
import argparse
import ctypes
import os
import random
import statistics
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

from paper_2309_10285_amd import latency_breakdown as lb  # noqa: E402

BLOCK_SOURCE = ("fls_spmm_block.hip",)


def products():
    """(M, K, sparsity, version, N) of products like those of a model's layers."""
    out = [(7168, 28672, 0.8, 1, n) for n in (80, 128, 192, 256, 384, 1000, 4096)]
    out += [(12288, 12288, 0.8, 1, n) for n in (80, 128, 192, 256, 384, 512, 1000, 4096)]
    out += [(12288, 12288, 0.7, 2, n) for n in (128, 256, 384, 1000, 4096)]
    out += [(m, m, 0.9, 1, n) for m in (9216, 12288) for n in (128, 256, 512, 1024, 2048, 4096)]
    out += [(12288, 12288, 0.6, 1, n) for n in (128, 256, 512, 2048)]
    out += [(28672, 7168, 0.9, 1, n) for n in (128, 256, 512, 1000, 4096)]
    return out + [(4096, 4096, 0.6, 1, n) for n in (80, 128, 256, 384, 512, 1000, 4096)]


def drawn(count, seed):
    """Products of any size: M and K spread over the logarithm of 128 ... 49152 and 32 ... 49152, N of 65 ... 4096."""
    rng, out = random.Random(seed), []
    for _ in range(count):
        M, K = int(128 * 384 ** rng.random()) // 128 * 128, int(32 * 1536 ** rng.random()) // 32 * 32
        K = min(K, 12288 * 49152 // M // 32 * 32)
        N = min(int(65 * 63 ** rng.random()), max(65, 12288 * 12288 * 4096 // (M * K)))
        out.append((M, K, round(rng.uniform(0.5, 0.9), 2), rng.choice((1, 1, 2)), N))
    return out


def ends():
    """K tiles that fill no body of the 64-column pass (eight tiles up to four rounds a tile, four beyond), at every density."""
    out = []
    for sparsity, version in ((0.9, 1), (0.85, 1), (0.8, 1), (0.7, 1), (0.6, 1), (0.5, 1), (0.8, 2), (0.6, 2)):
        for kt in ((96, 97, 98, 100, 103) if sparsity >= 0.8 else (96, 97, 98, 99)):
            out.append((12288, 32 * kt, sparsity, version, 512))
    return out


def small():
    """Few K tiles."""
    return [(M, 32 * kt, s, 1, n) for M, n in ((12288, 4096), (4096, 1000), (28672, 256)) for s in (0.9, 0.8, 0.6) for kt in (1, 2, 3, 5, 7, 8, 11, 15)]


def measure(libs, fls, M, K, sparsity, version, N):
    import torch

    gen = torch.Generator(device="cuda").manual_seed(M + K + N)
    W = torch.empty((M, K), dtype=torch.float16, device="cuda")
    for r in range(0, M, 4096):
        w = torch.randn((min(4096, M - r), K), generator=gen, device="cuda") * 0.02
        W[r:r + 4096] = torch.where(torch.rand(w.shape, generator=gen, device="cuda") < 1.0 - sparsity, w, torch.zeros_like(w)).half()
    X = torch.randn((N, K), generator=gen, device="cuda").half()
    C = torch.empty((N, M), dtype=torch.float16, device="cuda")
    blob, st = (fls.fls_compress_v2 if version == 2 else fls.fls_compress)(W)
    del W
    blobs = [blob.clone() for _ in range(max(2, min(32, -(-(1 << 29) // st["bytes_total"]))))]
    plan = fls.spmm_plan(st, N, torch.cuda.get_device_properties(0).multi_processor_count)
    ws = torch.empty(fls.fls_workspace_bytes(M, K, N), dtype=torch.uint8, device="cuda")
    vp = ctypes.c_void_p
    stream = vp(torch.cuda.current_stream().cuda_stream)
    stats = fls.FlsStats(**{k: st[k] for k, _ in fls.FlsStats._fields_})
    passes = [0, 1, 2] if -(-st["max_tile_words"] // (192 if version == 2 else 256)) <= 6 else [0, 2]
    times = {p: [] for p in passes}

    def loop(L, n):
        for i in range(n):
            rc = L.fls_spmm_stats(vp(blobs[i % len(blobs)].data_ptr()), ctypes.byref(stats), vp(X.data_ptr()), vp(C.data_ptr()), M, K, N, stream)
            assert rc == 0, rc

    for p in passes:
        assert libs[p].fls_set_workspace(vp(ws.data_ptr()), ws.numel(), stream) == 0
        loop(libs[p], 3)
    torch.cuda.synchronize()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    n = max(5, min(100, int(4e12 / (2.0 * M * K * N))))
    for _ in range(5):
        for p in passes:
            a.record()
            loop(libs[p], n)
            b.record()
            b.synchronize()
            times[p].append(a.elapsed_time(b) / n * 1e3)
    us = {p: statistics.median(t) for p, t in times.items()}
    pick = plan["share"] if plan["pass"] == "block" else 0
    print("%6d %6d %.2f v%d N %4d R %2d | %s | pick %d %.3f of the best, %.3f of the 64-column pass" % (
        M, K, sparsity, version, N, -(-st["max_tile_words"] // (192 if version == 2 else 256)),
        " ".join("%8.1f" % us[p] if p in us else "       -" for p in (0, 1, 2)), pick, us[pick] / min(us.values()), us[pick] / us[0]), flush=True)
    return us[pick] / min(us.values())


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--keep", default="", help="folder for the builds (kept); default: a temporary directory")
    ap.add_argument("--build-only", action="store_true")
    ap.add_argument("--prebuilt", default="", help="folder with builds made by --build-only")
    ap.add_argument("--only", choices=("products", "ends", "small", "drawn"), default="")
    ap.add_argument("--draw", type=int, default=60)
    ap.add_argument("--seed", type=int, default=5)
    args = ap.parse_args()
    tmp = None if args.prebuilt or args.keep else tempfile.TemporaryDirectory()
    folder = args.prebuilt or args.keep or tmp.name
    if not args.prebuilt:
        for p in (0, 1, 2):
            lb.build_with(f"pass{p}", f"-DFLS_PASS={p}", BLOCK_SOURCE, folder)
    if args.build_only:
        return

    import torch  # noqa: F401  (first: the libraries are to use the HIP runtime that torch brings)

    import paper_2309_10285_amd as fls

    vp, i64 = ctypes.c_void_p, ctypes.c_int64
    libs = {}
    for p in (0, 1, 2):
        L = libs[p] = ctypes.CDLL(os.path.join(folder, f"libfls_pass{p}.so"))
        L.fls_spmm_stats.argtypes = [vp, ctypes.POINTER(fls.FlsStats), vp, vp, i64, i64, i64, vp]
        L.fls_set_workspace.argtypes = [vp, ctypes.c_size_t, vp]
    for name, what in (("products", products), ("ends", ends), ("small", small), ("drawn", lambda: drawn(args.draw, args.seed))):
        if args.only in ("", name):
            print(name + ": M K sparsity version N, rounds of the densest tile | us in the 64-column pass, share 1, share 2 | the library's pick", flush=True)
            regret = [measure(libs, fls, *c) for c in what()]
            print("%s: %d, the pick takes %.3f of the best pass's time (geometric mean), %.3f at most" % (
                name, len(regret), statistics.geometric_mean(regret), max(regret)), flush=True)
    if tmp:
        tmp.cleanup()


if __name__ == "__main__":
    main()
