"""The compressor works on chunks of 16 tiles and stages 2048 entries of a tile at a time: bit for bit against the oracle
around both edges, in both formats, and within a buffer that is too small."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fls():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2309_10285_amd as f

    f.lib()
    return f


def _dev(bits):
    import torch

    return torch.from_numpy(bits.view(np.float16)).cuda()


def _weights(bands, kt, stored, seed):
    """Tile j (band-major) holds exactly stored[j % len(stored)] elements at random places."""
    g = np.random.Generator(np.random.Philox(seed))
    W = np.zeros((bands, kt, 4096), dtype=np.uint16)
    for j in range(bands * kt):
        n = stored[j % len(stored)]
        W[j // kt, j % kt, g.permutation(4096)[:n]] = g.integers(1, 65536, size=n, dtype=np.uint32).astype(np.uint16)
    return np.ascontiguousarray(W.reshape(bands, kt, 128, 32).transpose(0, 2, 1, 3).reshape(bands * 128, kt * 32))


@pytest.mark.parametrize("version", [1, 2])
@pytest.mark.parametrize("bands,kt", [(1, 1), (1, 15), (2, 8), (1, 17), (3, 5), (67, 17), (5, 1025)])
def test_chunk_edges(fls, oracle_mod, version, bands, kt):
    W = _weights(bands, kt, [800, 0, 1, 2047, 2048, 2049, 4096, 5, 64], 11)
    blob, st = (fls.fls_compress_v2 if version == 2 else fls.fls_compress)(_dev(W))
    ref = (oracle_mod.ref_compress_v2 if version == 2 else oracle_mod.ref_compress)(W)
    assert np.array_equal(blob.cpu().numpy(), ref)
    assert st["nnz"] == int(np.count_nonzero(W))


@pytest.mark.parametrize("version", [1, 2])
def test_too_small_buffer_is_not_overrun(fls, version):
    import torch

    compress = fls.fls_compress_v2 if version == 2 else fls.fls_compress
    W = _dev(_weights(3, 17, [700, 3000], 12))
    size = compress(W)[1]["bytes_total"]
    index = 64 + 4 * ((3 * 17 + 4 + 15) // 16 * 16)
    for room in (size - 16, size // 2 // 16 * 16, index):
        buf = torch.full((size + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        with pytest.raises(fls.FlsError) as e:
            compress(W, buf[:room])
        assert e.value.code == fls.ECAPACITY
        assert bool((buf[room:] == 0xA5).all())
    assert compress(W, torch.empty(size, dtype=torch.uint8, device="cuda"))[1]["bytes_total"] == size


@pytest.mark.parametrize("version", [1, 2])
def test_lane_edges(fls, oracle_mod, version):
    """A lane walks 64 consecutive locations in two words of 32: one to four elements a tile around those edges, gaps about the
    63 locations that a distance reaches, in either half of a word of W, among them bit patterns with an empty byte."""
    g = np.random.Generator(np.random.Philox(21))
    bands, kt = 6, 96
    flat = np.zeros((bands * kt, 4096), dtype=np.uint16)
    values = np.array([0x8000, 0x0001, 0x00FF, 0x0100, 0xFF00, 0xFFFF, 0x7C00], dtype=np.uint16)
    for t in flat:
        at = int(g.choice([0, 1, 31, 32, 33, 62, 63, 64, 65, 127, 128, 4032, 4094, 4095])) if g.random() < 0.5 else int(g.integers(4096))
        for _ in range(int(g.integers(0, 5))):
            t[at % 4096] = g.choice(values)
            at += int(g.choice([1, 2, 31, 32, 62, 63, 64, 65, 126, 127, 128, 190, 1000, 3969]))
    # location l of a tile is row (l % 1024) // 8, column 8 * (l // 1024) + l % 8
    tiles = flat.reshape(bands, kt, 4, 128, 8).transpose(0, 3, 1, 2, 4)
    W = np.ascontiguousarray(tiles.reshape(bands * 128, kt * 32))
    blob, st = (fls.fls_compress_v2 if version == 2 else fls.fls_compress)(_dev(W))
    assert np.array_equal(blob.cpu().numpy(), (oracle_mod.ref_compress_v2 if version == 2 else oracle_mod.ref_compress)(W))
    assert st["nnz"] == int(np.count_nonzero(W))


def test_more_threads_than_the_library_has_scratch_for(fls, oracle_mod):
    """24 threads on streams of their own, several matrices each, against the oracle: a call waits for a place of the 16."""
    import threading

    import torch

    shapes = [(1, 1), (3, 5), (2, 40), (7, 33)]
    Ws = [_weights(b, kt, [700 + 40 * i, 3, 0, 2100], 31 + i) for i, (b, kt) in enumerate(shapes)]
    refs = {v: [(oracle_mod.ref_compress_v2 if v == 2 else oracle_mod.ref_compress)(W) for W in Ws] for v in (1, 2)}
    on_gpu = [_dev(W) for W in Ws]
    torch.cuda.synchronize()
    wrong = []

    def work(n):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for k in range(8):
                    i, v = (n + k) % len(Ws), 1 + (n + k // 4) % 2
                    blob, st = (fls.fls_compress_v2 if v == 2 else fls.fls_compress)(on_gpu[i])
                    if not np.array_equal(blob.cpu().numpy(), refs[v][i]) or st["nnz"] != int(np.count_nonzero(Ws[i])):
                        wrong.append((n, k))
        except Exception as e:  # an exception in a thread would go unseen
            wrong.append((n, repr(e)))

    threads = [threading.Thread(target=work, args=(n,)) for n in range(24)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


def _compress_as(fls, Wd, bands, kt, version, room, look_limit, by_ticket):
    """fls_compress with those looks before it gives up and that order of chunks: the buffer, nnz, kernel runs by number and by ticket."""
    import ctypes

    import torch

    f = fls.lib().fls_internal_compress
    f.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_int,
                  ctypes.POINTER(ctypes.c_uint32), ctypes.POINTER(fls.FlsStats), ctypes.c_void_p]
    out = torch.zeros(room, dtype=torch.uint8, device="cuda")
    st, runs = fls.FlsStats(), (ctypes.c_uint32 * 2)()
    stream = torch.cuda.current_stream().cuda_stream
    assert f(Wd.data_ptr(), bands * 128, kt * 32, out.data_ptr(), out.numel(), version, look_limit, by_ticket, runs, ctypes.byref(st), stream) == fls.OK
    return out.cpu().numpy(), st.nnz, tuple(runs)


@pytest.mark.parametrize("version", [1, 2])
@pytest.mark.parametrize("bands,kt", [(1, 1), (3, 5), (4, 33), (16, 1025)])
def test_chunks_by_ticket(fls, oracle_mod, version, bands, kt):
    """One chunk, several, and four to a CU, in the order in which workgroups start: three times on one place of the scratch (the
    ticket counts from 0 each time), and by number on that place afterwards."""
    W = _weights(bands, kt, [800, 0, 2049, 30], 41)
    ref = (oracle_mod.ref_compress_v2 if version == 2 else oracle_mod.ref_compress)(W)
    Wd, nnz = _dev(W), int(np.count_nonzero(W))
    for by_ticket in (1, 1, 1, 0):
        got, stored, runs = _compress_as(fls, Wd, bands, kt, version, len(ref) + 16, 1 << 22, by_ticket)
        assert np.array_equal(got[:len(ref)], ref) and stored == nnz and runs == (1 - by_ticket, by_ticket)


@pytest.mark.parametrize("version", [1, 2])
def test_a_kernel_that_gives_up_is_run_again_by_ticket(fls, oracle_mod, version):
    """With 1025 chunks, four to a CU, some workgroup looks for a word that is not there yet: the call is made again with chunks by
    ticket, on the place that the run before left marked and that is cleared first.  Several in a row, and ordinary ones in between."""
    bands, kt = 16, 1025
    W = _weights(bands, kt, [800, 0, 2049, 30], 41)
    ref = (oracle_mod.ref_compress_v2 if version == 2 else oracle_mod.ref_compress)(W)
    Wd, nnz = _dev(W), int(np.count_nonzero(W))
    again = 0
    for look_limit in (1, 1, 1 << 22, 1):
        got, stored, runs = _compress_as(fls, Wd, bands, kt, version, len(ref) + 16, look_limit, 0)
        assert np.array_equal(got[:len(ref)], ref) and stored == nnz
        assert runs in ((1, 0), (1, 1)) and (look_limit == 1 or runs == (1, 0))
        again += runs[1]
    assert again > 0
