// C ABI of libfls (see include/fls.h): argument checks on the host, blob header bookkeeping,
// workspace registration, kernel launches.  No device memory is allocated here.
#include "../../include/fls.h"

#include <hip/hip_runtime.h>

#include <condition_variable>
#include <cstring>
#include <mutex>
#include <unordered_map>

#include "fls_launch.h"

namespace {

constexpr uint32_t kMagic = 0x31534C46u;   // "FLS1"
constexpr uint32_t kMagic2 = 0x32534C46u;  // "FLS2"

struct BlobInfo {
  uint64_t M, K;
  uint32_t max_tile_words;
  uint32_t version;
  uint64_t n_off;
};

std::mutex g_mu;
std::unordered_map<const void*, BlobInfo> g_blobs;  // blob address -> validated header
constexpr size_t kMaxRememberedBlobs = 4096;  // beyond this the map is emptied (entries only save a header read-back)
void* g_ws = nullptr;
size_t g_ws_bytes = 0;
int g_num_cus = 0;

// Scratch of fls_spmm_noalloc: the same areas a registered workspace has (control words, then the
// fp32 partial sums of up to 32 columns), in device memory that exists from the moment the library
// is loaded.  Host code never uses the array's name as an address: hipGetSymbolAddress gives the
// address on the current device (every device has its own copy), looked up once per device.
constexpr size_t kScratchControlBytes = 8192;  // control words of the hand-over, none to spare
static_assert(fls::kControlWords * sizeof(uint32_t) <= kScratchControlBytes, "partial sums follow");
constexpr size_t kScratchPartsBytes = (size_t)fls::kMaxWorkgroups * 2 * 2048 * sizeof(float);  // 8 MiB
constexpr size_t kScratchBytes = kScratchControlBytes + kScratchPartsBytes;
static_assert(kScratchBytes == FLS_NOALLOC_SCRATCH_BYTES && FLS_NOALLOC_MAX_N == fls::kGroupCols, "as the header says");
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[kScratchBytes];
constexpr int kMaxDevices = 64;
unsigned char* g_scratch_ptr[kMaxDevices] = {};  // by device id; guarded by g_mu
uint32_t g_scratch_calls = 0;                    // calls of fls_spmm_noalloc; guarded by g_mu

// Address of `scratch` on the current device (nullptr after setting *err on failure).
unsigned char* scratch_on_current_device(int* err) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    *err = FLS_EHIP;
    return nullptr;
  }
  std::lock_guard<std::mutex> lk(g_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      *err = FLS_EHIP;
      return nullptr;
    }
    g_scratch_ptr[dev] = (unsigned char*)ptr;
  }
  return g_scratch_ptr[dev];
}

// Scratch of fls_compress: a device array like the one above and a piece of pinned host memory for what the call returns
// (allocated with the first call).  A call takes one of the kCompressSlots places of its device for its duration - it waits for its kernel -
// and calls of other threads take others; when all are taken a call waits for one.
constexpr int kCompressSlots = 16;
static __device__ __align__(256) __attribute__((used)) unsigned char compress_scratch[kCompressSlots * sizeof(fls::CompressScratch)];
struct CompressSlot {
  bool busy = false;
  bool dirty = false;  // a call on it failed: cleared before the next one
  uint32_t calls = 0;
};
CompressSlot g_compress_slots[kMaxDevices][kCompressSlots];  // guarded by g_mu, as the next two
fls::CompressScratch* g_compress_ptr[kMaxDevices] = {};
fls::CompressHost* g_compress_host = nullptr;  // kMaxDevices x kCompressSlots
std::condition_variable g_compress_free;

// One call's place in it.
struct CompressPlace {
  int dev = -1, slot = -1;
  bool failed = true;  // until the call says otherwise
  fls::CompressScratch* scratch = nullptr;
  fls::CompressHost *host = nullptr, *host_on_device = nullptr;
  uint32_t call = 0;

  bool take(hipStream_t stream) {
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
    bool clear = false;
    {
      std::unique_lock<std::mutex> lk(g_mu);
      if (!g_compress_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(compress_scratch)) != hipSuccess || !ptr) return false;
        g_compress_ptr[dev] = (fls::CompressScratch*)ptr;
      }
      if (!g_compress_host) {
        void* ptr = nullptr;
        if (hipHostMalloc(&ptr, sizeof(fls::CompressHost) * kMaxDevices * kCompressSlots, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) !=
            hipSuccess)
          return false;
        g_compress_host = (fls::CompressHost*)ptr;
      }
      for (;;) {
        for (int i = 0; i < kCompressSlots && slot < 0; ++i)
          if (!g_compress_slots[dev][i].busy) slot = i;
        if (slot >= 0) break;
        g_compress_free.wait(lk);
      }
      CompressSlot& s = g_compress_slots[dev][slot];
      s.busy = true;
      clear = s.dirty || s.calls + 1 == fls::kCompressCalls;
      if (clear) s.calls = 0;
      s.dirty = false;
      call = ++s.calls;
      scratch = g_compress_ptr[dev] + slot;
      host = g_compress_host + dev * kCompressSlots + slot;
    }
    memset(host, 0, sizeof(*host));
    void* ptr = nullptr;
    if (hipHostGetDevicePointer(&ptr, host, 0) != hipSuccess) return false;
    host_on_device = (fls::CompressHost*)ptr;
    return !clear || fls::launch_fill_zero(scratch, sizeof(*scratch), stream) == hipSuccess;
  }
  ~CompressPlace() {
    if (slot < 0) return;
    {
      std::lock_guard<std::mutex> lk(g_mu);
      g_compress_slots[dev][slot].dirty = failed;
      g_compress_slots[dev][slot].busy = false;
    }
    g_compress_free.notify_all();
  }
};

// Looks of a waiting compress workgroup (a microsecond or more each): a tenth of a second before the call is made again with chunks
// by ticket, some seconds then.
constexpr uint32_t kLookLimitByNumber = 1u << 16, kLookLimit = 1u << 22;

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline uint64_t round_up(uint64_t v, uint64_t m) { return (v + m - 1) / m * m; }

bool shape_ok(int64_t M, int64_t K) {
  if (M <= 0 || K <= 0) return false;
  if (M % FLS_TILE_M != 0 || K % FLS_TILE_K != 0) return false;
  // K: byte offsets inside a 128-row band (and inside X) are 32 bit
  if (M > 0x7fffffffll || K > (1ll << 23)) return false;
  // word offsets are 32 bit: the densest possible blob must stay below 2^32 words
  if ((uint64_t)M * (uint64_t)K >= (1ull << 32)) return false;
  return true;
}

uint64_t num_tiles(int64_t M, int64_t K) { return (uint64_t)(M / FLS_TILE_M) * (uint64_t)(K / FLS_TILE_K); }
uint64_t n_off_of(uint64_t tiles) { return round_up(tiles + 4, 16); }

int parse_header(const unsigned char* h, fls_stats* st, BlobInfo* info) {
  uint32_t u[8];
  uint64_t q[4];
  memcpy(u, h, 32);
  memcpy(q, h + 32, 32);
  const bool v2 = u[0] == kMagic2 && u[1] == FLS_FORMAT_VERSION_2;
  if (!v2 && (u[0] != kMagic || u[1] != FLS_FORMAT_VERSION)) return FLS_EFORMAT;
  if (u[2] != FLS_TILE_M || u[3] != FLS_TILE_K || u[4] != FLS_PAD_WORDS || u[5] > (v2 ? 0u : 1u)) return FLS_EFORMAT;
  if (q[0] > 0x7fffffffull || q[1] > 0x7fffffffull || !shape_ok((int64_t)q[0], (int64_t)q[1])) return FLS_EFORMAT;
  const uint64_t tiles = num_tiles((int64_t)q[0], (int64_t)q[1]);
  if (v2) {
    // three words per group of four entries; a tile has at most 4096 stored elements and no bridge then
    if (q[3] % 3 != 0 || q[3] > tiles * (uint64_t)(FLS_TILE_M * FLS_TILE_K / 4 * 3) || q[2] > q[3] / 3 * 4) return FLS_EFORMAT;
    if (u[6] % 3 != 0 || u[6] > FLS_TILE_M * FLS_TILE_K / 4 * 3) return FLS_EFORMAT;
  } else {
    if (q[2] > q[3] || q[3] > tiles * (uint64_t)(FLS_TILE_M * FLS_TILE_K) || q[3] % FLS_PAD_WORDS != 0) return FLS_EFORMAT;
    if (u[6] > FLS_TILE_M * FLS_TILE_K || u[6] % FLS_PAD_WORDS != 0) return FLS_EFORMAT;
  }
  if (st) {
    st->format_version = u[1];
    st->tile_m = u[2];
    st->tile_k = u[3];
    st->order_policy = u[5];
    st->M = q[0];
    st->K = q[1];
    st->nnz = q[2];
    st->num_tiles = tiles;
    st->max_tile_words = u[6];
    st->bytes_header = FLS_HEADER_BYTES;
    st->bytes_offsets = 4 * n_off_of(tiles);
    st->bytes_nonzeros = 4 * q[3];
    st->bytes_total = st->bytes_header + st->bytes_offsets + st->bytes_nonzeros;
  }
  if (info) {
    info->M = q[0];
    info->K = q[1];
    info->max_tile_words = u[6];
    info->version = u[1];
    info->n_off = n_off_of(tiles);
  }
  return FLS_OK;
}

int num_cus() {
  if (g_num_cus == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    g_num_cus = n;
  }
  return g_num_cus;
}

int check_mm_args(const void* W, const void* X, void* C, int64_t M, int64_t K, int64_t N) {
  if (!W || !X || !C) return FLS_EINVAL;
  if (!shape_ok(M, K) || N < 1 || N > FLS_MAX_N) return FLS_EINVAL;
  // X and C are addressed with 32-bit byte offsets through buffer descriptors
  if ((uint64_t)K * (uint64_t)N * 2u > 0x7fffffffull || (uint64_t)M * (uint64_t)N * 2u > 0x7fffffffull) return FLS_EINVAL;
  if (!aligned16(W) || !aligned16(X) || !aligned16(C)) return FLS_EALIGN;
  return FLS_OK;
}

// Workspace: a fixed 4 MiB control area (the control words of the hand-over; the rest
// is spare; cleared when the workspace is registered, and every launch leaves its flags lowered and its owners' XCDs taken back),
// then the split-K partial slots (fp32), then, for N > 32, X repacked into MFMA fragment order
// (K x N rounded up to 16 columns, fp16).  The control area has the same place for every shape, so
// partial sums of one call can never be read as flags by the next.
constexpr size_t kCounterAreaBytes = (size_t)4 << 20;
static_assert(fls::kControlWords * sizeof(uint32_t) <= kCounterAreaBytes, "partial sums follow");

void workspace_layout(int64_t K, int64_t N, size_t* total, size_t* xpack_offset) {
  const size_t parts = fls::parts_floats((uint32_t)N) * sizeof(float);
  if (xpack_offset) *xpack_offset = kCounterAreaBytes + parts;
  *total = kCounterAreaBytes + parts + fls::xpack_bytes((uint32_t)K, (uint32_t)N);
}

}  // namespace

extern "C" {

int fls_compress_bound(int64_t M, int64_t K, size_t* bytes_host) {
  if (!bytes_host || !shape_ok(M, K)) return FLS_EINVAL;
  const uint64_t tiles = num_tiles(M, K);
  *bytes_host = (size_t)(FLS_HEADER_BYTES + 4 * n_off_of(tiles) + 4 * tiles * (uint64_t)(FLS_TILE_M * FLS_TILE_K));
  return FLS_OK;
}

int fls_inspect(const void* header_host, fls_stats* stats_host) {
  if (!header_host || !stats_host) return FLS_EINVAL;
  return parse_header((const unsigned char*)header_host, stats_host, nullptr);
}

static int compress_impl(const void* W_dev, int64_t M, int64_t K, void* out_dev, size_t out_capacity, int order_policy,
                         uint32_t version, fls_stats* stats_host, fls_stream_t stream, uint32_t look_limit = kLookLimitByNumber,
                         bool by_ticket = false, uint32_t* runs = nullptr) {
  if (!W_dev || !out_dev || !shape_ok(M, K)) return FLS_EINVAL;
  if (order_policy != FLS_ORDER_LOCATION) return FLS_EINVAL;  // FLS_ORDER_BANK: not built yet
  if (!aligned16(W_dev) || !aligned16(out_dev)) return FLS_EALIGN;
  const uint64_t tiles = num_tiles(M, K);
  const size_t index_bytes = (size_t)(FLS_HEADER_BYTES + 4 * n_off_of(tiles));
  if (out_capacity < index_bytes) {
    if (stats_host) {
      memset(stats_host, 0, sizeof(*stats_host));
      // the words are not counted yet: the worst case is a size that is certainly enough
      size_t bound = 0;
      if (version == FLS_FORMAT_VERSION_2) fls_compress_bound_v2(M, K, &bound);
      else fls_compress_bound(M, K, &bound);
      stats_host->bytes_total = bound;
    }
    return FLS_ECAPACITY;
  }
  hipStream_t s = (hipStream_t)stream;
  fls::CompressLaunch a;
  a.W = (const uint16_t*)W_dev;
  a.out = (unsigned char*)out_dev;
  a.M = (uint32_t)M;
  a.K = (uint32_t)K;
  a.policy = (uint32_t)order_policy;
  a.version = version;
  a.capacity = out_capacity;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    g_blobs.erase(out_dev);
  }
  unsigned char hdr[FLS_HEADER_BYTES];
  a.look_limit = look_limit;
  a.by_ticket = by_ticket;
  for (;;) {
    if (runs) ++runs[a.by_ticket ? 1 : 0];
    CompressPlace place;
    if (!place.take(s)) return FLS_EHIP;
    a.scratch = place.scratch;
    a.host = place.host_on_device;
    a.call = place.call;
    if (fls::launch_compress(a, s) != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return FLS_EHIP;
    if (!place.host->gave_up) {
      place.failed = false;
      memcpy(hdr, place.host->header, sizeof(hdr));
      break;
    }
    if (a.by_ticket) return FLS_EHIP;
    a.look_limit = kLookLimit;
    a.by_ticket = true;  // workgroups did not start in the order of their numbers
  }
  fls_stats st;
  BlobInfo info;
  if (parse_header(hdr, &st, &info) != FLS_OK) return FLS_EHIP;  // our own kernels wrote it
  if (st.bytes_total > out_capacity) {
    if (stats_host) *stats_host = st;
    return FLS_ECAPACITY;
  }
  if (stats_host) *stats_host = st;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (g_blobs.size() >= kMaxRememberedBlobs) g_blobs.clear();
    g_blobs[out_dev] = info;
  }
  return FLS_OK;
}

int fls_compress(const void* W_dev, int64_t M, int64_t K, void* out_dev, size_t out_capacity, int order_policy,
                 fls_stats* stats_host, fls_stream_t stream) {
  return compress_impl(W_dev, M, K, out_dev, out_capacity, order_policy, FLS_FORMAT_VERSION, stats_host, stream);
}

int fls_compress_bound_v2(int64_t M, int64_t K, size_t* bytes_host) {
  if (!bytes_host || !shape_ok(M, K)) return FLS_EINVAL;
  const uint64_t tiles = num_tiles(M, K);
  *bytes_host = (size_t)(FLS_HEADER_BYTES + 4 * n_off_of(tiles) + 3 * tiles * (uint64_t)(FLS_TILE_M * FLS_TILE_K));
  return FLS_OK;
}

int fls_compress_v2(const void* W_dev, int64_t M, int64_t K, void* out_dev, size_t out_capacity, fls_stats* stats_host,
                    fls_stream_t stream) {
  return compress_impl(W_dev, M, K, out_dev, out_capacity, FLS_ORDER_LOCATION, FLS_FORMAT_VERSION_2, stats_host, stream);
}

size_t fls_workspace_bytes(int64_t M, int64_t K, int64_t N) {
  if (!shape_ok(M, K) || N < 1 || N > FLS_MAX_N) return 0;
  size_t total;
  workspace_layout(K, N, &total, nullptr);
  return total;
}

int fls_set_workspace(void* ws_dev, size_t bytes, fls_stream_t stream) {
  if (!ws_dev && bytes != 0) return FLS_EINVAL;
  if (!aligned16(ws_dev) || bytes % 16 != 0) return FLS_EALIGN;
  if (bytes && fls::launch_fill_zero(ws_dev, bytes, (hipStream_t)stream) != hipSuccess) return FLS_EHIP;
  std::lock_guard<std::mutex> lk(g_mu);
  g_ws = ws_dev;
  g_ws_bytes = bytes;
  return FLS_OK;
}

int fls_check_workspace(fls_stream_t stream) {
  void* ws;
  unsigned char* st = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    int dev = 0;
    if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices) st = g_scratch_ptr[dev];
    if (!st && (!g_ws || g_ws_bytes < kCounterAreaBytes)) return FLS_EWORKSPACE;
    ws = g_ws && g_ws_bytes >= kCounterAreaBytes ? g_ws : nullptr;
  }
  hipStream_t s = (hipStream_t)stream;
  uint32_t word = 0;
  if (st) {  // the scratch of fls_spmm_noalloc, if this device has used it
    if (hipMemcpyAsync(&word, (const uint32_t*)st + fls::kErrorWord, sizeof(word), hipMemcpyDeviceToHost, s) != hipSuccess)
      return FLS_EHIP;
    if (hipStreamSynchronize(s) != hipSuccess) return FLS_EHIP;
    if (word != 0) {
      if (fls::launch_fill_zero(st, kScratchControlBytes, s) != hipSuccess) return FLS_EHIP;
      return FLS_EHANDOVER;
    }
    if (!ws) return FLS_OK;
  }
  if (hipMemcpyAsync(&word, (const uint32_t*)ws + fls::kErrorWord, sizeof(word), hipMemcpyDeviceToHost, s) != hipSuccess)
    return FLS_EHIP;
  if (hipStreamSynchronize(s) != hipSuccess) return FLS_EHIP;
  if (word == 0) return FLS_OK;
  // flags of the launch that gave up may have stayed up
  if (fls::launch_fill_zero(ws, kCounterAreaBytes, s) != hipSuccess) return FLS_EHIP;
  return FLS_EHANDOVER;
}

void fls_forget(const void* Wc_dev) {
  std::lock_guard<std::mutex> lk(g_mu);
  if (Wc_dev) g_blobs.erase(Wc_dev);
  else g_blobs.clear();
}

int fls_spmm(const void* Wc_dev, const void* X_dev, void* C_dev, int64_t M, int64_t K, int64_t N,
             fls_stream_t stream) {
  int rc = check_mm_args(Wc_dev, X_dev, C_dev, M, K, N);
  if (rc != FLS_OK) return rc;
  size_t need, xpack_offset;
  workspace_layout(K, N, &need, &xpack_offset);
  void* ws;
  BlobInfo info;
  bool known;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_ws || g_ws_bytes < need) return FLS_EWORKSPACE;
    ws = g_ws;
    auto it = g_blobs.find(Wc_dev);
    known = it != g_blobs.end();
    if (known) info = it->second;
  }
  if (!known || info.M != (uint64_t)M || info.K != (uint64_t)K) {
    // unknown address, or the memory now holds another blob than the one remembered: read the header
    // on the call's stream: the blob may have been put there by work still queued on it
    unsigned char hdr[FLS_HEADER_BYTES];
    if (hipMemcpyAsync(hdr, Wc_dev, FLS_HEADER_BYTES, hipMemcpyDeviceToHost, (hipStream_t)stream) != hipSuccess) return FLS_EHIP;
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return FLS_EHIP;
    rc = parse_header(hdr, nullptr, &info);
    std::lock_guard<std::mutex> lk(g_mu);
    if (rc != FLS_OK) {
      g_blobs.erase(Wc_dev);
      return rc;
    }
    if (g_blobs.size() >= kMaxRememberedBlobs) g_blobs.clear();
    g_blobs[Wc_dev] = info;
  }
  if (info.M != (uint64_t)M || info.K != (uint64_t)K) return FLS_EFORMAT;
  const int cus = num_cus();
  if (cus <= 0) return FLS_EHIP;
  fls::SpmmLaunch a;
  a.offs = (const uint32_t*)((const unsigned char*)Wc_dev + FLS_HEADER_BYTES);
  a.words = a.offs + info.n_off;
  a.X = (const _Float16*)X_dev;
  a.C = (_Float16*)C_dev;
  a.flags = (uint32_t*)ws;
  a.parts = (float*)((unsigned char*)ws + kCounterAreaBytes);
  a.xpack = (_Float16*)((unsigned char*)ws + xpack_offset);
  a.M = (uint32_t)M;
  a.K = (uint32_t)K;
  a.N = (uint32_t)N;
  a.max_tile_words = info.max_tile_words;
  a.version = info.version;
  a.num_cus = cus;
  a.wide32 = true;
  a.raised = 1u;
  return fls::launch_spmm(a, (hipStream_t)stream) == hipSuccess ? FLS_OK : FLS_EHIP;
}

// Do the caller's statistics describe a blob of this shape?  (They stand in for the header read-back of fls_spmm.)
static bool stats_match(const fls_stats* st, int64_t M, int64_t K) {
  return (st->format_version == FLS_FORMAT_VERSION || st->format_version == FLS_FORMAT_VERSION_2) && st->tile_m == FLS_TILE_M &&
         st->tile_k == FLS_TILE_K && st->M == (uint64_t)M && st->K == (uint64_t)K && st->num_tiles == num_tiles(M, K) &&
         st->max_tile_words <= FLS_TILE_M * FLS_TILE_K && st->bytes_offsets == 4 * n_off_of(num_tiles(M, K));
}

int fls_spmm_stats(const void* Wc_dev, const fls_stats* stats_host, const void* X_dev, void* C_dev, int64_t M, int64_t K,
                   int64_t N, fls_stream_t stream) {
  if (!stats_host) return FLS_EINVAL;
  int rc = check_mm_args(Wc_dev, X_dev, C_dev, M, K, N);
  if (rc != FLS_OK) return rc;
  if (!stats_match(stats_host, M, K)) return FLS_EFORMAT;
  size_t need, xpack_offset;
  workspace_layout(K, N, &need, &xpack_offset);
  void* ws;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_ws || g_ws_bytes < need) return FLS_EWORKSPACE;
    ws = g_ws;
  }
  const int cus = num_cus();
  if (cus <= 0) return FLS_EHIP;
  fls::SpmmLaunch a;
  a.offs = (const uint32_t*)((const unsigned char*)Wc_dev + FLS_HEADER_BYTES);
  a.words = a.offs + n_off_of(num_tiles(M, K));
  a.X = (const _Float16*)X_dev;
  a.C = (_Float16*)C_dev;
  a.flags = (uint32_t*)ws;
  a.parts = (float*)((unsigned char*)ws + kCounterAreaBytes);
  a.xpack = (_Float16*)((unsigned char*)ws + xpack_offset);
  a.M = (uint32_t)M;
  a.K = (uint32_t)K;
  a.N = (uint32_t)N;
  a.max_tile_words = (uint32_t)stats_host->max_tile_words;
  a.version = stats_host->format_version;
  a.num_cus = cus;
  a.wide32 = true;
  a.raised = 1u;
  return fls::launch_spmm(a, (hipStream_t)stream) == hipSuccess ? FLS_OK : FLS_EHIP;
}

int fls_spmm_noalloc(const void* Wc_dev, const fls_stats* stats_host, const void* X_dev, void* C_dev, int64_t M,
                     int64_t K, int64_t N, fls_stream_t stream) {
  if (!stats_host) return FLS_EINVAL;
  int rc = check_mm_args(Wc_dev, X_dev, C_dev, M, K, N);
  if (rc != FLS_OK) return rc;
  if (N > FLS_NOALLOC_MAX_N) return FLS_ESCRATCH;  // partial sums of wider calls do not fit the static array
  // the caller's stats stand in for the header read-back of fls_spmm: nothing is copied, nothing is waited for
  if (!stats_match(stats_host, M, K)) return FLS_EFORMAT;
  unsigned char* ptr = scratch_on_current_device(&rc);
  if (!ptr) return rc;
  const int cus = num_cus();
  if (cus <= 0) return FLS_EHIP;
  hipStream_t s = (hipStream_t)stream;
  // Every call leaves its flags lowered, unless it gave up: the flag it no longer waited for stays up.  A call's flags bear its number, so a
  // later call does not take one for its own.  A recorded call bears the same number in every replay, so it lowers all flags before its kernel (not the
  // error word: fls_check_workspace shall hear of a replay that gave up).
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  const bool asked = hipStreamIsCapturing(s, &capture) == hipSuccess;
  if (!asked) (void)hipGetLastError();
  if ((!asked || capture != hipStreamCaptureStatusNone) && fls::launch_lower_flags((uint32_t*)ptr, s) != hipSuccess) return FLS_EHIP;
  uint32_t number;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    number = ++g_scratch_calls;
    if (number == 0) number = ++g_scratch_calls;
  }
  fls::SpmmLaunch a;
  a.offs = (const uint32_t*)((const unsigned char*)Wc_dev + FLS_HEADER_BYTES);
  a.words = a.offs + n_off_of(num_tiles(M, K));
  a.X = (const _Float16*)X_dev;
  a.C = (_Float16*)C_dev;
  a.flags = (uint32_t*)ptr;
  a.parts = (float*)(ptr + kScratchControlBytes);
  a.xpack = nullptr;  // only calls of more than 32 columns repack X
  a.M = (uint32_t)M;
  a.K = (uint32_t)K;
  a.N = (uint32_t)N;
  a.max_tile_words = (uint32_t)stats_host->max_tile_words;
  a.version = stats_host->format_version;
  a.num_cus = cus;
  a.raised = number;
  a.wide32 = false;  // the static array has the narrow kernel's partial sums only
  return fls::launch_spmm(a, s) == hipSuccess ? FLS_OK : FLS_EHIP;
}

int fls_dense_gemm(const void* W_dev, const void* X_dev, void* C_dev, int64_t M, int64_t K, int64_t N,
                   fls_stream_t stream) {
  int rc = check_mm_args(W_dev, X_dev, C_dev, M, K, N);
  if (rc != FLS_OK) return rc;
  size_t need, xpack_offset;
  workspace_layout(K, N, &need, &xpack_offset);
  void* ws;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_ws || g_ws_bytes < need) return FLS_EWORKSPACE;
    ws = g_ws;
  }
  const int cus = num_cus();
  if (cus <= 0) return FLS_EHIP;
  fls::DenseLaunch a;
  a.W = (const _Float16*)W_dev;
  a.X = (const _Float16*)X_dev;
  a.C = (_Float16*)C_dev;
  a.flags = (uint32_t*)ws;
  a.parts = (float*)((unsigned char*)ws + kCounterAreaBytes);
  a.xpack = (_Float16*)((unsigned char*)ws + xpack_offset);
  a.M = (uint32_t)M;
  a.K = (uint32_t)K;
  a.N = (uint32_t)N;
  a.num_cus = cus;
  return fls::launch_dense(a, (hipStream_t)stream) == hipSuccess ? FLS_OK : FLS_EHIP;
}

void fls_internal_spmm_plan(uint32_t max_tile_words, uint32_t version, uint32_t M, uint32_t K, uint32_t N, int cus, int wide32,
                            uint32_t* out) {
  const fls::SpmmPlan plan = fls::spmm_plan(max_tile_words, version, M / FLS_TILE_M, K / FLS_TILE_K, N, cus, wide32 != 0);
  out[0] = (uint32_t)plan.pass;
  out[1] = plan.share;
  out[2] = plan.rounds;
  out[3] = plan.slices;
}

void fls_internal_dense_plan(uint32_t M, uint32_t K, uint32_t N, int cus, uint32_t* out) {
  out[0] = fls::dense_col_groups(M, K, N, cus);
  out[1] = fls::wide_slices(M / FLS_TILE_M, out[0], (K + 63u) / 64u, cus);
}

void fls_internal_shares(uint32_t M, uint32_t K, int cus, float tile_us, int wide, uint32_t* out) {
  const fls::Shares s = fls::pick_shares(M / FLS_TILE_M, K / FLS_TILE_K, cus, tile_us, wide != 0);
  out[0] = s.P;
  out[1] = s.unit;
  out[2] = s.grid;
}

uint32_t fls_internal_divide(uint32_t n, uint32_t d) { return fls::divide(n, fls::divisor(d)); }

// The control words of fls_spmm_noalloc on the current device, the partial sums behind them, and the number of the last call.  As below.
int fls_internal_noalloc_scratch(void** control, void** parts, uint32_t* number) {
  int rc = FLS_OK;
  unsigned char* ptr = scratch_on_current_device(&rc);
  if (!ptr) return rc;
  *control = ptr;
  *parts = ptr + kScratchControlBytes;
  std::lock_guard<std::mutex> lk(g_mu);
  *number = g_scratch_calls;
  return FLS_OK;
}

// fls_compress (version 1 or 2) with the looks after which its kernel gives up and the order of chunks that it starts with; runs_host gets the
// number of kernel runs by number and by ticket.  With one look it gives up at the first word that another workgroup has not published
// yet, and is run again by ticket.  For tests, not part of the C ABI.
int fls_internal_compress(const void* W_dev, int64_t M, int64_t K, void* out_dev, size_t out_capacity, uint32_t version, uint32_t look_limit,
                          int by_ticket, uint32_t* runs_host, fls_stats* stats_host, fls_stream_t stream) {
  runs_host[0] = runs_host[1] = 0;
  return compress_impl(W_dev, M, K, out_dev, out_capacity, FLS_ORDER_LOCATION, version, stats_host, stream, look_limit, by_ticket != 0, runs_host);
}

const char* fls_strerror(int code) {
  switch (code) {
    case FLS_OK: return "ok";
    case FLS_EINVAL: return "invalid argument (null pointer, shape not a multiple of the tile, N out of range, or policy)";
    case FLS_EALIGN: return "device pointer or size not 16-byte aligned";
    case FLS_ECAPACITY: return "output buffer too small";
    case FLS_EFORMAT: return "compressed blob header is malformed or does not match M, K";
    case FLS_EWORKSPACE: return "workspace missing or too small (see fls_workspace_bytes / fls_set_workspace)";
    case FLS_EHIP: return "a HIP runtime call failed";
    case FLS_ESCRATCH: return "the call needs more scratch than the library's static array holds (fls_spmm_noalloc: N <= 32)";
    case FLS_EHANDOVER: return "a kernel gave up waiting for another workgroup's partial sum; results since the last check are not to be trusted";
    default: return "unknown error code";
  }
}

}  // extern "C"
