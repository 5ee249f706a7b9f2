// fls_compress: dense masked W -> Tiled-CSL blob on the GPU (the paper's offline weight
// reformatting step, Sec. 5; format Sec. 4.3.1-4.3.2; tile walk of Alg. 3), both format versions.
//
// All integer work on fp16 bit patterns (no value passes through a float op).  One kernel that reads W from memory
// once: a workgroup takes a chunk of 16 consecutive tiles, holds it in registers, counts it, learns
// where its words start from the chunks before it while they are still at work (a scan by look-back over
// published chunk sums), and writes its TileOffsets and words.  The header's sums meet in the scratch of the call; the workgroup that
// adds the last chunk's writes the header, to the blob and to host memory that the caller waits for anyway.
// Format version 1: an entry is a stored element, one 32-bit word (value, location), runs padded to a
// multiple of four.  Format version 2, three bytes per entry: a tile's entries, in ascending location, go in
// groups of four that take three words - two of values, one with the first entry's location in
// 12 bits and the other three as 6-bit distances from the entry before.  An entry is a stored
// element, a bridge (value 0) every 63 locations where the next stored element lies more than 63
// behind the entry before it, or padding (value 0, distance 1) up to a multiple of four.
#include "fls_device.h"
#include "fls_launch.h"

namespace fls {

constexpr uint32_t kMagic = 0x31534C46u;   // "FLS1"
constexpr uint32_t kMagic2 = 0x32534C46u;  // "FLS2"
constexpr uint32_t kPad = 4;               // words a run is padded to (version 1), entries per group (version 2)
constexpr uint32_t kReach2 = 63;           // largest distance a 6-bit field holds

constexpr int kChunkWaves = 8;
constexpr int kTilesPerWave = 2;
constexpr int kChunkTiles = kChunkWaves * kTilesPerWave;
constexpr int kCells = kTileElems / 8 / 64;  // (row, K chunk) cells of a tile that a lane holds: 8 halves each
// Entries that a wave's 8 KB of LDS stages at once, a word (value, location) each in either version; a denser tile goes
// out in two rounds.
constexpr uint32_t kStageEntries = 2048;

// A chunk's words in the scratch, with the call's number in bits 32 - 61; those of an earlier call count as missing.
//   sums:   words in bits 0 - 31, kState* in bits 62 - 63
//   counts: stored elements in bits 0 - 16, words of its longest tile in bits 17 - 29
constexpr uint64_t kStateSum = 1ull << 62;     // the sum is the chunk's own
constexpr uint64_t kStatePrefix = 2ull << 62;  // the sum is that of all chunks up to and including this one
constexpr uint64_t kStateCounts = 3ull << 62;
constexpr int kCountsLongest = 17;
static_assert(kChunkTiles == kCompressChunkTiles, "the scratch has words for every chunk of the largest matrix");

struct CompressParams {
  const uint16_t* W;
  unsigned char* out;
  CompressScratch* scratch;
  CompressHost* host;
  uint64_t capacity_words;  // words that fit behind TileOffsets
  uint32_t M, K, KT, T, n_off, policy, chunks;
  uint32_t call;            // number of the call on this scratch
  uint32_t look_limit;      // looks at a word that another workgroup publishes, before a workgroup gives up
  bool by_ticket;
};

__device__ __forceinline__ uint32_t* offs_of(const CompressParams& p) { return (uint32_t*)(p.out + 64); }
__device__ __forceinline__ uint32_t* words_of(const CompressParams& p) { return (uint32_t*)(p.out + 64 + 4 * (size_t)p.n_off); }
__device__ __forceinline__ void publish(const CompressParams& p, uint64_t* to, uint64_t kind, uint32_t value) {
  __hip_atomic_store(to, kind | (uint64_t)p.call << 32 | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t published(const uint64_t* from) { return __hip_atomic_load(from, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ bool of_call(const CompressParams& p, uint64_t word) { return ((uint32_t)(word >> 32) & 0x3fffffffu) == p.call; }

template <int FMT>
__device__ __forceinline__ uint32_t run_words(uint32_t entries) {
  return FMT == 2 ? (entries + kPad - 1) / kPad * 3u : (entries + kPad - 1) / kPad * kPad;
}

// inclusive prefix sum over the 64 lanes
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return v;
}

// A tile as a wave holds it for the walk in location order: a lane has 64 consecutive locations, from 64 * lane on (eight
// rows of one K chunk: eight cells of eight halves).  One prefix sum over the lanes then places every entry, a lane's masks of
// stored elements give its first and last one, and a gap that takes bridges only ever lies before a lane's first element.
struct TileCells {
  u32x4 v[kCells];
  uint32_t before;   // entries of the lanes before this one
  uint32_t bridges;  // (version 2) entries needed to reach the lane's first stored element,
  uint32_t prev;     // ... from this location: that of the stored element before it, 0 if there is none
  uint32_t entries;  // of the tile, padding not counted
  uint32_t last;     // (version 2) location of its last stored element
};

// Bit e of the lowest eight: element e of the cell is stored.  min(half, 1) of two halves at a time as an asm statement: of the
// same min in C++ the compiler makes a compare and a select per half and a merge.  (And __builtin_bit_cast(u16x2, v[i]), the obvious way to
// write it, counts v[0] four times: given an element of a vector clang reads the vector's first one, whatever i, in host code and
// without optimisation too - clang 22 of ROCm 7.2.  A scalar copy of the element casts right; nothing here casts an element of a vector.)
__device__ __forceinline__ uint32_t cell_mask(const u32x4& v) {
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t one;
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(one) : "v"(v[i]), "v"(0x00010001u));
    m |= one << (2 * i);  // even halves in bits 0, 2, 4, 6, odd ones in bits 16, 18, 20, 22
  }
  return m | m >> 15;
}

// Masks of a lane's stored elements: bit 8 i + e of the two words together is element e of cell i.
__device__ __forceinline__ void tile_masks(const TileCells& t, uint32_t& lo, uint32_t& hi) {
  uint32_t w[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    // byte 0 of the second operand, then byte 0 of the first; then the two pairs
    const uint32_t a = __builtin_amdgcn_perm(cell_mask(t.v[4 * h + 1]), cell_mask(t.v[4 * h]), 0x0c0c0400u);
    const uint32_t b = __builtin_amdgcn_perm(cell_mask(t.v[4 * h + 3]), cell_mask(t.v[4 * h + 2]), 0x04000c0cu);
    w[h] = a | b;
  }
  lo = w[0];
  hi = w[1];
}

// Counts a lane's entries of the tile; `stored` = its stored elements.
template <int FMT>
__device__ __forceinline__ uint32_t count_lane(TileCells& t, uint32_t& stored, int lane) {
  uint32_t lo, hi;
  tile_masks(t, lo, hi);
  stored = (uint32_t)__popc(lo) + (uint32_t)__popc(hi);
  t.bridges = t.prev = t.last = 0;
  if constexpr (FMT == 2) {
    const bool any = (lo | hi) != 0u;
    const uint32_t loc0 = 64u * (uint32_t)lane;
    const uint32_t first = loc0 + (lo ? (uint32_t)__builtin_ctz(lo) : 32u + (uint32_t)__builtin_ctz(hi | 0x80000000u));
    const uint32_t last = loc0 + (hi ? 63u - (uint32_t)__builtin_clz(hi) : 31u - (uint32_t)__builtin_clz(lo | 1u));
    const uint64_t have = __builtin_amdgcn_ballot_w64(any);
    const uint64_t below = have & ((1ull << lane) - 1ull);
    const uint32_t of_lane = (uint32_t)__builtin_amdgcn_ds_bpermute((below ? 63 - __builtin_clzll(below) : 0) * 4, (int)last);
    t.prev = below ? of_lane : 0u;
    t.bridges = any && first > t.prev ? (first - t.prev - 1u) / kReach2 : 0u;
    if (have) t.last = (uint32_t)__builtin_amdgcn_readlane((int)last, 63 - __builtin_clzll(have));
  }
  return stored + t.bridges;
}

// A wave's LDS operations execute in order; this keeps the compiler from moving them.
__device__ __forceinline__ void lds_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// Puts entries [base, base + kStageEntries) of the tile into the wave's stage.  ALL: they are all the tile has.  Per element a
// compare that switches off the lanes whose element is zero, the step to the lane's next word, and the store, as an asm
// statement: the compiler puts a branch around such a store, which costs more than the store, and keeps the words of a tile
// for the rounds of a dense one.
template <int FMT, bool ALL>
__device__ __forceinline__ void stage_entries(TileCells& t, unsigned char* stage, uint32_t base, int lane) {
  uint32_t* words = (uint32_t*)stage;
  uint32_t slot = t.before - base;
  if constexpr (FMT == 2)
    for (uint32_t b = t.bridges, loc = t.prev; b > 0; --b, ++slot) {
      loc += kReach2;
      if (ALL || slot < kStageEntries) words[slot] = loc;
    }
  const uint32_t stage_at = (uint32_t)(uintptr_t)stage;  // LDS addresses are the low 32 bits
  uint32_t at = slot * 4u - 4u, loc = 64u * (uint32_t)lane, word, to;
  if (ALL) at += stage_at;
  const uint64_t all = __builtin_amdgcn_read_exec();
#pragma unroll
  for (int s = 0; s < kCells; ++s)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (ALL)
        asm volatile(
            "v_lshl_or_b32 %2, %3, 16, %1\n\t"
            "v_add_u32 %1, 1, %1\n\t"
            "v_cmpx_ne_u16 vcc, 0, %3\n\t"
            "v_add_u32 %0, 4, %0\n\t"
            "ds_write_b32 %0, %2\n\t"
            "s_mov_b64 exec, %4\n\t"
            "v_and_or_b32 %2, %3, %5, %1\n\t"
            "v_add_u32 %1, 1, %1\n\t"
            "v_cmpx_lt_u32 vcc, %6, %3\n\t"
            "v_add_u32 %0, 4, %0\n\t"
            "ds_write_b32 %0, %2\n\t"
            "s_mov_b64 exec, %4"
            : "+&v"(at), "+&v"(loc), "=&v"(word)
            : "v"(t.v[s][i]), "s"(all), "s"(0xffff0000u), "s"(0xffffu)
            : "vcc", "memory");
      else
        asm volatile(
            "v_lshl_or_b32 %2, %4, 16, %1\n\t"
            "v_add_u32 %1, 1, %1\n\t"
            "v_cmpx_ne_u16 vcc, 0, %4\n\t"
            "v_add_u32 %0, 4, %0\n\t"
            "v_cmpx_gt_u32 vcc, %8, %0\n\t"
            "v_add_u32 %3, %9, %0\n\t"
            "ds_write_b32 %3, %2\n\t"
            "s_mov_b64 exec, %5\n\t"
            "v_and_or_b32 %2, %4, %6, %1\n\t"
            "v_add_u32 %1, 1, %1\n\t"
            "v_cmpx_lt_u32 vcc, %7, %4\n\t"
            "v_add_u32 %0, 4, %0\n\t"
            "v_cmpx_gt_u32 vcc, %8, %0\n\t"
            "v_add_u32 %3, %9, %0\n\t"
            "ds_write_b32 %3, %2\n\t"
            "s_mov_b64 exec, %5"
            : "+&v"(at), "+&v"(loc), "=&v"(word), "=&v"(to)
            : "v"(t.v[s][i]), "s"(all), "s"(0xffff0000u), "s"(0xffffu), "s"(kStageEntries * 4u), "s"(stage_at)
            : "vcc", "memory");
    }
  // padding: version 1 words of value +0 one past the tile, version 2 entries of value 0 at distance 1
  slot = t.entries + (uint32_t)lane;
  if (lane < (int)kPad && slot < (t.entries + kPad - 1) / kPad * kPad && (ALL || slot - base < kStageEntries))
    words[slot - base] = FMT == 2 ? t.last + 1u + (uint32_t)lane : (uint32_t)kTileElems;
}

// Copies n staged entries and their padding to the blob.
template <int FMT>
__device__ __forceinline__ void flush_stage(uint32_t n, const unsigned char* stage, uint32_t* dst, int lane) {
  const uint32_t groups = (n + kPad - 1) / kPad;
  for (uint32_t g = (uint32_t)lane; g < groups; g += 64) {
    if constexpr (FMT == 2) {
      const u32x4 w = ((const u32x4*)stage)[g];
      const uint32_t l0 = w[0] & 0xffffu, l1 = w[1] & 0xffffu, l2 = w[2] & 0xffffu, l3 = w[3] & 0xffffu;
      dst[g * 3] = w[0] >> 16 | (w[1] & 0xffff0000u);
      dst[g * 3 + 1] = w[2] >> 16 | (w[3] & 0xffff0000u);
      dst[g * 3 + 2] = l0 | (l1 - l0) << 12 | (l2 - l1) << 18 | (l3 - l2) << 24;
    } else {
      ((u32x4*)dst)[g] = ((const u32x4*)stage)[g];
    }
  }
}

// Words of all chunks before chunk q.  Run by one whole wave; q's own sum is published.  Each look takes the
// states of 64 chunks, nearest first, and ends at the nearest one that knows its prefix already.
__device__ __forceinline__ uint32_t look_back(const CompressParams& p, uint32_t q, int lane) {
  uint32_t sum = 0, looks = 0;
  for (uint32_t top = q; top > 0;) {
    uint64_t st = kStatePrefix | (uint64_t)p.call << 32;  // before the first chunk: nothing
    if ((uint32_t)lane < top) st = published(p.scratch->sums + (top - 1u - (uint32_t)lane));
    const bool known = of_call(p, st);
    const uint64_t prefix = __builtin_amdgcn_ballot_w64(known && (st & kStatePrefix) != 0);
    const uint64_t missing = __builtin_amdgcn_ballot_w64(!known);
    const int end = prefix ? __builtin_ctzll(prefix) : 63;  // last lane that counts
    if (missing & (~0ull >> (63 - end))) {
      if (++looks == p.look_limit) {
        if (lane == 0) p.host->gave_up = 1u;
        return sum;
      }
      __builtin_amdgcn_s_sleep(1);
      continue;
    }
    const uint32_t part = lane <= end ? (uint32_t)st : 0u;
    sum += (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(part), 63);
    if (prefix) break;
    top = top > 64u ? top - 64u : 0u;
  }
  return sum;
}

// By the last chunk's workgroup, the one that finds all others at work or done: what all chunks counted, and the header.  (All
// workgroups adding to one address took 5 % of a large call, looks at one address as much again.)
template <int FMT>
__device__ __forceinline__ void finish_header(const CompressParams& p, uint32_t total_words, uint32_t* of_wave, uint32_t wave, int lane) {
  uint32_t stored = 0, longest = 0;  // (2^16 chunks of 2^16 elements: a thread's part is at most 2^24)
  for (uint32_t c0 = threadIdx.x; c0 < p.chunks; c0 += 4u * kChunkWaves * 64) {
    uint64_t w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t c = c0 + j * (kChunkWaves * 64);
      w[j] = published(p.scratch->counts + (c < p.chunks ? c : c0));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t c = c0 + j * (kChunkWaves * 64);
      if (c >= p.chunks) continue;
      uint32_t looks = 0;
      while (!of_call(p, w[j])) {
        if (++looks == p.look_limit) {
          p.host->gave_up = 1u;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
        w[j] = published(p.scratch->counts + c);
      }
      stored += (uint32_t)w[j] & ((1u << kCountsLongest) - 1u);
      const uint32_t l = ((uint32_t)w[j] & 0x3fffffffu) >> kCountsLongest;
      longest = l > longest ? l : longest;
    }
  }
  uint64_t nnz = (uint64_t)stored;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    nnz += __shfl_xor(nnz, d, 64);
    const uint32_t l = (uint32_t)__shfl_xor((int)longest, d, 64);
    longest = l > longest ? l : longest;
  }
  if (lane == 0) {
    of_wave[3 * wave] = (uint32_t)nnz;
    of_wave[3 * wave + 1] = (uint32_t)(nnz >> 32);
    of_wave[3 * wave + 2] = longest;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  nnz = 0;
  for (int i = 0; i < kChunkWaves; ++i) {
    nnz += (uint64_t)of_wave[3 * i + 1] << 32 | of_wave[3 * i];
    longest = of_wave[3 * i + 2] > longest ? of_wave[3 * i + 2] : longest;
  }
  const uint32_t h[kHeaderWords] = {FMT == 2 ? kMagic2 : kMagic, FMT, (uint32_t)kTileM, (uint32_t)kTileK, kPad, p.policy, longest, 0u,
                                    p.M, 0u, p.K, 0u, (uint32_t)nnz, (uint32_t)(nnz >> 32), total_words, 0u};
#pragma unroll
  for (int i = 0; i < kHeaderWords; ++i) {
    ((uint32_t*)p.out)[i] = h[i];
    p.host->header[i] = h[i];
  }
  if (p.by_ticket) p.scratch->ticket = 0u;  // every workgroup has taken its own
}

// Near its memory bound: with the place of a chunk's words a constant, no look back, whole calls take 135 us (28672 x 7168 at 80 %: 411 MB in,
// 164 MB out) and 94 us (12288 x 12288 at 90 % in version 2: 302 and 45), some 17 us of each the host's; with the look back 145.5 and 94.5.  What it came from:
//  - three and four kernels that each read W or its counts again: 491 and 744 us;
//  - this kernel between a fill of the index, a kernel for offsets and header, and a copy of the header to the host, each lane walking eight
//    cells strewn over a tile with a prefix sum, a search for the element before and a loop for bridges per cell: 165.7 and 162.5 us, the vector ALUs
//    72 % busy in version 2 (1509 instructions a tile);
//  - a lane walking 64 consecutive locations: 157.1 and 118.1 us;
//  - one kernel and a header in host memory: 151.1 and 107.1 us;
//  - no address that all workgroups add to or look at (16 ns each, one after the other), both tiles of a wave in one run: 145.5 and 94.5 us.
// Sixteen tiles to a chunk keep the look-back rare (eight: 166 and 123 us; 256 instead of 64 chunks to a look 164 and 111); eight waves with two tiles
// each leave room for two workgroups on a CU, one loading while the other writes.
template <int FMT>
__global__ __launch_bounds__(kChunkWaves * 64, 4) void compress_kernel(CompressParams p) {
  __shared__ __align__(16) unsigned char stages[kChunkWaves][kTileBytes];
  __shared__ uint32_t entries_of[kChunkTiles];
  __shared__ uint32_t stored_of[kChunkWaves];
  __shared__ uint32_t ticket, chunk_base, total_words;
  const int lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // A workgroup waits for the chunks before its own.  By number, chunk = workgroup: the chip starts workgroups in the order of their
  // numbers, so those run or have run; but nothing promises that order, and where one waits in vain it gives up after p.look_limit looks.  By
  // ticket, chunks are numbered in the order in which workgroups start, so whatever that is, the wait ends; the host
  // takes this way only when the other gave up, because all workgroups adding to one address delays the first ones: 28672 x 7168 at 80 % 145.5 us by
  // number, 146.8 by ticket, 12288 x 12288 at 90 % in version 2 94.5 and 103.3, 22656 x 2112 at 76 % in version 2 48.2 and 56.2.
  uint32_t q = blockIdx.x;
  if (p.by_ticket) {
    if (threadIdx.x == 0) ticket = atomicAdd(&p.scratch->ticket, 1u);
    __syncthreads();
    q = __builtin_amdgcn_readfirstlane(ticket);
  }
  unsigned char* stage = stages[wave];

  // Loads: lane j takes row 16 i + (j >> 2), K chunk j & 3 - a quad reads the 64 contiguous bytes of a row of the tile.
  // The wave's tiles are neighbours in K, two to a 128 B line of W (but at a band's end): the two halves of a line are
  // asked for one after the other, in an order that the compiler is kept from changing, and the line stays in the caches in between.  (All
  // loads of a tile before the other's: 160.5 us against 157.1 for 28672 x 7168 at 80 %, 124.4 against 118.1 for 12288 x 12288 at 90 % in
  // version 2; as non-temporal ones, which fetch lines twice, a third slower.)
  TileCells t[kTilesPerWave];
  // (A tile past the last one has an empty descriptor: its loads return 0.)
  __amdgpu_buffer_rsrc_t src[kTilesPerWave];
  uint32_t at[kTilesPerWave];
#pragma unroll
  for (int a = 0; a < kTilesPerWave; ++a) {
    const uint32_t tile = q * kChunkTiles + wave * kTilesPerWave + a, live = tile < p.T ? tile : 0u;
    const uint32_t band = live / p.KT, kt = live - band * p.KT;
    src[a] = __builtin_amdgcn_make_buffer_rsrc((void*)(p.W + (size_t)band * kTileM * p.K), 0,
                                               tile < p.T ? (int)(kTileM * 2u * p.K) : 0, kBufferFlags);
    at[a] = ((lane >> 2) * p.K + kt * kTileK + (lane & 3) * 8) * 2u;
  }
#pragma unroll
  for (int i = 0; i < kCells; ++i) {
#pragma unroll
    for (int a = 0; a < kTilesPerWave; ++a) t[a].v[i] = __builtin_amdgcn_raw_buffer_load_b128(src[a], at[a], i * 32u * p.K, 0);
    __builtin_amdgcn_sched_barrier(0);  // in this order
  }
  // ... and through LDS into the order of the walk.  Cell (row, K chunk c), row bits b6 ... b0, is in slot
  // ((c, b6 b5, b2), c ^ b4 b3, b1 b0 ^ b6 b5): any 16 neighbouring lanes touch 16 different 16 B bank groups, both ways.
  uint32_t entries[kTilesPerWave], stored[kTilesPerWave];
  const uint32_t c = lane & 3, r = lane >> 2, h = (lane >> 2) & 3;  // store: K chunk, row in its 16; read: b6 b5 of the lane's rows
  const uint32_t put_at = ((c * 8 + ((r >> 2) & 1)) * 16 + (c ^ (r >> 3)) * 4 + (r & 3)) * 16;
  const uint32_t get_at = (((lane >> 4) * 8 + h * 2) * 16 + ((lane >> 4) ^ (lane & 3)) * 4) * 16;
#pragma unroll
  for (int a = 0; a < kTilesPerWave; ++a) {
#pragma unroll
    for (int i = 0; i < kCells; ++i) *(u32x4*)(stage + ((put_at ^ ((i & 1) * 128u + (i >> 1) * 16u)) + (i >> 1) * 512u)) = t[a].v[i];
    lds_order();
#pragma unroll
    for (int i = 0; i < kCells; ++i) t[a].v[i] = *(const u32x4*)(stage + get_at + (i >> 2) * 256u + (((i & 3) ^ h) * 16u));
    lds_order();
    entries[a] = count_lane<FMT>(t[a], stored[a], lane);
  }
  // both tiles in one prefix sum: a tile has at most 4096 stored elements and 65 bridges
  static_assert(kTilesPerWave == 2, "two sums of 16 bits to a word");
  const uint32_t incl = wave_inclusive_scan(entries[0] | entries[1] << 16), sums = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
  t[0].before = (incl & 0xffffu) - entries[0];
  t[1].before = (incl >> 16) - entries[1];
  t[0].entries = sums & 0xffffu;
  t[1].entries = sums >> 16;
  uint32_t wave_stored = t[0].entries + t[1].entries;
  if constexpr (FMT == 2) {
    const uint32_t bridges = t[0].bridges + t[1].bridges;
    if (__builtin_amdgcn_ballot_w64(bridges != 0u) != 0u) wave_stored -= (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(bridges), 63);
  }
  if (lane < kTilesPerWave) entries_of[wave * kTilesPerWave + lane] = lane == 0 ? t[0].entries : t[1].entries;
  if (lane == 0) stored_of[wave] = wave_stored;
  __syncthreads();

  // The chunk's sum and counts go out first; its place is looked up after the wave's tiles have been compacted, one behind the other
  // (the first of them, if they have more entries than the stage holds).
  uint32_t words = 0, incl_words = 0;
  if (wave == 0) {
    words = run_words<FMT>(lane < kChunkTiles ? entries_of[lane] : 0u);
    incl_words = wave_inclusive_scan(words);
    const uint32_t nz = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(lane < kChunkWaves ? stored_of[lane] : 0u), 63);
    uint32_t longest = words;  // of 16 lanes
#pragma unroll
    for (int d = kChunkTiles / 2; d >= 1; d >>= 1) {
      const uint32_t v = (uint32_t)__shfl_xor((int)longest, d, 64);
      longest = v > longest ? v : longest;
    }
    if (lane == 0) {
      publish(p, p.scratch->sums + q, q == 0 ? kStatePrefix : kStateSum, (uint32_t)__builtin_amdgcn_readlane((int)incl_words, 63));
      publish(p, p.scratch->counts + q, kStateCounts, nz | longest << kCountsLongest);
    }
  }
  const uint32_t padded0 = (t[0].entries + kPad - 1) / kPad * kPad, padded1 = (t[1].entries + kPad - 1) / kPad * kPad;
  const bool together = padded0 + padded1 <= kStageEntries;
  if (t[0].entries <= kStageEntries) stage_entries<FMT, true>(t[0], stage, 0, lane);
  if (together) stage_entries<FMT, true>(t[1], stage + padded0 * 4u, 0, lane);
  if (wave == 0) {
    const uint32_t before = look_back(p, q, lane), chunk_words = (uint32_t)__builtin_amdgcn_readlane((int)incl_words, 63);
    if (lane == 0) {
      if (q != 0) publish(p, p.scratch->sums + q, kStatePrefix, before + chunk_words);
      chunk_base = before;
      total_words = before + chunk_words;
    }
    // TileOffsets of the chunk's tiles; behind the last tile, up to the end (at most 16 entries past the last chunk's), the total
    const uint32_t off = q * kChunkTiles + (uint32_t)lane;
    if (lane < kChunkTiles || (q + 1 == p.chunks && off < p.n_off))
      offs_of(p)[off] = before + (lane < kChunkTiles ? incl_words - words : chunk_words);
  }
  __syncthreads();

  uint32_t begin = chunk_base;
  for (uint32_t j = 0; j < wave * kTilesPerWave; ++j) begin += run_words<FMT>(entries_of[j]);
  // (a buffer that turns out too small gets the tiles that fit)
  auto fits = [&](uint32_t words) { return (uint64_t)begin + words <= p.capacity_words; };
  const uint32_t words0 = run_words<FMT>(t[0].entries), words1 = run_words<FMT>(t[1].entries);
  if (together && fits(words0 + words1)) {
    lds_order();
    flush_stage<FMT>(padded0 + padded1, stage, words_of(p) + begin, lane);
  } else {
#pragma unroll
    for (int a = 0; a < kTilesPerWave; ++a) {
      const uint32_t n = t[a].entries;
      if (fits(run_words<FMT>(n))) {
        uint32_t* dst = words_of(p) + begin;
        for (uint32_t base = 0; base < n; base += kStageEntries) {
          lds_order();
          if (n <= kStageEntries) {
            if (a > 0) stage_entries<FMT, true>(t[a], stage, 0, lane);
          } else {
            stage_entries<FMT, false>(t[a], stage, base, lane);
          }
          lds_order();
          flush_stage<FMT>(n - base < kStageEntries ? n - base : kStageEntries, stage, dst + run_words<FMT>(base), lane);
        }
      }
      begin += run_words<FMT>(n);
    }
  }
  if (q + 1 == p.chunks) {
    __syncthreads();  // the stages are free
    finish_header<FMT>(p, total_words, (uint32_t*)stages[0], wave, lane);
  }
}

__global__ void fill_zero_kernel(u32x4* p, size_t n16) {
  const u32x4 z = {0u, 0u, 0u, 0u};
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x) p[i] = z;
}

__global__ __launch_bounds__(kMaxWorkgroups) void lower_flags_kernel(uint32_t* flags) {
#pragma unroll
  for (uint32_t i = threadIdx.x; i < kControlWords; i += kMaxWorkgroups)
    if (i != kErrorWord) flags[i] = 0u;
}

hipError_t launch_lower_flags(uint32_t* flags, hipStream_t stream) {
  hipLaunchKernelGGL(lower_flags_kernel, dim3(1), dim3(kMaxWorkgroups), 0, stream, flags);
  return hipGetLastError();
}

hipError_t launch_fill_zero(void* ptr, size_t bytes, hipStream_t stream) {
  const size_t n16 = bytes / 16;
  if (n16 == 0) return hipSuccess;
  size_t blocks = (n16 + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, (u32x4*)ptr, n16);
  return hipGetLastError();
}

hipError_t launch_compress(const CompressLaunch& a, hipStream_t stream) {
  CompressParams p;
  p.W = a.W;
  p.out = a.out;
  p.scratch = a.scratch;
  p.host = a.host;
  p.call = a.call;
  p.look_limit = a.look_limit;
  p.by_ticket = a.by_ticket;
  p.M = a.M;
  p.K = a.K;
  p.KT = a.K / kTileK;
  p.T = (a.M / kTileM) * p.KT;
  p.n_off = (p.T + 4 + 15) / 16 * 16;
  p.policy = a.policy;
  p.chunks = (p.T + kChunkTiles - 1) / kChunkTiles;
  p.capacity_words = (a.capacity - (64 + 4 * (size_t)p.n_off)) / 4;
  if (a.version == 2) hipLaunchKernelGGL((compress_kernel<2>), dim3(p.chunks), dim3(kChunkWaves * 64), 0, stream, p);
  else hipLaunchKernelGGL((compress_kernel<1>), dim3(p.chunks), dim3(kChunkWaves * 64), 0, stream, p);
  return hipGetLastError();
}

}  // namespace fls
