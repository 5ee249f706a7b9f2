// fls_compress: dense masked W -> Tiled-CSL blob on the GPU (the paper's offline weight
// reformatting step, Sec. 5; format Sec. 4.3.1-4.3.2; tile walk of Alg. 3), both format versions.
//
// All integer work on fp16 bit patterns (no value passes through a float op).  W is read from memory
// once: a workgroup takes a chunk of 16 consecutive tiles, holds it in registers, counts it, learns
// where its words start from the chunks before it while they are still at work (a scan by look-back over
// published chunk sums), and writes the words.  Two kernels:
//   emit   : everything but the index; leaves the chunk's running sum and its tiles' counts in the
//            place of the chunk's own TileOffsets entries
//   finish : turns those into TileOffsets, fills the guard entries and writes the header
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

// Where chunk q's state stands until the finish kernel runs: in words 16 q ... 16 q + 9 of TileOffsets (n_off
// is a multiple of 16 and at least T + 4, so the last, partly empty chunk has room too).
//   words 0, 1  running sum of words in bits 0 - 31, the chunk's stored elements in bits 32 - 48, kState* in bits 62 - 63
//   words 2 - 9 entries of its 16 tiles, 16 bits each
constexpr uint64_t kStateSum = 1ull << 62;     // the sum is the chunk's own
constexpr uint64_t kStatePrefix = 2ull << 62;  // the sum is that of all chunks up to and including this one
static_assert(kChunkTiles == 16, "the state of a chunk stands in the place of its 16 offsets");

constexpr int kHeaderTicket = 7;   // header word: next chunk to be taken (0 again in a finished blob)
constexpr int kHeaderGaveUp = 15;  // header word (upper half of total_words): 1 if a look-back gave up

struct CompressParams {
  const uint16_t* W;
  unsigned char* out;
  uint64_t capacity_words;  // words that fit behind TileOffsets
  uint32_t M, K, KT, T, n_off, policy;
};

__device__ __forceinline__ uint32_t* offs_of(const CompressParams& p) { return (uint32_t*)(p.out + 64); }
__device__ __forceinline__ uint32_t* words_of(const CompressParams& p) { return (uint32_t*)(p.out + 64 + 4 * (size_t)p.n_off); }
__device__ __forceinline__ uint64_t* state_of(const CompressParams& p, uint32_t q) { return (uint64_t*)(p.out + 64 + (size_t)q * 64); }

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

__device__ __forceinline__ uint64_t wave_sum64(uint64_t v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
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

// Copies the staged part of the run to the blob; dst = where the words of entry `base` go.
template <int FMT>
__device__ __forceinline__ void flush_stage(const TileCells& t, const unsigned char* stage, uint32_t base, uint32_t* dst, int lane) {
  const uint32_t left = t.entries - base, n = left < kStageEntries ? left : kStageEntries;
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
  constexpr uint32_t kLookLimit = 1u << 22;
  uint32_t sum = 0, looks = 0;
  for (uint32_t top = q; top > 0;) {
    uint64_t st = kStatePrefix;  // before the first chunk: nothing
    if ((uint32_t)lane < top)
      st = __hip_atomic_load(state_of(p, top - 1u - (uint32_t)lane), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t prefix = __builtin_amdgcn_ballot_w64((st & kStatePrefix) != 0);
    const uint64_t missing = __builtin_amdgcn_ballot_w64((st >> 62) == 0);
    const int end = prefix ? __builtin_ctzll(prefix) : 63;  // last lane that counts
    if (missing & (~0ull >> (63 - end))) {
      // chunks are taken in order, so every chunk before this one is being worked on and the wait ends; bounded all the same
      if (++looks == kLookLimit) {
        if (lane == 0) __hip_atomic_store((uint32_t*)p.out + kHeaderGaveUp, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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

// Bound by memory, at 0.85 of a copy's rate: 28672 x 7168 at 80 % (411 MB in, 164 MB out) 123 us, 12288 x 12288 at 90 % in version 2
// (302 in, 45 out) 85 us.  The walk of a lane over 64 consecutive locations takes a third of the vector instructions that one over eight
// cells strewn over the tile took, with a prefix sum, a search for the element before and a loop for bridges per cell: the whole call 165.7 ->
// 157.1 us in version 1 and 162.5 -> 118.1 us in version 2, whose vector ALUs were 72 % busy (1509 instructions a tile).  The same work as count, scan
// and emit kernels that each read W (or its counts) again: 491 and 744 us a call.  Sixteen tiles to a chunk keep the look-back and the ticket rare (one of
// each per 128 KB of W); eight waves with two tiles each leave room for two workgroups on a CU, one loading while the other writes.
template <int FMT>
__global__ __launch_bounds__(kChunkWaves * 64, 4) void compress_emit_kernel(CompressParams p) {
  __shared__ __align__(16) unsigned char stages[kChunkWaves][kTileBytes];
  __shared__ uint32_t entries_of[kChunkTiles];
  __shared__ uint32_t stored_of[kChunkWaves];
  __shared__ uint32_t ticket, chunk_base;
  const int lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Chunks are numbered in the order in which workgroups start, not by workgroup id: whatever the order in which
  // the chip starts them, a workgroup only waits for others that run already.
  if (threadIdx.x == 0) ticket = atomicAdd((uint32_t*)p.out + kHeaderTicket, 1u);
  __syncthreads();
  const uint32_t q = __builtin_amdgcn_readfirstlane(ticket);
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

  // the chunk's sum goes out first, its place is looked up after the first tile has been compacted
  uint32_t words = 0, chunk_words = 0, nz = 0;
  if (wave == 0) {
    const uint32_t mine = lane < kChunkTiles ? entries_of[lane] : 0u;
    words = run_words<FMT>(mine);
    chunk_words = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(words), 63);
    nz = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(lane < kChunkWaves ? stored_of[lane] : 0u), 63);
    if (lane == 0)
      __hip_atomic_store(state_of(p, q), (q == 0 ? kStatePrefix : kStateSum) | (uint64_t)nz << 32 | chunk_words, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t next = (uint32_t)__shfl_down((int)mine, 1, 64);
    if (lane < kChunkTiles && (lane & 1) == 0) offs_of(p)[(size_t)q * kChunkTiles + 2 + lane / 2] = mine | next << 16;
  }
  if (t[0].entries <= kStageEntries) stage_entries<FMT, true>(t[0], stage, 0, lane);
  if (wave == 0) {
    const uint32_t before = look_back(p, q, lane);
    if (lane == 0) {
      if (q != 0)
        __hip_atomic_store(state_of(p, q), kStatePrefix | (uint64_t)nz << 32 | (uint64_t)(before + chunk_words), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      chunk_base = before;
    }
  }
  __syncthreads();

  uint32_t begin = chunk_base;
  for (uint32_t j = 0; j < wave * kTilesPerWave; ++j) begin += run_words<FMT>(entries_of[j]);
#pragma unroll
  for (int a = 0; a < kTilesPerWave; ++a) {
    const uint32_t n = t[a].entries, end = begin + run_words<FMT>(n);
    uint32_t* dst = words_of(p) + begin;
    const bool fits = (uint64_t)begin + (end - begin) <= p.capacity_words;  // (a buffer that turns out too small gets the tiles that fit)
    if (n <= kStageEntries) {
      if (a > 0) stage_entries<FMT, true>(t[a], stage, 0, lane);
      lds_order();
      if (fits) flush_stage<FMT>(t[a], stage, 0, dst, lane);
    } else {
      for (uint32_t base = 0; base < n; base += kStageEntries) {
        stage_entries<FMT, false>(t[a], stage, base, lane);
        lds_order();
        if (fits) flush_stage<FMT>(t[a], stage, base, dst + run_words<FMT>(base), lane);
        lds_order();
      }
    }
    lds_order();
    begin = end;
  }
}

// A thread per chunk: its state -> its TileOffsets (nothing of another chunk's is read).
template <int FMT>
__global__ __launch_bounds__(256) void compress_finish_kernel(CompressParams p) {
  const uint32_t q = blockIdx.x * 256 + threadIdx.x, chunks = (p.T + kChunkTiles - 1) / kChunkTiles;
  uint32_t* h = (uint32_t*)p.out;
  uint64_t stored = 0;
  uint32_t longest = 0;
  if (q < chunks) {
    u32x4* cell = (u32x4*)(offs_of(p) + (size_t)q * kChunkTiles);
    u32x4 in[3], o[4];
#pragma unroll
    for (int i = 0; i < 3; ++i) in[i] = cell[i];
    const uint64_t st = (uint64_t)in[0][1] << 32 | in[0][0];
    stored = (st >> 32) & 0x1ffffu;
    uint32_t w[kChunkTiles], sum = 0;
#pragma unroll
    for (int j = 0; j < kChunkTiles; ++j) {
      const uint32_t pair = in[(2 + j / 2) / 4][(2 + j / 2) % 4];
      w[j] = run_words<FMT>((j & 1) ? pair >> 16 : pair & 0xffffu);
      sum += w[j];
      longest = w[j] > longest ? w[j] : longest;
    }
    uint32_t run = (uint32_t)st - sum;
#pragma unroll
    for (int j = 0; j < kChunkTiles; ++j) {
      o[j / 4][j % 4] = run;  // the tiles past the end of a last, partly empty chunk have no words: their entries are the total
      run += w[j];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) cell[i] = o[i];
    if (q + 1 == chunks) {
      for (uint32_t i = chunks * kChunkTiles; i < p.n_off; ++i) offs_of(p)[i] = run;
      h[0] = FMT == 2 ? kMagic2 : kMagic;
      h[1] = FMT;
      h[2] = kTileM;
      h[3] = kTileK;
      h[4] = kPad;
      h[5] = p.policy;
      h[kHeaderTicket] = 0u;
      unsigned long long* d = (unsigned long long*)(p.out + 32);
      d[0] = p.M;
      d[1] = p.K;
      h[kHeaderTotalWords] = run;
    }
  }
  stored = wave_sum64(stored);
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const uint32_t v = (uint32_t)__shfl_xor((int)longest, d, 64);
    longest = v > longest ? v : longest;
  }
  if ((threadIdx.x & 63) == 0) {
    atomicAdd((unsigned long long*)(p.out + 48), (unsigned long long)stored);
    atomicMax(h + kHeaderMaxTileWords, longest);
  }
}

__global__ void fill_zero_kernel(u32x4* p, size_t n16) {
  const u32x4 z = {0u, 0u, 0u, 0u};
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x) p[i] = z;
}

hipError_t launch_fill_zero(void* ptr, size_t bytes, hipStream_t stream) {
  const size_t n16 = bytes / 16;
  if (n16 == 0) return hipSuccess;
  size_t blocks = (n16 + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, (u32x4*)ptr, n16);
  return hipGetLastError();
}

template <int FMT>
static hipError_t launch_compress_fmt(const CompressParams& p, hipStream_t stream) {
  const uint32_t chunks = (p.T + kChunkTiles - 1) / kChunkTiles;
  // states and header start at zero
  hipError_t e = launch_fill_zero(p.out, 64 + 4 * (size_t)p.n_off, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((compress_emit_kernel<FMT>), dim3(chunks), dim3(kChunkWaves * 64), 0, stream, p);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL((compress_finish_kernel<FMT>), dim3((chunks + 255) / 256), dim3(256), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_compress(const CompressLaunch& a, hipStream_t stream) {
  CompressParams p;
  p.W = a.W;
  p.out = a.out;
  p.M = a.M;
  p.K = a.K;
  p.KT = a.K / kTileK;
  p.T = (a.M / kTileM) * p.KT;
  p.n_off = (p.T + 4 + 15) / 16 * 16;
  p.policy = a.policy;
  p.capacity_words = (a.capacity - (64 + 4 * (size_t)p.n_off)) / 4;
  return a.version == 2 ? launch_compress_fmt<2>(p, stream) : launch_compress_fmt<1>(p, stream);
}

}  // namespace fls
