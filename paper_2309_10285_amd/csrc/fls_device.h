// Device-side building blocks shared by the sparse and the dense kernel: MFMA operand types,
// the split-K hand-over of partial bands.  gfx950 only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fls_launch.h"

namespace fls {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kTileM = 128;               // rows of a tile (one row band)
constexpr int kTileK = 32;                // K extent of a tile = K of one 16x16x32 MFMA
constexpr int kTileElems = kTileM * kTileK;
constexpr int kTileBytes = kTileElems * 2;  // dense fp16 tile in LDS
constexpr int kRowBlocks = kTileM / 16;     // 16-row MFMA blocks per tile

constexpr int kHeaderWords = 16;            // the blob's 64-byte header, in 32-bit words; TileOffsets follow it
constexpr int kHeaderMaxTileWords = 6;      // header word that holds the length of the longest tile
constexpr int kHeaderTotalWords = 14;       // header word that holds the number of words in NonZeros (low half of a u64)

constexpr int kAccPerBlock = kTileM * 16;   // fp32 values of one 128 x 16 column block
constexpr int kBufferFlags = 0x00020000;    // raw buffer, 32-bit data format (gfx9 descriptor word 3)
constexpr int kAuxNonTemporal = 2;          // nt: streamed once, do not keep in the caches
constexpr int kAuxCoherent = 16;            // sc1: device scope - through to memory / past the per-XCD L2

// LDS byte address a word of a tile goes to: base + 2 * location (the word's low half), in one
// instruction (v_mad_u32_u16: D = S0.u16 * S1.u16 + S2.u32).
__device__ __forceinline__ uint32_t scatter_addr(uint32_t word, uint32_t base) {
  uint32_t addr;
  asm("v_mad_u32_u16 %0, %1, 2, %2" : "=v"(addr) : "v"(word), "v"(base));
  return addr;
}

// What both kernels need to hand results over.
//
// Split-K: the band-major tile sequence [0, T) is cut evenly over the workgroups, then over the
// waves of a workgroup.  Partial results of one band meet in two steps:
//   1. inside a workgroup, in LDS (wg_reduce): waves add their accumulators to one of two band
//      slots and count their tiles; the wave that completes the workgroup's share takes the sum;
//   2. between workgroups, in HBM: that wave stores the sum to its workgroup's slot and later
//      raises the workgroup's flag; the workgroup that owns the band adds up the slots in
//      workgroup order and writes fp16 C (see "between workgroups" below).
// No floating-point atomics touch HBM.
struct OutParams {
  _Float16* C;      // column-major M x N
  float* parts;     // [workgroup][NB * 2048] fp32 partial sums in accumulator order
  uint32_t* flags;  // control words (kControlWords of them); [share] `raised` while a published partial sum waits for its band's owner
  uint32_t raised;  // a flag that is up, nonzero
  uint32_t P;       // shares
  uint32_t unit;    // ... that stay together on an XCD, `units` such groups; 0: shares are whole bands, nothing is handed over
  uint32_t units;
  uint32_t bands;
  Divisor by_P, by_KT;
  uint32_t M, N;    // N = columns of the whole problem
  uint32_t n0;      // first column of this launch's column group
  uint32_t KT;      // K tiles per band
  uint32_t T;       // tiles in total
};

// The unit of work of this workgroup when the grid is units rounded up to a multiple of eight.  Consecutive workgroup
// ids go to the chip's eight XCDs in turn, so id 8 i + x takes the i-th unit of the x-th eighth: neighbouring units
// run on one XCD, one after the other, and find in its L2 what they share.
__device__ __forceinline__ bool xcd_unit(uint32_t units, uint32_t& unit) {
  const uint32_t x = blockIdx.x & 7u;
  unit = x * units / 8u + (blockIdx.x >> 3);
  return unit < (x + 1u) * units / 8u;
}

// The 64-column passes: group of four bands, K slice and group of 64 columns of this workgroup.  The G workgroups that
// stream the same words run on one XCD, one after the other, and all but the first find them in its L2.
// `whole` (see whole_pairs of the launchers): (quad, slice) pair 8 i + x goes to XCD x with all its column groups.
// Otherwise every XCD takes an eighth of all units, slice by slice.  (Two branches, not one formula with selects: that cost 1 - 2 % of
// calls of 5 - 10 us and half a percent of longer ones.)
__device__ __forceinline__ bool wide_unit(const WideParams& p, uint32_t quads, uint32_t& quad, uint32_t& slice, uint32_t& cg) {
  if (p.whole) {
    const uint32_t i = blockIdx.x >> 3, j = divide(i, p.by_G), pair = j * 8u + (blockIdx.x & 7u);
    cg = i - j * p.G;
    quad = divide(pair, p.by_S);
    slice = pair - quad * p.S;
    return pair < quads * p.S;
  }
  uint32_t unit;
  if (!xcd_unit(quads * p.S * p.G, unit)) return false;
  const uint32_t pair = divide(unit, p.by_G);
  cg = unit - pair * p.G;
  slice = divide(pair, p.by_groups);
  quad = pair - slice * quads;
  return true;
}

// First tile of share q: all tiles cut evenly over the shares, or the bands.  (At most kMaxWorkgroups shares, fewer than 2^20 tiles.)
__device__ __forceinline__ uint32_t share_begin(const OutParams& o, uint32_t q) {
  return o.unit == 0 ? divide(q * o.bands, o.by_P) * o.KT : divide(q * o.T, o.by_P);
}

// This workgroup's share, and the end of the shares that go to the same XCD.  Consecutive workgroup ids go to the chip's
// eight XCDs in turn, so id 8 i + x takes the i-th share of the x-th eighth of the units: neighbouring shares, which hand partial
// sums of a cut band to each other, run on one XCD.  (share_grid of the launchers sizes the grid.)
__device__ __forceinline__ bool share_of_block(const OutParams& o, uint32_t& wg, uint32_t& near_end) {
  if (o.unit == 0) {  // nothing to hand over
    wg = blockIdx.x;
    near_end = 0;
    return wg < o.P;
  }
  const uint32_t x = blockIdx.x & 7u;
  wg = x * o.units / 8u * o.unit + (blockIdx.x >> 3);
  near_end = (x + 1u) * o.units / 8u * o.unit;
  return wg < near_end;
}

// The XCD this wave runs on (hardware register XCC_ID, bits 0 - 3).
__device__ __forceinline__ uint32_t my_xcd() { return __builtin_amdgcn_s_getreg(20 | (4 - 1) << 11); }

// MFMA 16x16 accumulator layout: lane l holds column (l & 15), rows 4*(l >> 4) .. +3 of its block.
// Converts a wave's 128 x (NB*16) accumulators to fp16 and stores them to column-major C.
template <int NB>
__device__ __forceinline__ void store_band(const OutParams& o, const float4v (&acc)[kRowBlocks][NB], uint32_t band,
                                           int lane) {
  const uint32_t col = lane & 15, rsub = (lane >> 4) * 4;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const uint32_t n = o.n0 + nb * 16 + col;
    if (n < o.N) {
#pragma unroll
      for (int rb = 0; rb < kRowBlocks; ++rb) {
        half4 h;
#pragma unroll
        for (int r = 0; r < 4; ++r) h[r] = (_Float16)acc[rb][nb][r];
        *(half4*)(o.C + (size_t)n * o.M + band * kTileM + rb * 16 + rsub) = h;
      }
    }
  }
}

// LDS area of the in-workgroup step: band slots and their control words.  A slot keeps a band's
// running sum as [column block][row block][lane] float4.  Consecutive bands of a workgroup's
// share alternate between two slots, so that waves already in the next band need not wait for
// the previous one to be collected.
template <int NB>
struct WgReduceLds {
  static constexpr uint32_t kSlots = 2;
  static constexpr int kParts = 4;  // a slot is added to in four parts, each under its own lock
  float4v slot[kSlots][NB * kRowBlocks * 64];
  uint32_t cnt[kSlots];           // tiles added to the slot so far
  uint32_t gen[kSlots];           // how many bands the slot has served
  uint32_t lock[kSlots][kParts];  // 1 while a wave is adding to that part of the slot
  uint32_t far;                   // 1 once a wave has stored its part of the workgroup's partial sum through to memory
};

template <int NB>
__device__ __forceinline__ void wg_reduce_init(WgReduceLds<NB>* red, int tid, int nthreads) {
  for (int i = tid; i < (int)WgReduceLds<NB>::kSlots * NB * kRowBlocks * 64; i += nthreads) (&red->slot[0][0])[i] = float4v{0.f, 0.f, 0.f, 0.f};
  if (tid == 0) red->far = 0;
  if (tid < (int)WgReduceLds<NB>::kSlots) {
    red->cnt[tid] = 0;
    red->gen[tid] = 0;
#pragma unroll
    for (int part = 0; part < WgReduceLds<NB>::kParts; ++part) red->lock[tid][part] = 0;
  }
}

// Adds a wave's accumulators for the seq-th band of its workgroup (seq counts from the
// workgroup's first band) to the band's slot.  Returns true for exactly one wave per band: the
// one whose tiles complete `expected`; the slot then holds the workgroup's sum (wg_reduce_take
// collects it).  Waves add with plain 16 B read-add-write under spin locks, one per quarter of
// the slot, all taking the quarters in the same order: waves that arrive together follow each
// other through the slot like an assembly line instead of waiting for the whole of it.  (LDS
// floating-point atomics would need no lock but run about fifty times slower per instruction
// on this chip than a plain LDS access.)
template <int NB>
__device__ __forceinline__ bool wg_reduce_add(WgReduceLds<NB>* red, const float4v (&acc)[kRowBlocks][NB], uint32_t seq,
                                              uint32_t tiles, uint32_t expected, int lane) {
  const uint32_t s = seq % WgReduceLds<NB>::kSlots, turn = seq / WgReduceLds<NB>::kSlots;
  // the slot may still serve an earlier band (only when a share spans more bands than there are slots)
  while (__hip_atomic_load(&red->gen[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != turn)
    __builtin_amdgcn_s_sleep(2);
  constexpr int kParts = WgReduceLds<NB>::kParts, kPerPart = NB * kRowBlocks / kParts;
  float4v* d = &red->slot[s][lane];
#pragma unroll
  for (int part = 0; part < kParts; ++part) {
    for (;;) {
      uint32_t got = 1;
      if (lane == 0) got = __hip_atomic_exchange(&red->lock[s][part], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (__builtin_amdgcn_readfirstlane(got) == 0) break;
      __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
#pragma unroll
    for (int e = part * kPerPart; e < (part + 1) * kPerPart; ++e) d[e * 64] += acc[e % kRowBlocks][e / kRowBlocks];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    if (lane == 0) __hip_atomic_store(&red->lock[s][part], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  // counted in after the last part: the wave that completes the count finds every part added
  uint32_t old = 0;
  if (lane == 0) old = __hip_atomic_fetch_add(&red->cnt[s], tiles, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  old = __builtin_amdgcn_readfirstlane(old);
  return old + tiles == expected;
}

// Run by the wave wg_reduce_add picked: moves the slot's sum into acc and frees the slot for band seq + 2.
template <int NB>
__device__ __forceinline__ void wg_reduce_take(WgReduceLds<NB>* red, float4v (&acc)[kRowBlocks][NB], uint32_t seq,
                                               int lane) {
  const uint32_t s = seq % WgReduceLds<NB>::kSlots, turn = seq / WgReduceLds<NB>::kSlots;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  float4v* d = &red->slot[s][lane];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int rb = 0; rb < kRowBlocks; ++rb) {
      acc[rb][nb] = d[(nb * kRowBlocks + rb) * 64];
      d[(nb * kRowBlocks + rb) * 64] = float4v{0.f, 0.f, 0.f, 0.f};
    }
  if (lane == 0) red->cnt[s] = 0;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  if (lane == 0) __hip_atomic_store(&red->gen[s], turn + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// A wave that saw a whole band by itself has nothing to reduce, but the band still takes its turn
// on the slot so that the turn count of later bands stays right.
template <int NB>
__device__ __forceinline__ void wg_reduce_skip(WgReduceLds<NB>* red, uint32_t seq, int lane) {
  const uint32_t s = seq % WgReduceLds<NB>::kSlots, turn = seq / WgReduceLds<NB>::kSlots;
  while (__hip_atomic_load(&red->gen[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != turn)
    __builtin_amdgcn_s_sleep(2);
  if (lane == 0) __hip_atomic_store(&red->gen[s], turn + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// ---- between workgroups
//
// A band that is cut between workgroups is finished by its owner: the workgroup whose share holds
// the band's first tile.  The owner's piece of the band is the last thing in its share, so its
// sum is still in registers when its run ends.  Every other workgroup that holds tiles of the
// band stores its sum to its slot when its piece ends (nothing waits for the stores) and publishes
// the slot when its own run ends, by raising its flag.  The owner then polls those flags, adds the
// slots in workgroup order and writes fp16 C.
//
// How a sum gets across depends on where the two run.  On one XCD they share an L2: a store has arrived there once
// it counts as done, and loads that miss the CU's L1 find it.  The L2 caches of different XCDs are not coherent with each
// other inside a kernel: there the contributor stores through to memory and releases at device scope before it raises its flag,
// and the owner loads at device scope after it has seen the flags - trips to memory, one after the other, when
// the kernel is about to end.  Which way a contributor takes it decides from the owner's word: a workgroup that will own a cut
// band writes the XCD it runs on there when it starts (the hardware's number, not one worked out from the workgroup's
// number: that only decides how likely the short way is), and takes it back once it has seen all flags.  An owner that has not
// started yet, or runs elsewhere, gets the long way.  Each way has its own flags, so the owner knows which one it was.
// Measured, against the long way for all: 12288 x 12288 at 80 %, N = 13 30.4 -> 27.9 us a call (0.67 of the bands cut), 48640 x 1056 at 89 %, N = 4 17.1 ->
// 14.0, 49152 x 12288 at 70 % in version 2, N = 8 96.6 -> 94.7, a 7168-wide decoder layer, N = 16 114.5 -> 110.3; with the shares of a band kept together
// 1536 x 17312 at 71 %, N = 2 17.4 -> 14.9.
//
// A workgroup publishes at most one
// partial sum per launch (only the first band of a share can begin outside it) and exactly one
// owner waits for it; the owner lowers the flag it has seen, so all flags are down again when the
// launch ends: nothing is cleared between calls, and a launch recorded in a graph can be replayed.
//
// A workgroup publishes before it polls, and only polls workgroups of higher index, so the wait
// ends as soon as those workgroups have run; the spin is bounded all the same.  How long that is: a look is a trip to the L2, some 600 clocks,
// or to memory, some 2000, and a sleep.  (A launch whose workgroups wait for room because another stream's kernel holds the chip must outlast
// that kernel, so the bound is a second or more at the shorter of the two.)
constexpr int kSpinSleep = 2;  // x 64 clocks: sums are due within a microsecond or two
constexpr uint32_t kSpinLimit = 1u << 22;
static_assert((uint64_t)kSpinLimit * (64u * kSpinSleep + 600u) >= 2400000000ull, "a second at 2.4 GHz");

// Does share [share0, share1) hold the first tile of a band that it does not hold the last tile of?
__device__ __forceinline__ bool owns_cut_band(const OutParams& o, uint32_t share0, uint32_t share1) {
  const uint32_t first = divide(share1, o.by_KT) * o.KT;  // of the band that share1 lies in
  return first != share1 && first >= share0;
}
// By one thread of a workgroup when it starts.
__device__ __forceinline__ void announce_owner(const OutParams& o, uint32_t wg, uint32_t share0, uint32_t share1) {
  if (owns_cut_band(o, share0, share1))
    __hip_atomic_store(o.flags + kOwnerXcd + wg, my_xcd() + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// XCD + 1 of the owner of `band`, 0 if it has not started: a load that the caller lets run until it needs the answer.
__device__ __forceinline__ uint32_t owner_word(const OutParams& o, uint32_t band) {
  const uint32_t first = band * o.KT;
  uint32_t q = first * o.P / o.T;
  while (q + 1 < o.P && share_begin(o, q + 1) <= first) ++q;
  return __hip_atomic_load(o.flags + kOwnerXcd + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool runs_here(uint32_t owner_word) { return __builtin_amdgcn_readfirstlane(owner_word) == my_xcd() + 1u; }

template <int NB, int AUX>
__device__ __forceinline__ void store_partial_as(const OutParams& o, const float4v (&acc)[kRowBlocks][NB], uint32_t wg,
                                                 int lane) {
  const __amdgpu_buffer_rsrc_t mine = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(o.parts + (size_t)wg * (NB * kAccPerBlock)), 0, NB * kAccPerBlock * 4, kBufferFlags);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int rb = 0; rb < kRowBlocks; ++rb)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[rb][nb]), mine,
                                             ((nb * kRowBlocks + rb) * 64 + lane) * 16, 0, AUX);
}
template <int NB>
__device__ __forceinline__ void store_partial(const OutParams& o, const float4v (&acc)[kRowBlocks][NB], uint32_t wg, bool local,
                                              int lane) {
  if (local) store_partial_as<NB, 0>(o, acc, wg, lane);
  else store_partial_as<NB, kAuxCoherent>(o, acc, wg, lane);
}

// A device-scope release in two halves, so that the time the write-back takes can pass behind
// other work: release_begin right after the stores (the L2 of this XCD starts writing back what
// it holds), release_end before the flag is raised (waits for that and for every earlier store).
// Together they are the instruction sequence of a release fence at device scope.  Waiting for the
// stores alone is not enough across XCDs: a store counts as done when the XCD's L2 has it, and the flag could
// reach memory before the data does (seen as a wrong band about once in a thousand calls).
__device__ __forceinline__ void release_begin() { asm volatile("buffer_wbl2 sc1" ::: "memory"); }
__device__ __forceinline__ void release_end() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// A flag of the short way, raised and taken down again as instructions of this chip: no scope of the memory model stands for "the
// workgroups of one XCD" (workgroup scope promises nothing beyond the workgroup, agent scope is the trip to memory that is to be saved).  What they rely on: a
// store passes through the CU's L1 and is done when the XCD's L2 has it; an atomic is executed by the L2 (sc0: it returns the old value), where a load may be
// served by the L1 for ever.
__device__ __forceinline__ void raise_local(uint32_t* flag, uint32_t raised) {
  asm volatile("global_store_dword %0, %1, off sc0" ::"v"(flag), "v"(raised) : "memory");
}
__device__ __forceinline__ bool lower_local(uint32_t* flag, uint32_t raised) {
  uint32_t old;
  const uint64_t swap = (uint64_t)raised << 32;  // the new value, 0; the one to compare with
  asm volatile("global_atomic_cmpswap %0, %1, %2, off sc0\n\ts_waitcnt vmcnt(0)" : "=&v"(old) : "v"(flag), "v"(swap) : "memory");
  return old == raised;
}

// By the wave that called store_partial, once its run is over; `begun` tells whether it has called
// release_begin behind the stores already.
__device__ __forceinline__ void publish_partial(const OutParams& o, uint32_t wg, int lane, bool local, bool begun) {
  if (local) {
    release_end();  // the stores have reached the L2
    if (lane == 0) raise_local(o.flags + kLocalFlags + wg, o.raised);
    return;
  }
  if (!begun) release_begin();
  release_end();
  if (lane == 0) __hip_atomic_store(o.flags + wg, o.raised, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// acc holds the owner's own sum for `band`; adds the other workgroups' and writes C.
template <int NB>
__device__ __forceinline__ void owner_finish(const OutParams& o, float4v (&acc)[kRowBlocks][NB], uint32_t band,
                                             uint32_t wg, uint32_t near_end, int lane) {
  const uint32_t band_hi = (band + 1) * o.KT;
  // The flags of up to 64 contributors are polled at once, one per lane: a look at a flag is a trip to
  // L2 or memory, and one after the other those trips would add up at the very end of the kernel.
  for (uint32_t base = wg + 1; base < o.P && share_begin(o, base) < band_hi; base += 64) {
    const uint32_t q = base + (uint32_t)lane;
    // workgroup q holds tiles of the band (an empty share contributes nothing)
    const bool mine = q < o.P && share_begin(o, q) < band_hi && share_begin(o, q + 1) != share_begin(o, q);
    uint32_t spins = 0;
    bool seen = !mine, local = false;
    for (;;) {
      if (!seen) {
        // (the kind of flag that the contributor's number lets expect each time, the other one now and then)
        const bool expected = q < near_end, both = (spins & 7u) == 7u;
        if (expected || both) local = lower_local(o.flags + kLocalFlags + q, o.raised);
        seen = local;
        if (!seen && (!expected || both)) seen = __hip_atomic_load(o.flags + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == o.raised;
      }
      if (__builtin_amdgcn_ballot_w64(!seen) == 0) break;
      __builtin_amdgcn_s_sleep(kSpinSleep);
      if (++spins == kSpinLimit) {  // never seen; gives up rather than hang, and says so
        if (lane == 0) __hip_atomic_store(o.flags + kErrorWord, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
    }
    // workgroup q raises one flag once per launch and nobody else looks at it: down again for the next launch
    if (mine && seen && !local) __hip_atomic_store(o.flags + q, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // The loads below are issued after the flags have been seen.  Slots filled through this XCD's L2 are read by ordinary loads: no line of
    // theirs can be in this CU's L1, which starts a launch empty and has seen no read of them since.  Loads at device scope are what pairs with the contributors'
    // release: nothing that this CU's L1 or this XCD's L2 still holds of the slots may serve them.  (An acquire fence here would invalidate
    // both caches wholesale on top of that: a microsecond at the very end of the kernel.)
    asm volatile("" ::: "memory");
    // As many loads as the registers allow are issued before the first is used: nothing is left to hide one behind.
    constexpr int kBatch = NB == 1 ? 4 : 2;  // slots in flight
    uint64_t left = __builtin_amdgcn_ballot_w64(mine);
    const uint64_t far = __builtin_amdgcn_ballot_w64(mine && !local);
    while (left != 0) {
      u32x4 v[kBatch][NB][kRowBlocks];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        // the next contributor; past the last one the descriptor is empty and reads 0
        const uint32_t i = left ? (uint32_t)__builtin_ctzll(left) : 0u;
        const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc((void*)(o.parts + (size_t)(base + i) * (NB * kAccPerBlock)), 0,
                                                                             left ? NB * kAccPerBlock * 4 : 0, kBufferFlags);
        if (left & far & (1ull << i)) {
#pragma unroll
          for (int e = 0; e < NB * kRowBlocks; ++e)
            v[j][e / kRowBlocks][e % kRowBlocks] = __builtin_amdgcn_raw_buffer_load_b128(src, (e * 64 + lane) * 16, 0, kAuxCoherent);
        } else {
#pragma unroll
          for (int e = 0; e < NB * kRowBlocks; ++e)
            v[j][e / kRowBlocks][e % kRowBlocks] = __builtin_amdgcn_raw_buffer_load_b128(src, (e * 64 + lane) * 16, 0, 0);
        }
        left &= left - 1;
      }
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int rb = 0; rb < kRowBlocks; ++rb) acc[rb][nb] += __builtin_bit_cast(float4v, v[j][nb][rb]);
    }
  }
  // all contributors have read the owner's word
  if (lane == 0) __hip_atomic_store(o.flags + kOwnerXcd + wg, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  store_band<NB>(o, acc, band, lane);
}

// What a wave carries from the tile loop to the end of its run.
struct HandoverState {
  bool publish = false;  // it stored its workgroup's partial sum and still has to publish it
  bool local = false;    // ... to the owner's L2
  bool released = false; // release_begin has been called behind those stores
  bool own = false;      // it holds the owner's sum of band own_band in its accumulators
  uint32_t own_band = 0;
};

// Hand-over of a wave's piece (tiles of one band), inside the tile loop: LDS work and, at most,
// stores that nothing waits for.  `tiles` = tiles in the piece, [share0, share1) = the
// workgroup's share.  Leaves acc cleared for the next band unless the wave became an owner.
template <int NB>
__device__ __forceinline__ void hand_over_piece(const OutParams& o, WgReduceLds<NB>* red, float4v (&acc)[kRowBlocks][NB],
                                                HandoverState& st, uint32_t band, uint32_t tiles, uint32_t share0,
                                                uint32_t share1, uint32_t wg, int lane, bool local_only,
                                                bool early_release) {
  const uint32_t seq = band - divide(share0, o.by_KT);
  if (tiles == o.KT) {
    store_band<NB>(o, acc, band, lane);  // this wave alone saw the whole band
    wg_reduce_skip<NB>(red, seq, lane);
  } else {
    const uint32_t band_lo = band * o.KT, band_hi = band_lo + o.KT;
    const uint32_t lo = share0 > band_lo ? share0 : band_lo;
    const uint32_t hi = share1 < band_hi ? share1 : band_hi;
    uint32_t owner = 0;
    // asked for here, needed once the workgroup's sum is complete (in the dense kernel asked for then: a load that is not waited for on
    // every way through here would make its ring wait for everything)
    if (early_release && lo != band_lo) owner = owner_word(o, band);
    if (wg_reduce_add<NB>(red, acc, seq, tiles, hi - lo, lane)) {
      wg_reduce_take<NB>(red, acc, seq, lane);  // acc = the workgroup's sum over [lo, hi)
      if ((lo == band_lo && hi == band_hi) || local_only) {
        store_band<NB>(o, acc, band, lane);
      } else if (lo == band_lo) {
        st.own = true;  // the share ends inside this band: nothing follows, keep the sum
        st.own_band = band;
      } else {
        if (!early_release) owner = owner_word(o, band);
        st.local = runs_here(owner);
        store_partial<NB>(o, acc, wg, st.local, lane);
        // the sparse kernel's load ring is empty at the end of a piece, so nothing of it has to be
        // waited for to start the write-back here; the dense kernel keeps its ring going and
        // releases in one go at the end
        if (early_release && !st.local) {
          release_begin();
          st.released = true;
        }
        st.publish = true;
      }
    }
  }
  if (!st.own) {
#pragma unroll
    for (int rb = 0; rb < kRowBlocks; ++rb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[rb][nb] = float4v{0.f, 0.f, 0.f, 0.f};
  }
}

// After the tile loop.
template <int NB>
__device__ __forceinline__ void hand_over_finish(const OutParams& o, float4v (&acc)[kRowBlocks][NB],
                                                 const HandoverState& st, uint32_t wg, uint32_t near_end, int lane) {
  if (st.publish) {
    publish_partial(o, wg, lane, st.local, st.released);
  }
  if (st.own) {
    owner_finish<NB>(o, acc, st.own_band, wg, near_end, lane);
  }
}

// B operand fragments (X) of one K tile.  An MFMA wants lane l to hold column (l & 15) and the 8
// consecutive k of chunk (l >> 4), but loading X that way makes the four neighbouring lanes of
// every quad read four different cache lines (X is column-major).  So the load assigns lane j
// column (j >> 2) and chunk (j & 3) - a quad reads 64 contiguous bytes - and the fragment is put
// into MFMA order through a 1 KB LDS block per 16 columns: written as loaded, read back
// transposed.  The slot permutation keeps both the 16 B writes and the 16 B reads free of bank
// conflicts (any 16 neighbouring lanes touch 16 different 16 B slots modulo 256 B).
//
// The loads go through a buffer descriptor that ends after column N - 1, so the columns that pad
// N up to a multiple of 16 read as zero without a branch or a select after the load (either
// would make the compiler wait for the load on the spot).
struct XFrags {
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t lane_off;  // byte offset of the column and k chunk this lane loads
  uint32_t col_step;  // bytes between column blocks
  uint32_t wslot;     // byte offset in a column block's LDS stage where this lane's load goes
  uint32_t rslot;     // ... and where this lane's MFMA fragment comes from

  // 16 B slot of (column c, chunk g) of a 16-column block
  static __device__ __forceinline__ uint32_t slot(uint32_t c, uint32_t g) {
    return 16u * (c >> 2) + 4u * (c & 3u) + (g ^ (c >> 2));
  }
  __device__ __forceinline__ void init(const _Float16* X, uint32_t K, uint32_t N, uint32_t n0, int lane) {
    rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)X, 0, (int)(N * K * 2u), kBufferFlags);
    const uint32_t c = (uint32_t)lane >> 2, g = (uint32_t)lane & 3u;
    lane_off = ((n0 + c) * K + g * 8u) * 2u;
    col_step = 16u * K * 2u;
    wslot = slot(c, g) * 16u;
    rslot = slot((uint32_t)lane & 15u, (uint32_t)lane >> 4) * 16u;
  }
  template <int NB>
  __device__ __forceinline__ void load(u32x4 (&x)[NB], uint32_t kt) const {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      x[nb] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_off + nb * col_step, kt * (kTileK * 2u), 0);
  }
  // loaded registers -> the wave's LDS stage (NB KB)
  template <int NB>
  __device__ __forceinline__ void stage(unsigned char* xs, const u32x4 (&x)[NB]) const {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) *(u32x4*)(xs + nb * 1024 + wslot) = x[nb];
  }
  // MFMA B fragment of column block nb
  __device__ __forceinline__ half8 frag(const unsigned char* xs, int nb) const {
    return *(const half8*)(xs + nb * 1024 + rslot);
  }
};

}  // namespace fls
