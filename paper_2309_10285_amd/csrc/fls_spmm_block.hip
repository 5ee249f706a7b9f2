// fls_spmm for many columns: a workgroup decompresses a K tile once and multiplies it with 256 (or 128)
// columns of X.
//
// The 64-column pass extracts every tile once per 64 columns, and LDS then works longer on a tile
// (extraction, re-zeroing, fragment reads) than the matrix cores do: 765 TFLOP/s at 12288 x 12288 x 4096.
// Here a wave multiplies 128 rows x 128 columns (256 accumulator registers, one wave per SIMD with the whole
// register file), so an A fragment read feeds four MFMAs instead of two, and a tile serves more columns:
//   SHARE = 2: 2 row bands x 256 columns; the two waves of a band extract half of each tile's words each
//   SHARE = 1: 4 row bands x 128 columns; every wave extracts its own band's tiles
// Either way the four waves share all X in LDS and meet at one barrier per K tile.
//
// Pipeline, step t (three LDS buffers of W tiles and of X, loop unrolled by three so that every buffer and
// register stage is a constant): fragments of tile t are read from buffer t % 3; the words of tile t + 1
// are extracted and its X stored into buffer (t + 1) % 3; buffer (t + 2) % 3, whose fragments were read
// in step t - 1, is made zero; words and X of tile t + 4 are requested from memory.  The 32 MFMAs of a step
// (v_mfma_f32_32x32x16_f16 as asm statements in a fixed order) work half a step behind the fragment
// reads, and the step's other work is dealt out between them.
#include <atomic>
#include <type_traits>

#include "fls_device.h"
#include "fls_launch.h"
#include "fls_mfma32.h"
#include "fls_tile.h"

namespace fls {

constexpr int kBlockWaves = 4;
constexpr int kBlockCB = 4;                      // 32-column blocks of a wave
constexpr int kBlockStages = 3;                  // tiles in flight: register stages, LDS buffers
constexpr int kBlockTileLds = kTileBytes + 16;   // a tile + the slot padding words land in

template <int SHARE>
constexpr int block_lds_bytes() {
  return kBlockStages * ((kBlockWaves / SHARE) * kBlockTileLds + SHARE * 8192);
}

// Swizzle of an X slot by k chunk: makes the 16 B stores (16 lanes: 4 columns x 4 k chunks) hit 16 different
// slots modulo 256 B and any 8 neighbouring lanes 8 different ones modulo 128 B; the fragment reads
// permute 16 neighbouring slots.
__device__ __forceinline__ uint32_t x_swizzle(uint32_t ch) { return (ch & 1u) * 10u ^ (ch >> 1) * 4u; }

// RW = rounds of 256 entries that one wave stages per tile (all of the tile's with SHARE = 1, every other one
// with SHARE = 2).
template <int SHARE, int RW, int FMT>
__global__ __launch_bounds__(kBlockWaves * 64) __attribute__((amdgpu_waves_per_eu(1, 1))) void spmm_block_kernel(WideParams p) {
  constexpr int CB = kBlockCB, NST = kBlockStages;
  constexpr int kBands = kBlockWaves / SHARE;       // row bands of a workgroup
  constexpr int kXLoads = 2 * SHARE;                // X loads of a wave per K tile (16 columns each)
  constexpr uint32_t kCols = SHARE * CB * 32u;      // columns of a workgroup
  constexpr uint32_t kRoundWords = FMT == 2 ? kRoundWords2 : 256u;
  constexpr uint32_t kXBytes = kCols * kTileK * 2u;  // X of one K tile
  // X has at most 0x7fffffc0 bytes: an offset from kPast on reads as zero, also with kPastK added, and so does any
  // offset inside X with kPastK added
  constexpr uint32_t kPast = 0x80000000u, kPastK = 0x7fffffc0u;
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t wb = wave / SHARE, wh = wave % SHARE;  // band of the workgroup; half of the columns and of the tile's words

  // Unit of work -> (K slice, group of bands) pair and column group, eight pairs of neighbours at a time: the 32
  // workgroups that run on an XCD together are eight pairs x four column groups, which share words and X in its L2.
  const uint32_t bgroups = (p.bands + kBands - 1u) / kBands, cgroups = (p.N - p.n0 + kCols - 1u) / kCols;
  const uint32_t pairs = bgroups * p.S;
  uint32_t w;
  if (!xcd_unit(pairs * cgroups, w)) return;
  const uint32_t set = divide(w, p.by_G), in_set = w - set * 8u * cgroups, set_pairs = pairs - set * 8u < 8u ? pairs - set * 8u : 8u;
  const uint32_t cg = set_pairs == 8u ? in_set / 8u : in_set / set_pairs, pair = set * 8u + in_set - cg * set_pairs;
  const uint32_t slice = divide(pair, p.by_groups), bgroup = pair - slice * bgroups;
  const uint32_t band = bgroup * kBands + wb;
  const bool active = band < p.bands;  // a wave past the last band loads no words but shares the X work
  const uint32_t n0 = p.n0 + cg * kCols;  // first column of the workgroup
  const uint32_t KT = p.KT, T = p.bands * KT;
  // the slice: whole bodies of three tiles; the last body of all may reach past K (no words, X reads as zero)
  const uint32_t bodies_all = (KT + NST - 1u) / NST;
  const uint32_t b0 = divide(slice * bodies_all, p.by_S), b1 = divide((slice + 1) * bodies_all, p.by_S);
  const uint32_t k0 = b0 * NST, k1 = b1 * NST < KT ? b1 * NST : KT;
  const uint32_t t0 = active ? band * KT + k0 : T;
  const uint32_t ntiles = active ? k1 - k0 : 0;

  unsigned char* const wbuf = lds;                                          // [stage][band] tiles
  unsigned char* const xbuf = lds + NST * kBands * kBlockTileLds;           // [stage] X
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  for (uint32_t i = threadIdx.x; i < (uint32_t)(NST * kBands * kBlockTileLds / 16); i += kBlockWaves * 64) *(u32x4*)(wbuf + i * 16) = zero4;

  float16v acc[kRowBlocks32][CB];
#pragma unroll
  for (int rb = 0; rb < kRowBlocks32; ++rb)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[rb][cb][r] = 0.f;

  // ---- X: load e of a wave takes 16 columns (lane l: column l >> 2, k chunk l & 3 of the tile), 16-column group
  // wave * kXLoads + e.  LDS: 1 KB blocks (32-column block, 16-k step) of 64 slots of 16 B; the fragment of MFMA lane
  // 32 h + c of step ks is in slot 32 h + (c ^ x_swizzle(2 ks + h)).
  const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)p.X, 0, (int)(p.N * p.K * 2u), kBufferFlags);
  uint32_t xoff[kXLoads], xw_addr[kXLoads];
  {
    const uint32_t ch = (uint32_t)lane & 3u;
#pragma unroll
    for (int e = 0; e < kXLoads; ++e) {
      const uint32_t g = wave * kXLoads + e, c = (g & 1u) * 16u + ((uint32_t)lane >> 2);  // column in its 32-column block
      const uint32_t col = n0 + (g >> 1) * 32u + c;
      xoff[e] = col < p.N ? (col * p.K + k0 * kTileK + ch * 8u) * 2u : kPast;
      xw_addr[e] = (uint32_t)(uintptr_t)xbuf + (g >> 1) * 2048u + (ch >> 1) * 1024u + (32u * (ch & 1u) + (c ^ x_swizzle(ch))) * 16u;
    }
  }
  uint32_t xr_addr[kSteps16];
#pragma unroll
  for (int ks = 0; ks < kSteps16; ++ks) {
    const uint32_t c = (uint32_t)lane & 31u, h = (uint32_t)lane >> 5;
    xr_addr[ks] = (uint32_t)(uintptr_t)xbuf + wh * (CB * 2048u) + ks * 1024u + (32u * h + (c ^ x_swizzle(2u * ks + h))) * 16u;
  }
  typedef __attribute__((address_space(3))) u32x4* lds_v4_ptr;
  typedef __attribute__((address_space(3))) const half8* lds_h8_ptr;
  typedef __attribute__((address_space(3))) uint16_t* lds_u16_ptr;
  // X of K tile k0 + rel; past the slice it reads as zero (an Inf of the next slice times the zero tile would be NaN)
  auto xload = [&](u32x4& x, int e, uint32_t rel) {
    x = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, xoff[e] + (k0 + rel < k1 ? rel * 64u : kPastK), 0, 0);
  };

  // ---- W: as in the 64-column pass, a window of TileOffsets in a VGPR, replaced once per body
  const uint32_t* offs = p.offs;
  auto window_at = [&](uint32_t first) {
    const uint32_t i = first + (uint32_t)lane;
    return offs[i < T ? i : T];
  };
  uint32_t window = window_at(t0);
  // tile `rel` of the run, whose offsets are lanes i, i + 1 of the window; n = words of the tile (0 past the run)
  auto issue = [&](u32x4(&s)[RW], uint32_t& n, int i, uint32_t rel) {
    const uint32_t begin = (uint32_t)__builtin_amdgcn_readlane((int)window, i);
    const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)window, i + 1);
    n = end - begin;
    if (n > RW * SHARE * kRoundWords) n = RW * SHARE * kRoundWords;
    if (rel >= ntiles) n = 0;
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)(p.words + begin), 0, (int)(n * 4u), kBufferFlags);
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      const uint32_t unit = ((uint32_t)(r * SHARE) + wh) * 64u + (uint32_t)lane;
      if constexpr (FMT == 2) {
        const u32x3 g = __builtin_amdgcn_raw_buffer_load_b96(rsrc, unit * 12u, 0, 0);
        s[r] = u32x4{g[0], g[1], g[2], 0u};
      } else {
        s[r] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, unit * 16u, 0, 0);
      }
    }
  };
  const uint32_t wtile_addr = (uint32_t)(uintptr_t)wbuf + wb * kBlockTileLds;  // the band's tile of stage 0
  uint32_t ebase = 0, eaddr = 0;
  // extraction of round r in five parts: the base (of the padding slot for a lane past the end of the run), then the four entries
  auto extract_part = [&](const u32x4& s, uint32_t n, uint32_t tile_addr, int r, int part) {
    if (part == 0) {
      const uint32_t unit = ((uint32_t)(r * SHARE) + wh) * 64u + (uint32_t)lane;
      ebase = unit * (FMT == 2 ? kGroupWords : 4u) < n ? tile_addr : tile_addr + (uint32_t)kTileBytes;
      return;
    }
    const int j = part - 1;
    if constexpr (FMT == 2) {
      const uint32_t w2 = s[2];
      if (j == 0) eaddr = ebase + 2u * (w2 & 0xfffu);
      else eaddr = eaddr + 2u * ((w2 >> (6 + 6 * j)) & 0x3fu);
      const uint32_t v = s[j >> 1];
      *(lds_u16_ptr)(uintptr_t)eaddr = (j & 1) ? (uint16_t)(v >> 16) : (uint16_t)v;
    } else {
      const uint32_t w = s[j];
      *(lds_u16_ptr)(uintptr_t)scatter_addr(w, ebase) = (uint16_t)(w >> 16);
    }
  };

  // A fragment (32-row block rb, 16-k step ks) of the band's tile in stage b
  const unsigned char* const frag = wbuf + wb * kBlockTileLds + ((lane >> 5) * kTileM + (lane & 31)) * 16;
  auto afrag = [&](int b, int rb, int ks) { return *(const half8*)(frag + b * (kBands * kBlockTileLds) + ks * 4096 + rb * 512); };
  auto xfrag = [&](int b, int cb, int ks) { return *(lds_h8_ptr)(uintptr_t)(xr_addr[ks] + (uint32_t)b * kXBytes + (uint32_t)cb * 2048u); };
  unsigned char* const clear_at = wbuf + wb * kBlockTileLds + wh * (kTileBytes / SHARE) + lane * 16;

  // Step t = body * 3 + it.  (fa, fb)[0] receive the fragments of tile t's first 16 k and [1] those of the second;
  // on entry [1] holds the second 16 k of tile t - 1.  `rel` = t.
  half8 fa[2][kRowBlocks32], fb[2][CB];
  u32x4 s[NST][RW], xs[NST][kXLoads];
  uint32_t sn[NST];
  auto step = [&](auto it_, uint32_t rel) {
    constexpr int it = decltype(it_)::value, nx = (it + 1) % NST, zr = (it + 2) % NST;
    constexpr int kReads = kRowBlocks32 + CB, kClear = kTileBytes / 1024 / SHARE;
    constexpr int kOps0 = kReads + kClear + kXLoads + 1;      // reads, re-zeroing, X stores, X loads
    constexpr int kE = 5 * RW;                                 // extraction
    constexpr int kFirst = kE > 16 ? (kE - 8) / 2 : 0;        // ... as much of it in the first half
    auto read = [&](auto ks_, auto o_) {
      constexpr int ks = decltype(ks_)::value, o = decltype(o_)::value;
      if constexpr (o < CB) fb[ks][o] = xfrag(it, o, ks);
      else fa[ks][o - CB] = afrag(it, o - CB, ks);
    };
    const uint32_t next_tile = wtile_addr + (uint32_t)nx * (kBands * kBlockTileLds);
    static_for<0, 2>([&](auto half_) {
      constexpr int half = decltype(half_)::value;
      auto other = [&](auto o_) {
        constexpr int o = decltype(o_)::value;
        if constexpr (o < kReads) {
          read(half_, o_);
        } else if constexpr (half == 0) {
          constexpr int q = o - kReads;
          if constexpr (q < kFirst) extract_part(s[nx][q / 5], sn[nx], next_tile, q / 5, q % 5);
          else if constexpr (q < kFirst + kXLoads) {
            constexpr int e = q - kFirst;
            *(lds_v4_ptr)(uintptr_t)(xw_addr[e] + (uint32_t)nx * kXBytes) = xs[nx][e];
          } else if constexpr (q < kFirst + kXLoads + kClear) {
            constexpr int z = q - kFirst - kXLoads;
            *(u32x4*)(clear_at + zr * (kBands * kBlockTileLds) + z * 1024) = zero4;
          } else {
#pragma unroll
            for (int e = 0; e < kXLoads; ++e) xload(xs[nx][e], e, rel + 1u + NST);
          }
        } else {
          constexpr int q = o - kReads + kFirst;
          if constexpr (q < kE) extract_part(s[nx][q / 5], sn[nx], next_tile, q / 5, q % 5);
          else issue(s[nx], sn[nx], it, rel + 1u + NST);
        }
      };
      constexpr int kOps = half == 0 ? kOps0 + kFirst : kReads + (kE - kFirst) + 1;
      constexpr int kMfmas = kRowBlocks32 * CB;
      // the MFMAs of the fragments read half a step ago
      static_for<0, kMfmas>([&](auto m_) {
        constexpr int m = decltype(m_)::value, rb = m / CB, cb = m % CB;
        mfma_in_place(acc[rb][cb], fb[1 - half][cb], fa[1 - half][rb]);
        static_for<m * kOps / kMfmas, (m + 1) * kOps / kMfmas>(other);
      });
    });
    // tile t + 1 is in LDS and tile t's buffers have been read, by all four waves
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };

  // As in the 64-column pass: a blob that is denser by now than the variant was picked for takes the plain loop.
  const uint32_t densest = offs[kHeaderMaxTileWords - kHeaderWords];
  __syncthreads();  // LDS is zero
  if (densest <= RW * SHARE * kRoundWords) {
    // Prologue: tiles 0, 1, 2 requested, tile 0 into LDS, tile 3 requested in its place.  (The window of offsets
    // is always requested before the loads that follow it, so waiting for it does not wait for them.)
    uint32_t next_window = window_at(t0 + NST + 1u);
#pragma unroll
    for (int i = 0; i < NST; ++i) {
      issue(s[i], sn[i], i, (uint32_t)i);
#pragma unroll
      for (int e = 0; e < kXLoads; ++e) xload(xs[i][e], e, (uint32_t)i);
    }
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
      for (int part = 0; part < 5; ++part) extract_part(s[0][r], sn[0], wtile_addr, r, part);
#pragma unroll
    for (int e = 0; e < kXLoads; ++e) *(lds_v4_ptr)(uintptr_t)xw_addr[e] = xs[0][e];
    issue(s[0], sn[0], NST, (uint32_t)NST);
#pragma unroll
    for (int e = 0; e < kXLoads; ++e) xload(xs[0][e], e, (uint32_t)NST);
    // nothing to multiply in the first half step
#pragma unroll
    for (int j = 0; j < kRowBlocks32; ++j) fa[1][j] = half8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < CB; ++j) fb[1][j] = half8{0, 0, 0, 0, 0, 0, 0, 0};
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const uint32_t steps = (b1 - b0) * NST;
    for (uint32_t rel = 0; rel < steps; rel += NST) {
      // this body's requests are tiles rel + 4 ... rel + 6: lanes 0 ... 3 of the window that starts at rel + 4
      window = next_window;
      next_window = window_at(t0 + rel + 2u * NST + 1u);
      step(std::integral_constant<int, 0>{}, rel);
      step(std::integral_constant<int, 1>{}, rel + 1u);
      step(std::integral_constant<int, 2>{}, rel + 2u);
    }
#pragma unroll
    for (int rb = 0; rb < kRowBlocks32; ++rb)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) mfma_in_place(acc[rb][cb], fb[1][cb], fa[1][rb]);
    // the accumulators, asm operands, are read by ordinary instructions next: the wait states are given by hand
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  } else if (active) {
    // One tile the plain way, each wave for itself: words into a tile buffer of the wave's own, X from memory.
    unsigned char* const tile = wbuf + wave * kBlockTileLds;
    const uint32_t xd_col = n0 + wh * (CB * 32u) + ((uint32_t)lane & 31u);
    for (uint32_t kt = k0; kt < k1; ++kt) {
      const uint32_t begin = (uint32_t)__builtin_amdgcn_readfirstlane((int)offs[band * KT + kt]);
      const uint32_t end = (uint32_t)__builtin_amdgcn_readfirstlane((int)offs[band * KT + kt + 1]);
      // (not the out-of-line loops of fls_tile.h: a call would cost registers in the pipelined loop too)
      if constexpr (FMT == 2) {
        for (uint32_t i = begin + (uint32_t)lane * kGroupWords; i < end; i += kRoundWords2)
          extract_group(p.words[i], p.words[i + 1], p.words[i + 2], (uint32_t)(uintptr_t)tile);
      } else {
        for (uint32_t i = begin + (uint32_t)lane * 4u; i < end; i += 256u) {
          const u32x4 w = *(const u32x4*)(p.words + i);
#pragma unroll
          for (int j = 0; j < 4; ++j) *(uint16_t*)(tile + ((w[j] & 0xffffu) << 1)) = (uint16_t)(w[j] >> 16);
        }
      }
      const unsigned char* f = tile + ((lane >> 5) * kTileM + (lane & 31)) * 16;
#pragma unroll
      for (int ks = 0; ks < kSteps16; ++ks) {
        half8 a[kRowBlocks32], b[CB];
#pragma unroll
        for (int rb = 0; rb < kRowBlocks32; ++rb) a[rb] = *(const half8*)(f + ks * 4096 + rb * 512);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          const uint32_t col = xd_col + cb * 32u;
          const uint32_t off = (col * p.K + kt * kTileK + ks * 16u + ((uint32_t)lane >> 5) * 8u) * 2u;
          b[cb] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, col < p.N ? off : kPast, 0, 0));
        }
#pragma unroll
        for (int rb = 0; rb < kRowBlocks32; ++rb)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b[cb], a[rb], acc[rb][cb], 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < kTileBytes / 1024; ++i) *(u32x4*)(tile + i * 1024 + lane * 16) = zero4;
    }
  }
  if (!active) return;

  const uint32_t nw = n0 + wh * (CB * 32u);  // first column of the wave
  if (p.S == 1) {
    store_band32<CB>(p.C, p.M, p.N, nw, acc, band, lane);
  } else {
    // partial sums, laid out for the 64-column pass's adding kernel: [band][group of 64 columns][slice][...]
#pragma unroll
    for (int g = 0; g < CB / 2; ++g) {
      const uint32_t g64 = (nw - p.n0) / 64u + g;
      if (g64 >= p.G) break;
      float4v* dst = (float4v*)p.parts + ((size_t)((band * p.G + g64) * p.S + slice) * 32) * 64 + lane;
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int rb = 0; rb < kRowBlocks32; ++rb)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            dst[((cb * kRowBlocks32 + rb) * 4 + q) * 64] =
                float4v{acc[rb][2 * g + cb][4 * q], acc[rb][2 * g + cb][4 * q + 1], acc[rb][2 * g + cb][4 * q + 2],
                        acc[rb][2 * g + cb][4 * q + 3]};
    }
  }
}

template <int SHARE, int RW, int FMT>
static hipError_t launch_block_variant(WideParams p, hipStream_t stream) {
  static std::atomic<bool> attr_done{false};  // per kernel variant; setting the attribute twice from two threads is harmless
  constexpr int kLds = block_lds_bytes<SHARE>();
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)spmm_block_kernel<SHARE, RW, FMT>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    if (e != hipSuccess) return e;
    attr_done.store(true, std::memory_order_release);
  }
  const uint32_t bgroups = block_band_groups(p.bands, SHARE), cgroups = block_col_groups(p.N - p.n0, SHARE);
  const uint32_t grid = (bgroups * p.S * cgroups + 7u) / 8u * 8u;
  p.by_S = divisor(p.S);
  p.by_G = divisor(8u * cgroups);
  p.by_groups = divisor(bgroups);
  hipLaunchKernelGGL((spmm_block_kernel<SHARE, RW, FMT>), dim3(grid), dim3(kBlockWaves * 64), kLds, stream, p);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && p.S > 1) e = launch_wide_reduce(p, true, stream);
  return e;
}

template <int FMT>
static hipError_t launch_block_fmt(const WideParams& p, uint32_t share, uint32_t rounds, hipStream_t stream) {
  if (share == 1u) {
    switch (rounds) {
      case 2: return launch_block_variant<1, 2, FMT>(p, stream);
      case 3: return launch_block_variant<1, 3, FMT>(p, stream);
      case 4: return launch_block_variant<1, 4, FMT>(p, stream);
      default: return launch_block_variant<1, 6, FMT>(p, stream);
    }
  }
  switch (rounds) {
    case 2: return launch_block_variant<2, 1, FMT>(p, stream);
    case 4: return launch_block_variant<2, 2, FMT>(p, stream);
    case 6: return launch_block_variant<2, 3, FMT>(p, stream);
    case 8: return launch_block_variant<2, 4, FMT>(p, stream);
    default: return launch_block_variant<2, 5, FMT>(p, stream);
  }
}

// Measurement builds (pass_times.py): 0, 1 or 2 takes that pass for every call of more than 64 columns.
#ifndef FLS_PASS
#define FLS_PASS -1
#endif

uint32_t spmm_pass_share(uint32_t need, uint32_t bands, uint32_t KT, uint32_t N, int cus) {
  if (FLS_PASS >= 0) return (uint32_t)FLS_PASS;
  const uint32_t R = wide_rounds(need), body = wide_body(R);  // of the 64-column pass
  // `round`: what a round of workgroups costs beside its steps
  auto estimate = [&](float start, uint32_t units, uint32_t S, float round, float steps) {
    const uint32_t wgs = units * S, rounds = (wgs + (uint32_t)cus - 1u) / (uint32_t)cus;
    const float fill = (float)wgs / ((float)rounds * (float)cus);
    float us = start + (float)rounds * (round + steps * (0.7f + 0.3f * fill));
    if (S > 1u) us += 1.0f + (float)bands * (float)((N + 63u) / 64u) * (float)S * (2.0f * 32768.0f / 7.0e6f);
    return us;
  };
  // the 64-column pass: whole bodies, and in the last slice tile by tile what is left of K
  const uint32_t groups = (N + 63u) / 64u, S0 = wide_quad_slices(bands, groups, KT, cus, R), bodies = (KT / body + S0 - 1u) / S0;
  float best = 0.97f * estimate(4.0f, (bands + 3u) / 4u * groups, S0, bodies > 0u ? 3.0f : 0.0f,
                                (float)(bodies * body) * (0.24f + 0.08f * (float)R) + (float)(KT % body) * (0.90f + 0.28f * (float)R));
  uint32_t pick = 0;
  for (uint32_t share = 1; share <= 2; ++share) {
    if (share == 1u && need > kBlockRounds1) continue;
    const uint32_t units = block_band_groups(bands, share) * block_col_groups(N, share), S = block_slices(units, KT, cus);
    const float r = (float)block_rounds(share, need), step = share == 1u ? 0.68f + 0.047f * r : 0.675f + 0.017f * r;
    const float us = estimate(4.0f + 3.0f, units, S, 4.0f, (float)(((KT + 2u) / 3u + S - 1u) / S * 3u) * step);
    if (us < best) {
      best = us;
      pick = share;
    }
  }
  return pick;
}

hipError_t launch_spmm_block(const SpmmLaunch& a, const SpmmPlan& plan, hipStream_t stream) {
  WideParams p;
  p.offs = a.offs;
  p.words = a.words;
  p.W = nullptr;
  p.X = a.X;
  p.Xp = nullptr;
  p.C = a.C;
  p.parts = a.parts;
  p.M = a.M;
  p.K = a.K;
  p.N = a.N;
  p.n0 = 0;
  p.KT = a.K / kTileK;
  p.bands = a.M / kTileM;
  p.S = plan.slices;
  p.G = (a.N + 63u) / 64u;
  p.cb = 2;
  return a.version == 2 ? launch_block_fmt<2>(p, plan.share, plan.rounds, stream) : launch_block_fmt<1>(p, plan.share, plan.rounds, stream);
}

}  // namespace fls
