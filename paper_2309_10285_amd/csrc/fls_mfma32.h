// What the 64-column pass and the block pass share: MFMAs of the 32x32x16 shape as asm statements in a fixed order,
// and the store of their accumulators.
#pragma once
#include <type_traits>

#include "fls_device.h"

namespace fls {

// Compile-time loop: f(integral_constant<int, I>) for I in [B, E).
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// acc += a . b with the accumulator kept where it is (sixteen AGPRs): as an asm statement, so that
// the instruction keeps its place between the memory operations around it.
//
// The 64-column pass multiplies with v_mfma_f32_32x32x16_f16 rather than 16x16x32: half as many
// instructions for the same work, each leaving eight issue slots in its shadow.  Operand layouts
// of the 32x32x16 shape, lane l = 32 h + c:
//   A: row c of the 32-row block, the 8 k of chunk h of the 16-k step;  B: column c, the same 8 k;
//   C/D: column c, rows 8 q + 4 h + (0..3) in registers 4 q .. 4 q + 3, q = 0..3.
// A and B hold the same thing in the same lanes, so either operand can be the W block.  The pass
// computes the transposed product, X block (A) times W block (B): the chip's clock under this
// kernel is set by power, the matrix cores draw less when the operand that is mostly zeros is B,
// and the call is 3 % faster for it (measured; with X all zeros instead of random values the same
// instruction stream runs 15 - 18 % faster still, with W's values all equal 2 %).  An accumulator block
// is therefore 32 columns of X (its rows) by 32 rows of W (its columns).
typedef float float16v __attribute__((ext_vector_type(16)));
__device__ __forceinline__ void mfma_in_place(float16v& acc, const half8& a, const half8& b) {
  asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
constexpr int kRowBlocks32 = kTileM / 32;  // 32-row blocks of a tile
constexpr int kSteps16 = kTileK / 16;      // 16-k steps of a tile

// Converts a wave's 128 x 64 accumulators (32x32 layout, transposed: see above) to fp16 and stores them
// to column-major C: register 4 q + r of block (rb, cb) is row 32 rb + c of the band, column
// 32 cb + 8 q + 4 h + r of the group - 64 contiguous bytes of C per store and half wave.
template <int CB>
__device__ __forceinline__ void store_band32(_Float16* C, uint32_t M, uint32_t N, uint32_t n0,
                                             const float16v (&acc)[kRowBlocks32][CB], uint32_t band, int lane) {
  const uint32_t c = lane & 31, h = lane >> 5;
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t n = n0 + cb * 32 + q * 8 + h * 4 + r;
        if (n < N) {
#pragma unroll
          for (int rb = 0; rb < kRowBlocks32; ++rb)
            C[(size_t)n * M + band * kTileM + rb * 32 + c] = (_Float16)acc[rb][cb][4 * q + r];
        }
      }
}

}  // namespace fls
