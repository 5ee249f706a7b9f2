// Host-side launch descriptors: the C ABI layer fills these, each kernel file implements its launcher.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace fls {

// Division by a number known at launch: n / d = n m >> k for n < 2^29 (Granlund and Montgomery 1994: m d - 2^k < d <= 2^(k - 29)).  On the
// GPU three scalar instructions, where a division is some thirty vector ones - at the start of a kernel, before the first load:
// 1024 x 1024 at 80 %, N = 8 6.66 -> 6.43 us, a 7168-wide decoder layer 108.9 -> 107.5.
struct Divisor {
  uint32_t m, k;
};
inline Divisor divisor(uint32_t d) {
  uint32_t l = 0;
  while (l < 31u && (1u << l) < d) ++l;
  return {(uint32_t)((((uint64_t)1 << (29 + l)) + d - 1u) / d), 29u + l};
}
__host__ __device__ inline uint32_t divide(uint32_t n, Divisor d) { return (uint32_t)((uint64_t)n * d.m >> d.k); }

struct SpmmLaunch {
  const uint32_t* offs;   // TileOffsets section of the blob
  const uint32_t* words;  // NonZeros section of the blob
  const _Float16* X;
  _Float16* C;
  float* parts;
  uint32_t* flags;
  _Float16* xpack;  // workspace area of xpack_bytes(K, N) for X in MFMA fragment order (used when N > 32)
  uint32_t M, K, N;
  uint32_t max_tile_words;
  uint32_t version;  // format version of the blob (1 or 2)
  int num_cus;
  uint32_t raised;   // what a raised flag of the hand-over holds, nonzero
  // the partial-sum area was sized by parts_floats(N): a call of 17 - 32 columns may take the 64-column pass
  // (false for the static scratch of the entry point that allocates nothing, which has the narrow kernel's area only)
  bool wide32;
};

struct DenseLaunch {
  const _Float16* W;
  const _Float16* X;
  _Float16* C;
  float* parts;
  uint32_t* flags;
  _Float16* xpack;  // as in SpmmLaunch
  uint32_t M, K, N;
  int num_cus;
};

// Scratch of a compress call on the GPU: the next chunk to be taken (zero between calls) and, for every chunk, two words that
// bear the number of the call that wrote them, so that nothing else is cleared between calls.
constexpr uint32_t kCompressChunkTiles = 16;
constexpr uint32_t kCompressMaxChunks = (1u << 20) / kCompressChunkTiles;  // M * K < 2^32: fewer than 2^20 tiles
constexpr uint32_t kCompressCalls = 1u << 30;                              // a call's number is 1 ... kCompressCalls - 1
struct CompressScratch {
  alignas(256) uint32_t ticket;
  alignas(256) uint64_t sums[kCompressMaxChunks];
  uint64_t counts[kCompressMaxChunks];
};
// What a call leaves in host memory.
struct alignas(64) CompressHost {
  uint32_t header[16];
  uint32_t gave_up;  // 1 if a look-back gave up
};

struct CompressLaunch {
  const uint16_t* W;
  CompressScratch* scratch;
  CompressHost* host;  // as the device addresses it
  uint32_t call;       // 1 ... kCompressCalls - 1, another one than those of the calls before on this scratch
  uint32_t look_limit; // looks at another workgroup's word before the kernel gives up (host->gave_up; the blob is of no use then)
  bool by_ticket;      // chunks in the order in which workgroups start, not by their number
  unsigned char* out;  // blob
  size_t capacity;     // bytes of `out`, at least header and TileOffsets: no word goes past it
  uint32_t M, K;
  uint32_t policy;
  uint32_t version;  // 1: 32-bit words (value, location); 2: groups of four entries in three words, three bytes per entry
};

// Columns are processed in groups, one pass over W per group.  The dense baseline and the sparse
// kernel's narrow variants take up to kGroupCols columns (1 or 2 MFMA column blocks of 16 per
// wave); more than that goes to the sparse kernel's 64-column pass (four column blocks, four waves
// per workgroup with the whole register file each).
constexpr uint32_t kGroupCols = 32;
constexpr uint32_t kSpmmGroupCols = 64;
inline uint32_t group_blocks(uint32_t ncols) { return ncols <= 16 ? 1u : (ncols <= 32 ? 2u : 4u); }
constexpr uint32_t kMaxWorkgroups = 512;    // most shares of a launch of up to 32 columns, most K slices x units of the wider passes
// Control words of the hand-over between workgroups, one array of kMaxWorkgroups words after the other: flags of partial sums released at device
// scope; the error word, the rest of its array unused; the XCDs of waiting owners; flags of partial sums that stay in an XCD's L2.
constexpr uint32_t kErrorWord = kMaxWorkgroups, kOwnerXcd = 2 * kMaxWorkgroups, kLocalFlags = 3 * kMaxWorkgroups, kControlWords = 4 * kMaxWorkgroups;
// The 64-column pass of the dense kernel cuts its work as (group of 4 bands) x (K slice), one wave
// per band, and keeps one 128 x 64 fp32 partial result per band and slice.  Slices per group: as
// many as fill the CUs, none shorter than 16 steps of 64 k, or than two where the steps that a workgroup has less to walk (2.4 us each) take longer than what the
// further slices cost: their sums out and back at 4.2 TB/s and 2.5 us for the second kernel where there was none.  1408 x 1120, N = 182 37.9 us with slices
// of 16 steps, 18.0 with two, 5120 x 1120, N = 51 71.2 / 22.8, 1280 x 1888, N = 97 90.0 / 18.3; but 7424 x 224, N = 356 16.8 / 30.7, 15744 x 352, N = 240 20.9 /
// 36.7, 28928 x 384, N = 78 25.1 / 34.3.  On 306 products of 33 - 640 columns on which the two differ (M 128 ... 50000, K 64 ... 4096) two steps always are 1.60 times
// faster and up to 1.8 times slower, the pick 1.62 and (128 rows, a microsecond) 1.15, the better of both 1.63.  groups * slices <= kMaxWorkgroups, so
// bands * slices <= 4 * kMaxWorkgroups partial results at most (what parts_floats provides).
inline uint32_t wide_slices(uint32_t bands, uint32_t col_groups, uint32_t KT, int cus) {
  if (cus > (int)kMaxWorkgroups) cus = (int)kMaxWorkgroups;
  const uint64_t units = (uint64_t)((bands + 3) / 4) * col_groups;  // (group of four bands, group of 64 columns)
  const uint32_t fill = units < (uint64_t)cus ? (uint32_t)((uint64_t)cus / units) : 1u;
  auto slices = [&](uint32_t shortest) {
    const uint32_t by_length = KT / shortest > 0 ? KT / shortest : 1u;
    return fill < by_length ? fill : by_length;
  };
  // (at most 128 of two steps: the second kernel adds them one after the other.  One unit, 256 / 128 slices: 128 x 30848, N = 52 27.9 / 20.5, 256 x 32640, N = 57 34.9 / 25.7, 128 x
  // 18368, N = 52 19.3 / 18.4; 64 are faster still there, and up to 1.29 times slower on two units.)
  const uint32_t S16 = slices(16u), S2 = slices(2u) < 128u ? slices(2u) : 128u;
  if (S2 <= S16) return S16;
  const float saved = 2.4f * (float)((KT + S16 - 1u) / S16 - (KT + S2 - 1u) / S2);
  const float sums = 2.f * 32768.f / 4.2e6f * (float)bands * (float)col_groups * (float)(S2 - (S16 > 1u ? S16 : 0u));
  return saved > sums + (S16 > 1u ? 0.f : 2.5f) ? S2 : S16;
}
// Steps that a CU takes one after the other in that pass.
inline uint32_t wide_steps(uint32_t bands, uint32_t col_groups, uint32_t KT, int cus) {
  const uint32_t S = wide_slices(bands, col_groups, KT, cus), wgs = (bands + 3u) / 4u * col_groups * S;
  return (wgs + (uint32_t)cus - 1u) / (uint32_t)cus * ((KT + S - 1u) / S);
}
// Groups of 64 columns in the launch that the dense product's `left` > 32 columns begin with.
// A rest of up to 32 columns joins the launch as its last, partly empty group, whose workgroups find W in their XCD's L2, instead of
// a pass of its own (12288 x 12288, N = 80: 163 -> 149 us; 9856 x 4672, N = 94: 74 -> 59; 1152 x 5792, N = 158: 50 -> 36), unless a further
// group takes so many K slices away, or a round of workgroups more, that it costs more than the pass: 3 us a step against 8 us and W at 4 TB/s (30848 x 5248,
// N = 143 217 us with a pass for the rest, 246 without, 6272 x 16544, N = 199 243 and 253, 35712 x 3808, N = 219 321 and 421).
inline uint32_t dense_col_groups(uint32_t M, uint32_t K, uint32_t left, int cus) {
  const uint32_t full = left / kSpmmGroupCols, rest = left % kSpmmGroupCols, bands = M / 128u, steps = (K + 63u) / 64u;
  const float longer = 3.f * ((float)wide_steps(bands, full + 1u, steps, cus) - (float)wide_steps(bands, full > 0 ? full : 1u, steps, cus));
  const bool join = rest > kGroupCols || (rest > 0 && longer < 8.f + (float)M * (float)K * 2.f / 4.0e6f);
  return full + (join ? 1u : 0u);
}
// The sparse 64-column pass: a workgroup takes four bands (one per wave), a group of 64 columns and a
// K slice made of whole loop bodies, and writes one partial result per band, column
// group and slice.  Slices per (group of four bands, column group): as many as fill the CUs, none
// shorter than two bodies, or one where that pays.  With S > 1, groups of bands x column groups x S <= CUs <= kMaxWorkgroups,
// so at most 4 * kMaxWorkgroups partial results exist (what parts_floats provides).
inline uint32_t wide_body(uint32_t rounds) { return rounds <= 4u ? 8u : 4u; }  // by the rounds of a tile that the variant stages
inline uint32_t wide_quad_slices(uint32_t bands, uint32_t col_groups, uint32_t KT, int cus, uint32_t rounds) {
  if (cus > (int)kMaxWorkgroups) cus = (int)kMaxWorkgroups;
  const uint32_t body = wide_body(rounds), bodies = KT / body;
  const uint64_t units = (uint64_t)((bands + 3) / 4) * col_groups;
  const uint32_t fill = units < (uint64_t)cus ? (uint32_t)((uint64_t)cus / units) : 1u;
  const uint32_t two = bodies / 2u > 0 ? bodies / 2u : 1u, S2 = fill < two ? fill : two;  // slices of two bodies and more
  // ... or of one, as long as that makes few workgroups and few sums of it (up to 96 and 16), where the bodies that a workgroup has less to walk take longer than
  // what the further slices cost: 0.96 of the pass's step times against 1.66 us for the second kernel, where there was none, and the sums out and back at 4.9 TB/s.
  // Fitted to 212 products of 33 - 640 columns on which the two differ (M 128 ... 6000, K 256 ... 16384, 60 - 90 %, both formats; rms 0.7 us): one body always is
  // 1.146 times faster than two and up to 1.46 times slower, the pick 1.157 and 1.06, the better of both 1.159.  On 238 others 1.186, 1.187 and
  // 1.190, at worst 1.17 times slower than two bodies (1024 x 2944, N = 192 17.5 / 20.4), next 1.10.  Some of them (us, two
  // bodies / one): 2944 x 1088, N = 58 16.3 / 14.2; 1152 x 1504, N = 110 18.7 / 14.9; 2560 x 288, N = 564 12.1 / 17.7; 3584 x 608, N = 378 14.9 / 17.8; 4608 x 416, N = 260
  // 14.5 / 18.6; 2176 x 1056, N = 360 17.4 / 19.0.  Beyond 96 workgroups: 1408 x 10944, N = 56, 42 slices, 19.8 / 23.9; 4608 x 1344, N = 264, 225 workgroups, 26.6 / 29.9.
  const uint32_t few = units <= 6u ? 16u : (uint32_t)(96u / units), one = bodies < few ? bodies : few, S1 = fill < one ? fill : one;
  if (S1 <= S2) return S2;
  const float saved = 0.96f * (float)((bodies + S2 - 1u) / S2 - (bodies + S1 - 1u) / S1) * (float)body * (0.16f + 0.081f * (float)rounds);
  const float sums = 2.f * 32768.f / 4.9e6f * (float)bands * (float)col_groups * (float)(S1 - (S2 > 1u ? S2 : 0u));
  return saved > sums + (S2 > 1u ? 0.f : 1.66f) ? S1 : S2;
}
// How the 64-column passes spread their (group of four bands, K slice) pairs over the eight XCDs: whole pairs, in turn,
// unless that leaves an XCD so many more workgroups than others that it takes a round more than an even cut of
// all units.  7168 x 28672 at 80 %, N = 384: three slices, 42 pairs of six column groups, 36 workgroups on two XCDs of 32
// CUs: 316 us, evenly cut 180; 12672 x 7840 at 82 %, N = 1085: 377 / 266; 5504 x 2752 at 64 %, N = 2735: 217 / 150.  The dense
// pass, 7168 x 28672, N = 384: 896 / 516, and level (1 % either way) on 170 shapes of which most keep whole pairs.  Where both
// take as many rounds whole pairs are up to 2 % faster (12288 x 12288 at 80 %, N = 128: 55.2 / 56.4 us; 27648 x 9216 at 70 %,
// N = 32: 58.1 / 59.2).
inline bool whole_pairs(uint32_t pairs, uint32_t G, int cus) {
  const uint64_t per_xcd = cus >= 8 ? (uint64_t)cus / 8u : 1u;
  const uint64_t whole = (uint64_t)((pairs + 7u) / 8u) * G, even = ((uint64_t)pairs * G + 7u) / 8u;
  return (whole + per_xcd - 1u) / per_xcd == (even + per_xcd - 1u) / per_xcd;
}
// Workgroups of such a launch.
inline uint32_t wide_grid(uint32_t pairs, uint32_t G, bool whole) {
  return whole ? (pairs + 7u) / 8u * 8u * G : (pairs * G + 7u) / 8u * 8u;
}
// The block pass: a workgroup takes 4 / share row bands x 128 * share columns x a K slice of whole bodies of three tiles.
inline uint32_t block_band_groups(uint32_t bands, uint32_t share) { return (bands * share + 3u) / 4u; }
inline uint32_t block_col_groups(uint32_t cols, uint32_t share) { return (cols + 128u * share - 1u) / (128u * share); }
// Slices per (group of bands, column group): as many as fill the CUs, none shorter than twelve tiles.  A workgroup leaves
// eight partial results of 128 x 64, and 4 * kMaxWorkgroups of them have room.
inline uint32_t block_slices(uint32_t units, uint32_t KT, int cus) {
  const uint32_t most = cus < (int)(kMaxWorkgroups / 2) ? (uint32_t)cus : kMaxWorkgroups / 2;
  const uint32_t S = units < most ? most / units : 1u, by_length = KT / 12u > 0 ? KT / 12u : 1u;
  return S < by_length ? S : by_length;
}
// Which pass a call of more than 64 columns takes: 0 the 64-column pass, else the block pass's share.
// The passes differ in what a tile step costs (extraction and fragment reads are shared by 64, 128 or 256 columns), in
// how evenly their units fill the CUs (a ragged last round, columns that only pad), in how many partial sums they leave when K is
// sliced (a CU of the block pass holds twice as many), in what a workgroup's start and end cost (the block pass clears three
// buffers and stores twice the sums), and in the K tiles that fill no body, which the 64-column pass takes one by one.  These
// pull apart, so the rule is an estimate of each pass in us, with constants fitted to 2600 products over the sizes that the calls take:
//   a step of one workgroup 0.24 + 0.08 R (64 columns x 4 bands), 0.68 + 0.047 R (128 x 4), 0.675 + 0.017 R (256 x 2) for R staged
//   rounds of a tile, 0.90 + 0.28 R for a tile outside the bodies; down to 0.7 of that where the chip idles (the matrix cores' clock is set by power);
//   a round of workgroups 3 (64-column pass, if it has a body at all) or 4; a call 4, in the block pass 7; partial sums
//   1 and their bytes out and back at 7 TB/s; and what is level to 3 % goes to the 64-column pass.
// On 400 other products (M 128 ... 49152, K 32 ... 49152, N 65 ... 4096, 50 - 90 %, both formats) its pick takes 1.009 times the best of the three,
// 1.24 at most, and 0.865 times the 64-column pass; on four of them it is more than 2 % slower than that pass.  Some of what was measured
// (us, 64-column / share 1 / share 2): 12288 x 12288 at 80 %, N = 128 57.8 / 60.5 / 68.2, 256 111 / 89 /
// 84, 384 189 / 127 / 143, 1000 384 / 285 / 259, 4096 1328 / 975 / 914; at 90 %, N = 256 78 / 79 / 78, 512 133 / 145 / 140, 1024 272 / 249 / 242, 2048
// 437 / 530 / 498; 7168 x 28672 at 80 %, N = 384 176 / 151 / 174; 12288 x 480 at 80 %, N = 4096 139 / 70 / 67; 12288 x 32 at 90 %, N = 4096
// 30 / 38 / 38.
uint32_t spmm_pass_share(uint32_t need, uint32_t bands, uint32_t KT, uint32_t N, int cus);
constexpr uint32_t kBlockRounds1 = 6, kBlockRounds2 = 10;  // rounds of a tile that the variants with share 1 / 2 stage
// Variants by the rounds of 256 entries that they stage of a tile: the smallest that holds the densest tile, which needs
// `need` (the largest where none does: the kernels have a slow path for that).
inline uint32_t wide_rounds(uint32_t need) { return need <= 2u ? 2u : need <= 4u ? need : need <= 6u ? 6u : need <= 8u ? 8u : 10u; }
inline uint32_t block_rounds(uint32_t share, uint32_t need) {
  if (share == 1u) return need <= 2u ? 2u : need <= 4u ? need : kBlockRounds1;
  return need <= 2u ? 2u : need <= 8u ? (need + 1u) / 2u * 2u : kBlockRounds2;  // two waves stage a tile, every other round each
}
// fp32 values of the split-K partial sums: [workgroup][column blocks][128 x 16] for the passes of
// up to 32 columns, [band][slice][4][128 x 16] for the 64-column pass
inline size_t parts_floats(uint32_t N) {
  // (from 17 columns on: a call of 17 - 32 columns takes the 64-column pass where that is faster, see wide_pays)
  if (N > 16u) return (size_t)4 * kMaxWorkgroups * 4 * 2048;
  return (size_t)kMaxWorkgroups * group_blocks(N) * 2048;
}

// Workspace bytes for X repacked into MFMA fragment order, [K tile][column block][lane][8 halves]
// (the sparse kernel's wide variant reads it instead of X; narrower calls do not need it).
inline size_t xpack_bytes(uint32_t K, uint32_t N) {
  return N > kGroupCols ? (size_t)K * ((N + 15u) / 16u * 16u) * 2u : 0;
}

// How the tiles of a matrix of `bands` row bands are shared out to workgroups, at most one per CU, in the passes of up to 32
// columns.
struct Shares {
  uint32_t P;     // shares
  uint32_t unit;  // shares that stay together on an XCD; 0: a share is whole bands, no partial sum crosses between workgroups
  uint32_t grid;  // workgroups, the idle ones that fill up the XCDs' parts among them (see share_of_block)
};
// What a tile costs a workgroup, in us, by the rounds that its variant stages, and a tile of W that was left dense.
constexpr float kDenseTileUs = 0.27f;
inline float tile_us(uint32_t rounds, bool wide) { return 0.035f + 0.0175f * (float)rounds + (wide ? 0.02f : 0.f); }
// ... and a hand-over, of a band cut into k shares on one XCD.
inline float hand_over_us(uint32_t k, bool wide) { return wide ? 1.9f + 0.52f * (float)(k / 2u) : 1.6f + 0.6f * (float)((k + 2u) / 4u); }
inline Shares shares_of(uint32_t P, uint32_t unit) { return {P, unit, unit == 0 ? P : (P / unit + 7u) / 8u * unit * 8u}; }
// Shares that cut bands.  Those of one band, or of a pair of bands, stay together where no XCD gets more workgroups than it has CUs.
inline Shares cut_shares(uint32_t P, uint32_t bands, int cus) {
  uint32_t unit = P % bands == 0 ? P / bands : bands % 2u == 0 && P % (bands / 2u) == 0 ? P / (bands / 2u) : 1u;
  const uint32_t per_xcd = cus >= 8 ? (uint32_t)cus / 8u : 1u;
  if ((P / unit + 7u) / 8u * unit > per_xcd) unit = 1u;
  return shares_of(P, unit);
}
// A workgroup should have enough tiles to pay for its start, and cutting a band costs a hand-over.  Up to 64 tiles per CU the shares are the
// ones with the lowest estimate
//   tile_us x tiles of a workgroup + (a band cut into k shares: 1.6 us and 0.6 for every four slots that the owner adds - with 17 - 32 columns
//   1.9 and 0.52 for every two -, and 1.5 more where the shares of a band do not stay on one XCD),
// fitted to forced cuts into 1 - 32 shares of bands of 16 - 512 tiles (8, 32, 60 and 100 bands, 65 - 90 %, both formats, dense); a workgroup's LDS work is
// what a tile costs there.  Some of them (us, N = 8, 80 %, 8 bands): 32 tiles a band 7.3 whole, 7.8 / 6.7 in 2 / 4 shares; 64 tiles 10.9
// whole, 9.5 / 7.8 / 7.4 / 9.0 in 2 / 4 / 8 / 10; 256 tiles 12.9 / 10.1 / 9.8 / 11.2 in 4 / 8 / 16 / 32; N = 32, 64 tiles 12.8 whole, 9.6 / 9.3 / 9.6 in 4 / 5 / 8.
// A share has at least eight tiles, one for every wave: fewer take the slow way to a sum (32 tiles in 5 shares 7.7).
inline Shares pick_shares(uint32_t bands, uint32_t KT, int cus, float tile_us, bool wide) {
  if (cus > (int)kMaxWorkgroups) cus = (int)kMaxWorkgroups;
  const uint64_t T = (uint64_t)bands * KT;
  // More bands than CUs, or bands of fewer than eight tiles: `per` whole bands to a workgroup, which leaves CUs idle, unless cutting
  // all tiles evenly gains more than the hand-over costs.  (49152 x 256 at 80 %, N = 8: 192 workgroups of two bands 7.3 us, 256 cut ones 9.7; 49152 x
  // 512 9.0 / 10.4; 34816 x 1024 13.4 / 13.0; 49152 x 12288 at 80 %, N = 16: 96.4 / 87.8; 1024 x 256: eight workgroups 4.5, one 9.3.)
  const uint32_t m = (bands + (uint32_t)cus - 1u) / (uint32_t)cus, eight = KT <= 2u ? 8u : (8u + KT - 1u) / KT, per = m > eight ? m : eight;
  if (per > 1u) {
    if (per > m || tile_us * ((float)per * (float)KT - (float)T / (float)cus) < 2.5f) return shares_of((bands + per - 1u) / per, 0u);
    return cut_shares((uint32_t)cus, bands, cus);
  }
  const uint32_t most = (uint32_t)cus / bands;
  if (T < 64u * (uint64_t)cus) {
    uint32_t best = 1;
    float us = tile_us * (float)KT;
    const uint32_t near = (uint32_t)(cus >= 8 ? cus / 8 : 1) / ((bands + 7u) / 8u);  // k up to which cut_shares keeps a band's shares on one XCD
    for (uint32_t k = 2; k <= most && k * 8u <= KT; ++k) {
      float t = tile_us * (float)((KT + k - 1u) / k) + hand_over_us(k, wide);
      if (k > near) t += 1.5f;
      if (t < us) {
        us = t;
        best = k;
      }
    }
    // k shares to a band leave up to half the CUs without one: all tiles cut evenly over all CUs instead where that is estimated to be 0.3 us less, for sparse
    // tiles 2.5.  (Dense, k shares / cut: 138 bands of 92 steps of 32, N = 9 36.9 / 26.7, 149 of 62, N = 21 29.1 / 25.1, 175 of 49, N = 22 24.7 / 24.1, 92 of 154, N = 6 34.2 / 29.3, 70 of
    // 123, N = 16 27.2 / 25.2; all 139 drawn products whose time it changed gain, up to 1.46 times.  Of 34 sparse ones that took another time without the 2.5 us
    // 27 were slower, by up to a tenth: 150 of 61, N = 24 14.6 / 16.1.)
    const float cut = tile_us * (float)((T + (uint64_t)cus - 1u) / (uint64_t)cus) + hand_over_us((uint32_t)cus / bands + 1u, wide) + 1.5f + (tile_us < kDenseTileUs ? 2.5f : 0.3f);
    if (T >= 8u * (uint64_t)cus && cut < us)
      return cut_shares((uint32_t)cus, bands, cus);
    return best > 1u ? cut_shares(bands * best, bands, cus) : shares_of(bands, 0u);
  }
  // Larger problems are paced by HBM, not by the CUs: a count of the form bands * k, where every band has its own k workgroups, is
  // worth leaving up to a fifth of the CUs without one.
  const int aligned = (int)(bands * most);
  if (aligned * 5 >= cus * 4) return most > 1u ? cut_shares((uint32_t)aligned, bands, cus) : shares_of(bands, 0u);
  // next best: every pair of bands to an odd number of workgroups (only the middle one of each
  // group spans two bands), if that leaves next to no CU idle - 168 bands on 256 CUs: 252
  // workgroups measured 3 % faster than 256
  const int halves = (int)bands * (2 * cus / (int)bands);
  if (halves % 2 == 0 && halves / 2 * 100 >= cus * 97) return cut_shares((uint32_t)halves / 2u, bands, cus);
  return cut_shares((uint32_t)cus, bands, cus);
}

// A call of 17 - 64 columns: passes of up to 32 columns, or the 64-column pass (up to 32 columns with one 32-column block multiplied).
// The narrow kernel streams W once per 32 columns and fetches X per tile and wave; the pass shares X between four bands and
// streams W once, but cuts K into slices whose sums a second kernel adds.  Which one is an estimate of each in us:
//   narrow, a pass   4.9 (6.1 on bands of fewer than eight tiles, whose sums take the slow way) + the larger of 1.02 tile_us x tiles of a workgroup and W at 7.3 TB/s + 64 B of X per tile and column at 8.8 TB/s + the
//                    hand-over of pick_shares, 1.5 more where the shares of a band are not kept on one XCD
//   64 columns       5.05, 0.7 less without a body + for a round of workgroups (0.16 + 0.081 R) x tiles of its bodies (0.9 of it with one block) + 1.09 x
//                    the K tiles that fill no body, or W at 8 TB/s, whichever is larger (fourth powers added); with more than one slice 1.65 for the second
//                    kernel and the partial sums out and back at 4.35 TB/s
// fitted to 300 products (M 1024 ... 49152, K 1024 ... 49152, 60 - 90 %, both formats; rms 5.5 and 7.5 %).  Its pick takes 1.005 times the better one of
// the two, and 0.964 and 0.85 times what the pass for all calls of 33 - 64 and a rule on K and density for 17 - 32 columns took.  (Charging the second kernel
// to calls of one slice, which have none, and to bands of less than a body cost short bands up to half: 41216 x 160, N = 35 13.2 / 8.7, 29952 x
// 192, N = 50 14.8 / 10.3, 384 x 224, N = 57 14.0 / 9.7, 34944 x 448, N = 62 19.1 / 15.4; of 1200 drawn calls of 33 - 64 columns 180 take narrow passes with that charge, and 49 of
// these the pass without it, 1.14 times faster in the mean, one 1.15 times slower.)  Some of
// what was measured (us, narrow / 64-column): N = 64, 80 %: 1024 x 1024 16.3 / 15.0, 32768 x 1024
// 18.3 / 26.5, 8192 x 8192 35.2 / 35.4, 12288 x 12288 63.7 / 43.8; at 90 % 8192 x 8192 27.7 / 32.7 (and 16384 x 4096 26.4 / 32.5, where it picks the pass); N = 31: 8832 x 48736 at 90 %
// 62.6 / 51.9, 6272 x 13440 at 90 % 16.6 / 25.4, 16128 x 10400 at 80 % 29.6 / 43.5; N = 32, 27648 x 9216 at 70 % 62.5 / 58.4.
inline float words_bytes(uint32_t max_tile_words, uint32_t version, uint32_t bands, uint32_t KT) {  // from the longest tile: four deviations above the mean
  const float longest = version == 2u ? (float)max_tile_words * (4.f / 3.f) : (float)max_tile_words;
  const float mean = longest - 4.f * sqrtf(longest) > 0.5f * longest ? longest - 4.f * sqrtf(longest) : 0.5f * longest;
  return (float)bands * (float)KT * mean * (version == 2u ? 3.f : 4.f);
}
inline float narrow_us(float w_bytes, uint32_t rounds, uint32_t bands, uint32_t KT, uint32_t N, int cus) {
  float us = 0.f;
  for (uint32_t n0 = 0; n0 < N; n0 += N - n0 <= 16u ? 16u : kGroupCols) {
    const bool wide = N - n0 > 16u;
    const float tile = tile_us(rounds < 8u ? rounds : 8u, wide), T = (float)bands * (float)KT;
    const Shares s = pick_shares(bands, KT, cus, tile, wide);
    const uint32_t cols = N - n0 < kGroupCols ? N - n0 : kGroupCols;
    const float work = 1.02f * tile * T / (float)s.P, memory = w_bytes / 7.3e6f + T * (float)cols * 64.f / 8.8e6f;
    us += (KT < 8u ? 6.1f : 4.9f) + (work > memory ? work : memory);
    if (s.unit != 0u) us += hand_over_us(s.unit > 1u ? s.unit : s.P / bands + 1u, wide) + (s.unit > 1u ? 0.f : 1.5f);
  }
  return us;
}
inline float wide_us(float w_bytes, uint32_t rounds, uint32_t bands, uint32_t KT, uint32_t N, int cus) {  // N <= 64
  const uint32_t body = wide_body(rounds), quads = (bands + 3u) / 4u, S = wide_quad_slices(bands, 1u, KT, cus, rounds);
  const uint32_t bodies = (KT / body + S - 1u) / S, turns = (quads * S + (uint32_t)cus - 1u) / (uint32_t)cus;
  const float work = (float)(bodies * body) * (0.16f + 0.081f * (float)rounds) * (N <= kGroupCols ? 0.9f : 1.f) + 1.09f * (float)(KT % body);
  const float memory = w_bytes / 8.0e6f;
  float us = (KT < body ? 4.35f : 5.05f) + (float)turns * sqrtf(sqrtf(work * work * work * work + memory * memory * memory * memory));
  if (S > 1u) us += 1.65f + 0.07f * (float)(1u + S / 8u) + 2.f * (float)bands * (float)S * (N <= kGroupCols ? 16384.f : 32768.f) / 4.35e6f;
  return us;
}
// May a call of 17 - 32 columns take the 64-column pass at all?  The narrow kernel takes no offset to lie beyond the header's word count and
// the pass trusts TileOffsets, so only calls on long bands leave the narrow kernel, however the estimate falls: in version 1 bands of at least 384 K tiles, or 288 with
// tiles of more than two rounds and K slices that come out even (the longest at most a tenth above the mean); in version 2, which has variants with
// one block for tiles of up to four rounds only, bands of at least 1024.  (These are the calls that a rule on K and density gave to the pass before
// there was an estimate; it would take some on shorter bands too.  The line is there for the check, not for time.)
inline bool wide32_allowed(uint32_t need, uint32_t version, uint32_t bands, uint32_t KT, int cus) {
  if (version == 2u) return need <= 4u && KT >= 1024u;
  if (KT >= 384u) return true;
  if (KT < 288u || need <= 2u) return false;
  const uint32_t bodies = KT / wide_body(wide_rounds(need)), S = wide_quad_slices(bands, 1u, KT, cus, wide_rounds(need));
  return (uint64_t)((bodies + S - 1u) / S) * S * 10u <= (uint64_t)bodies * 11u;
}
// `rounds` of the variant that the pass would run.
inline bool wide_pays(uint32_t max_tile_words, uint32_t rounds, uint32_t version, uint32_t bands, uint32_t KT, uint32_t N, int cus) {
  const float w = words_bytes(max_tile_words, version, bands, KT);
  return 0.98f * wide_us(w, rounds, bands, KT, N, cus) < narrow_us(w, rounds, bands, KT, N, cus);
}

// Arguments of the 64-column passes (sparse and dense) and of the kernel that adds their K slices.
struct WideParams {
  const uint32_t* offs;   // TileOffsets (sparse pass)
  const uint32_t* words;  // NonZeros (sparse pass)
  const _Float16* W;      // dense matrix (dense pass)
  const _Float16* X;      // X as the caller lays it out, column-major K x N (sparse pass)
  const _Float16* Xp;     // X in fragment order: [K tile][column block of all N][lane][8 halves] (dense pass)
  _Float16* C;
  float* parts;           // [band][slice][column block][row block][lane] float4, used when S > 1
  uint32_t M, K, N, n0, KT, bands, S;
  Divisor by_S, by_G, by_groups;  // of S, G (block pass: of 8 x its column groups), groups of bands
  bool whole;  // whole_pairs: how workgroups spread over the XCDs (64-column passes)
  uint32_t G;  // groups of 64 columns in the launch, from column n0 on (sparse pass; 1 in the dense pass)
  uint32_t cb; // 32-column blocks of a group that are multiplied and hold sums (sparse pass: 2, or 1 for a call of at most 32 columns)
};

// What a call of the sparse product runs.
enum class SpmmPass : uint32_t { kNarrow, kWide, kBlock };  // passes of up to 32 columns; all columns in the 64-column pass; ... in the block pass
struct SpmmPlan {
  SpmmPass pass;
  uint32_t share;   // block pass: 1 or 2, else 0
  uint32_t rounds;  // rounds of a tile that the variant stages
  uint32_t slices;  // K slices (block and 64-column pass); narrow: 1 where the 64-column pass could run too, else 0
};
SpmmPlan spmm_plan(uint32_t max_tile_words, uint32_t version, uint32_t bands, uint32_t KT, uint32_t N, int cus, bool wide32);
hipError_t launch_spmm(const SpmmLaunch& a, hipStream_t stream);
// X -> xpack (fragment order, all N columns): the dense 64-column passes read it
hipError_t launch_xpack(const _Float16* X, _Float16* xpack, uint32_t K, uint32_t N, hipStream_t stream);
// all columns in the sparse 64-column pass, in the block pass
hipError_t launch_spmm_wide(const SpmmLaunch& a, const SpmmPlan& plan, hipStream_t stream);
hipError_t launch_spmm_block(const SpmmLaunch& a, const SpmmPlan& plan, hipStream_t stream);
// C = sum over the S slices of parts, in slice order (the second kernel of a 64-column pass with S > 1);
// layout32: the partial results are in the 32x32 accumulator layout (sparse pass), else 16x16 (dense pass)
hipError_t launch_wide_reduce(const WideParams& p, bool layout32, hipStream_t stream);
hipError_t launch_dense(const DenseLaunch& a, hipStream_t stream);
// header, TileOffsets and every tile whose words fit the capacity: one kernel
hipError_t launch_compress(const CompressLaunch& a, hipStream_t stream);
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t stream);
// all control words of a hand-over but the error word
hipError_t launch_lower_flags(uint32_t* flags, hipStream_t stream);

}  // namespace fls

// What fls_spmm (wide32 = 1) or fls_spmm_noalloc (wide32 = 0) runs for a blob of that longest tile and version on a GPU of
// that many CUs: out = pass, share, rounds, slices of SpmmPlan.  Host arithmetic only; for tests and the benchmark's
// label, not part of the C ABI.
extern "C" void fls_internal_spmm_plan(uint32_t max_tile_words, uint32_t version, uint32_t M, uint32_t K, uint32_t N, int cus, int wide32,
                                       uint32_t* out);

// What fls_dense_gemm of more than 32 columns launches first: out = groups of 64 columns, K slices.  As above.
extern "C" void fls_internal_dense_plan(uint32_t M, uint32_t K, uint32_t N, int cus, uint32_t* out);

// How the tiles of an M x K matrix are shared out in the passes of up to 32 columns: out = P, unit, grid of Shares.  As above.
extern "C" uint32_t fls_internal_divide(uint32_t n, uint32_t d);  // as the kernels divide
extern "C" void fls_internal_shares(uint32_t M, uint32_t K, int cus, float tile_us, int wide, uint32_t* out);
