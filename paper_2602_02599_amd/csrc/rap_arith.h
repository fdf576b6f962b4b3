// The pieces of librap's arithmetic and indexing that are our own and can go wrong silently: the
// rounding to bf16, the sine / cosine of the rotation angle, the first (software) half of the
// rounding to E4M3, and the rule that says which 16-byte loads of a cache tile are issued.  They
// are plain functions of their arguments, compiled for the device and for the host, so that the
// CPU tests run the very code the kernels run (tests/host/rap_arith_host.hip, under the host
// sanitizers).
#ifndef RAP_ARITH_H_
#define RAP_ARITH_H_

#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

namespace rap {

__host__ __device__ __forceinline__ uint32_t f32_bits(float f) { return __builtin_bit_cast(uint32_t, f); }
__host__ __device__ __forceinline__ float bits_f32(uint32_t u) { return __builtin_bit_cast(float, u); }

// bf16 bit pattern -> fp32 (a bf16 is the upper half of a binary32)
__host__ __device__ __forceinline__ float bf16_lo(uint32_t packed) { return bits_f32(packed << 16); }
__host__ __device__ __forceinline__ float bf16_hi(uint32_t packed) { return bits_f32(packed & 0xffff0000u); }
__host__ __device__ __forceinline__ float bf16_to_f32(uint16_t b) { return bits_f32(static_cast<uint32_t>(b) << 16); }

// fp64 -> bf16 with a single round-to-nearest-even.  The conversion to fp32 (nearest even) cannot
// carry a value across a bf16 rounding boundary, because every such boundary is an fp32 number; it
// can only land ON one (low half exactly 0x8000) from either side.  In that case the fp32 is
// moved one step back towards the side x came from, after which rounding the fp32 to its upper 16
// bits gives the correctly rounded result.
__host__ __device__ __forceinline__ uint16_t f64_to_bf16_rne(double x) {
  const float f = static_cast<float>(x);
  const uint32_t u0 = f32_bits(f);
  const double fd = static_cast<double>(f);
  uint32_t u = u0 + ((fabs(x) > fabs(fd)) ? 1u : 0u);               // sign-magnitude: +1 is away from zero
  u -= (fabs(x) < fabs(fd)) ? 1u : 0u;
  u = (u0 & 0xffffu) == 0x8000u ? u : u0;
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(x != x ? (u0 >> 16) | 0x40u : u >> 16);   // NaN stays NaN
}

// sin and cos of an fp64 angle, both within about 1.5e-16 of the true values for |phi| up to 2^31:
// the nearest multiple of pi/2 is taken off with two fused multiply-adds against a two-part pi/2
// (a fused multiply-add rounds once, after the cancellation), then Taylor polynomials up to
// r^15 / r^16 on |r| <= pi/4, whose first left-out terms are below 5e-17.  The library routine
// costs several times as much because it also covers angles beyond 2^31 with a table-driven
// reduction.  Only multiplications, fused multiply-adds and one rounding to integer: the host and
// the device compute the same bits.
__host__ __device__ __forceinline__ void sincos_f64(double phi, double* s, double* c) {
  const double k = rint(phi * 0.63661977236758134308);
  double r = fma(-k, 1.5707963267948965580e+00, phi);
  r = fma(-k, 6.1232339957367660359e-17, r);
  const double z = r * r;
  double ps = -1.0 / 1307674368000.0;                 // -1/15!
  ps = fma(ps, z, 1.0 / 6227020800.0);
  ps = fma(ps, z, -1.0 / 39916800.0);
  ps = fma(ps, z, 1.0 / 362880.0);
  ps = fma(ps, z, -1.0 / 5040.0);
  ps = fma(ps, z, 1.0 / 120.0);
  ps = fma(ps, z, -1.0 / 6.0);
  const double sr = fma(r * z, ps, r);
  double pc = 1.0 / 20922789888000.0;                 // 1/16!
  pc = fma(pc, z, -1.0 / 87178291200.0);
  pc = fma(pc, z, 1.0 / 479001600.0);
  pc = fma(pc, z, -1.0 / 3628800.0);
  pc = fma(pc, z, 1.0 / 40320.0);
  pc = fma(pc, z, -1.0 / 720.0);
  pc = fma(pc, z, 1.0 / 24.0);
  pc = fma(pc, z, -0.5);
  const double cr = fma(z, pc, 1.0);
  const long long n = static_cast<long long>(k) & 3;   // quadrant
  const double a = (n & 1) ? cr : sr, b = (n & 1) ? sr : cr;
  *s = (n & 2) ? -a : a;
  *c = ((n + 1) & 2) ? -b : b;
}

// First half of fp64 -> E4M3: the value, clamped to the largest E4M3 magnitude 448, brought to
// fp32 by ROUNDING TO ODD (truncate towards zero, then set the last mantissa bit if anything was
// cut off).  A value rounded to odd keeps every fact a later nearest-even rounding to a format at
// least two bits shorter needs, so the conversion instruction that follows on the device
// (fp32 -> E4M3, nearest even) yields the single correct rounding of the fp64 value.  NaN must be
// handled by the caller.
__host__ __device__ __forceinline__ float f64_to_f32_odd_clamped448(double y) {
  y = y > 448.0 ? 448.0 : (y < -448.0 ? -448.0 : y);
  const float f = static_cast<float>(y);            // nearest-even; repaired to round-to-odd below
  uint32_t bits = f32_bits(f);
  const double d = static_cast<double>(f);
  if (d != y) {
    if (fabs(d) > fabs(y)) bits -= 1u;              // went away from zero: step back to the truncation
    bits |= 1u;
  }
  return bits_f32(bits);
}

// ---- 4-bit caches: microscaling FP4 (E2M1 elements, one E8M0 scale byte per block of 32) --------
// E2M1 code (S.EE.M; magnitudes 0, 0.5, 1, 1.5, 2, 3, 4, 6) nearest to y, ties to the code with
// mantissa bit 0, magnitudes above 6 saturate.  The thresholds are the midpoints between
// neighbouring magnitudes, each closed on the side of its even neighbour.
__host__ __device__ __forceinline__ uint32_t f64_to_e2m1(double y) {
  const double a = y < 0 ? -y : y;
  const uint32_t c = a <= 0.25 ? 0u : a < 0.75 ? 1u : a <= 1.25 ? 2u : a < 1.75 ? 3u : a <= 2.5 ? 4u : a < 3.5 ? 5u : a <= 5.0 ? 6u : 7u;
  return c | ((__builtin_bit_cast(uint64_t, y) >> 63) != 0 ? 8u : 0u);
}

// Scale exponent of a block whose largest magnitude is amax (finite, not subnormal as a double):
// floor(log2 amax) - 2, so that amax / 2^e lies in [4, 8), the top binade of E2M1; limited to
// [-126, 127]; 0 for a block of zeros.  The scale byte is e + 127.
__host__ __device__ __forceinline__ int mx_shared_exponent(double amax) {
  if (!(amax > 0.0)) return 0;
  const int e = static_cast<int>((__builtin_bit_cast(uint64_t, amax) >> 52) & 0x7ff) - 1023 - 2;
  return e < -126 ? -126 : (e > 127 ? 127 : e);
}

// 2^(-e) for e in [-126, 127], exact
__host__ __device__ __forceinline__ double pow2_neg(int e) {
  return __builtin_bit_cast(double, static_cast<uint64_t>(1023 - e) << 52);
}

constexpr int mx_blocks(int d) { return (d + 31) / 32; }
// V channels a lane of the decode kernel takes over 4-bit caches: four while 16 lanes cover the row
// (two blocks) that way, else eight.
constexpr int mx4_lane_channels(int nb) { return nb <= 2 ? 4 : 8; }

// Which loads of a cache tile the decode kernel issues.  A tile (32 rows of any width: a multiple
// of 64 bytes for two-byte elements, of 32 for one-byte ones, 16-byte aligned) is fetched as n_ld
// wave-wide loads of 1 KB, lane l of load j taking bytes [1024 j + 16 l, + 16).  n_ld is fixed at
// compile time from the instantiation (KCH = ceil(d_k / 32) score steps; NT output tiles of 16
// channels: ceil(d_v / 16) for bf16 caches, blocks of 64 channels, i.e. 4 or 8 tiles, for one-byte
// codes) and can exceed the number of loads the tile needs by one whole load (bf16 K tiles: 2 KCH
// against ceil(d_k / 16); one-byte V tiles: NT / 2 against ceil(d_v / 32)).  The last n_trim loads
// are therefore trimmed to the tile by lane, all earlier ones are issued whole.  In a partial tile
// (the last rows of a sequence) every load is trimmed to the bytes of the rows that exist.
constexpr int decode_v_tiles(int d_v, bool q8) { return q8 ? 4 * ((d_v + 63) / 64) : (d_v + 15) / 16; }
constexpr int k_tile_loads(int kch, bool q8) { return q8 ? kch : 2 * kch; }
constexpr int v_tile_loads(int nt, bool q8) { return q8 ? (nt + 1) / 2 : nt; }
constexpr int k_tile_trimmed(bool q8) { return q8 ? 1 : 2; }
constexpr int v_tile_trimmed(bool q8) { return q8 ? 2 : 1; }
__host__ __device__ __forceinline__ bool tile_load_issued(int j, int lane, int n_ld, int n_trim, int bytes, bool whole_tile) {
  if (whole_tile && j < n_ld - n_trim) return true;
  return 1024 * j + 16 * lane < bytes;
}

// Which sequence, row range and KV head scanning workgroup `wg` of a decode launch takes:
// sequence by sequence, within a sequence range by range, the KV heads innermost.  Hardware places
// workgroup L on XCD L mod 8, so with eight KV heads (or a multiple) every XCD gets the same rows
// whatever the lengths are.  Measured against slab by slab with the ranges innermost, which leaves the
// XCDs' shares of a ragged batch to chance: 64 sequences of 1024 to 16384 rows in ranges of 4096 rows 296
// -> 268 us, 64 up to 65536 rows 994 -> 977 us, fp8 32 up to 16384 92 -> 88 us; equal lengths 32 x 16384
// 237 -> 232 us.
//  * Within an XCD the workgroups go round its compute units in turn, and in a ragged batch the first
//    ranges are the ones that hold rows: those of following sequences should lie an odd number of
//    workgroups apart.  With an odd number of ranges they do; an even number is rotated by the
//    sequence.  Rotating odd ones too put them an even number apart: 12 sequences up to 51691 rows, d =
//    64, 13 ranges, 173 us, not rotated 126; fp8, d = 90, 120 and 87 (equal lengths, d = 64, 210 and 226).
//    Not rotating even ones: 24 up to 32768, d = 64, 8 ranges, 197 us, rotated 178; fp8 100 and 79.
//    With fewer KV heads than XCDs the same keeps the first ranges off the same XCDs.
//  * With up to eight sequences no ranges are rotated, but the heads are, by range and sequence, so that
//    the ranges of a head meet all XCDs: 4 x 131072 rows at d = 64, where the heads lie a power of two
//    apart, 171.5 -> 167 us, 8 x 65536 175 -> 171.5.  From 12 to 16 sequences either way is the same to 1 %,
//    from 24 on rotated heads cost 1 % on equal lengths (32 x 16384 238 -> 240.5).
__host__ __device__ __forceinline__ void decode_place(int wg, int n_split, int n_kv, int batch, int* b, int* split, int* h) {
  const int seq_range = wg / n_kv;
  *b = seq_range / n_split;
  const int nth = seq_range - *b * n_split;
  const bool few = batch <= 8;
  *split = few || (n_split & 1) != 0 ? nth : (nth + *b) % n_split;
  *h = (wg - seq_range * n_kv + (few ? nth + *b : 0)) % n_kv;
}

// Ranges by length: the rows of a batch's sequences, counted in units of kSplitQuantum rows, are cut into ranges that are
// about as long as each other whatever the sequences' lengths, which only the device knows.  What the host can say:
// `wgs` ranges at most per KV head for sequences of unequal length (0: ranges are of a fixed length), `full` of each
// sequence where all are as long as they may be, `few` of each that the chip holds at once, and room for `slots` partials.
constexpr int kSplitQuantum = 128;   // rows_per_split granularity
struct FlatPlan {
  int wgs, slots, full, few;
};
// floor(a / b) for 0 <= a < 2^21 and b > 0, from 1 / b to within one unit in the last place: (a + 0.5) / b is 0.5 / b or more
// away from any whole number, and the product is off by less than 2^-22 of itself.  Five instructions, where the general
// division of 32-bit numbers takes twenty to thirty in a chain, which workgroups that look for their range wait for.
constexpr int kFlatDivLimit = 1 << 21;
__host__ __device__ __forceinline__ float flat_inverse(int b) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rcpf(static_cast<float>(b));
#else
  return 1.0f / static_cast<float>(b);
#endif
}
__host__ __device__ __forceinline__ int flat_div(int a, float inv_b) {
  return static_cast<int>((static_cast<float>(a) + 0.5f) * inv_b);
}
// Two workgroups per compute unit where that leaves two and a half or more per sequence; else as many as the chip holds
// (three per unit up to d_k = 96), else four per sequence.  Fixed ranges and these (lengths spread evenly from max / 16 to
// max): bf16 4 x 131072, d = 64, 163.2 -> 95.0 us, 7 x 125041, 4 KV heads, 154.5 -> 119.3, 10 x 30925 84.1 -> 70.6, 16 x 8192 42.3
// -> 38.5, 48 x 3000, 4 KV heads, 32.0 -> 26.2; fp8 40 x 7989, 4 KV heads, 41.8 -> 34.2; 4-bit 16 x 32768 77.6 -> 54.8.  In 384 /
// 448 / 512 workgroups: 4 x 131072 124 / 108 / 98 us, 16 x 8192 44 / 42 / 41; in 512 / 768 / 1536 / 2048: fp8 32 x 16384 85 /
// 81 / 83 / 83, bf16 64 x 16384 (one per sequence / ) 285 / 264 / 257.  As many as the partials' room holds where
// that is two or more times as many: 33 x 16384, half of them an eighth as long, 146 -> 140 us, but fp8 24 x 16384 57 -> 62
// to 70, 12 x 30000 50 -> 59.  Not for ranges of full sequences below 768 rows (1024 where the combining kernel has more to
// do): looking at the lengths costs both kernels some 0.5 us.  Over codes, whose rows are half as long or less, nor for ranges
// below 2048 rows that do not all start together, where every round of workgroups pays for that look.  Fixed ranges as they
// were before the lean loop / by length / fixed, fp8: 116/115, 24 x 4096 full 40.9 / 44.0 / 40.1, spread 28.4 / 26.4 / 26.8;
// d = 60, 40 x 4096 34.1 / 35.6 / 33.8 and 23.3 / 25.3 / 22.6; 48 x 3000 32.0 / 34.0 / 31.8 and 22.6 / 24.7 / 21.9; d = 90, 36 x 6000
// 64.6 / 66.2 / 64.1 and 42.6 / 39.3 / 40.0.  What starts together gains: d = 90, 24 x 4096 31.7 / 31.1 / 30.0 and 28.5 / 23.6 / 25.5.
inline FlatPlan flat_plan(int batch, int n_kv, int d_k, int n_split, int rows_per_split, int max_len, int n_tok, bool fused_step,
                          bool codes, int cus) {
  const int places = cus * (d_k <= 96 ? 3 : 2);
  const bool one_round = static_cast<long long>(batch) * n_kv * n_split <= places;
  int w = 2 * cus / n_kv;
  if (2 * w < 5 * batch) w = places / n_kv;
  if (2 * w < 5 * batch) w = 4 * batch;
  const int room = batch * (fused_step ? n_split : n_split + 1);
  if (w > room) w = room;
  const int len = max_len - (fused_step ? 1 : n_tok > 1 ? n_tok : 0);
  const int shortest = codes && !one_round ? 2048 : fused_step || n_tok > 1 ? 1024 : 768;
  FlatPlan p = {0, 0, 0, 0};
  if (n_split < 2 || rows_per_split < shortest || w < 2 * batch || len < 1) return p;
  const int units = (len + kSplitQuantum - 1) / kSplitQuantum, r = (units + n_split - 1) / n_split;
  if (static_cast<long long>(units) * (batch + 1) >= kFlatDivLimit / 2) return p;   // (134 M rows a KV head)
  p.wgs = w;
  p.full = (units + r - 1) / r;
  p.few = places / (n_kv * batch);
  p.slots = (w > batch * n_split ? w : batch * n_split) + (fused_step ? batch : 0);
  return p;
}
// Whether sequences of `total` units in all have as many ranges each, cut evenly: where they are shorter than the longest by an
// eighth at most on average.  Ranges of one length for all of them then come to two or three per sequence at the
// same time and leave the chip part idle.  One range length for all / as many ranges for each: 24 x 8192 rows, one
// sequence 128 rows shorter, 96.1 / 88.2 us, lengths in 0.9..1 89.0 / 85.4; 33 x 16384 279 / 243; fp8 36 x 16384 161 /
// 139.5.  Lengths in 0.5..1: 16 x 8192 49.1 / 48.3, 22 x 8192 66.3 / 66.1, 4 x 131072 179 / 181, 12 x 30000, 4 KV heads, 71.5 /
// 72.9, 64 x 16384 340 / 347.
__host__ __device__ __forceinline__ bool flat_alike(int total, int longest, int batch) {
  return 8LL * total >= 7LL * batch * longest;
}
// How many: as many as of full sequences, but none shorter than 8 units beyond what the chip holds at once.  64 sequences of
// 1024 rows of at most 16384, in 8 ranges 51.6 us, so 38.1; fp8 46.1 -> 26.6; 48 of 512 of at most 4096 24.2 -> 20.3.
__host__ __device__ __forceinline__ int flat_alike_ranges(int longest, int full, int few) {
  int n = longest / 8;
  n = n < few ? few : n;
  n = n < longest ? n : longest;
  return n < full ? (n > 0 ? n : 1) : full;
}
// Else the shortest range, of four units or more, that leaves no more than `most` of them (most > batch); count(r): how many
// ranges of up to r units there are.  One unit or more / four: one sequence of 4096 rows and 47 of 256, 21.9 / 17.9 us; one
// of 8192 and 15 of 512, 17.1 / 15.6, 21 of 512, 17.8 / 18.3.
constexpr int kFlatLeast = 4;
template <class Count>
__host__ __device__ __forceinline__ int flat_length(int total, int batch, int most, Count count) {
  // a sequence has one range that is not whole at most, so no longer ones than hi are needed
  int hi = flat_div(total, flat_inverse(most - batch)) + 1, r = flat_div(total + most - 1, flat_inverse(most));
  r = r < kFlatLeast ? kFlatLeast : r;
  while (r < hi) {
    const int mid = (r + hi) >> 1;
    if (count(mid) <= most) hi = mid;
    else r = mid + 1;
  }
  return r;
}
// The most ranges one sequence can have, of up to `units` units (a plan with wgs > 0).
inline int flat_most(const FlatPlan& p, int units) {
  const int n = (units + kFlatLeast - 1) / kFlatLeast, most = n < p.wgs ? n : p.wgs;
  return most > p.full ? most : p.full;
}
// First unit of piece `nth` of `n` that a sequence of `units` is cut into: the longer ones first.
__host__ __device__ __forceinline__ int flat_begin(int nth, int n, int units) {
  const int whole = units / n, more = units - whole * n;
  return nth * whole + (nth < more ? nth : more);
}

// Which query block and slab (sequence and KV head) workgroup `wg` of a prefill launch takes that is not cut into key
// ranges and whose workgroups do not all start together.
// Hardware places workgroup L on XCD L mod 8, each with an L2 of its own, and all query blocks of a slab
// read the same K and V rows: with a multiple of 8 slabs, all workgroups of a slab go to one XCD, which
// works on `group` of its slabs side by side, the heaviest query blocks (the last tokens, which see the
// most rows) of all of them first.  Else the heaviest blocks of all slabs come first.
// One slab after the other keeps the fewest rows in use, but a launch of few rounds then ends with the heavy
// blocks of its last slabs; all slabs at once end evenly, but outgrow the caches where they are long.
// One after the other / 8 at a time / all (n = context; 32/8 heads): d = 90, 8 x 1024 131 / 106 / 106 us, 8 x
// 2048 350 / 299 / 297, 16 x 4096 2308 / 2195 / 2179, 8 x 8192 4202 / 4152, 16 x 8192 8737 / 8682 / 8839; 8
// query heads, 8 x 2395 183 / 125 / 125; codes 8 x 2048 377 / 316 / 315.  Wide rows (three column blocks)
// with 4 / 8 / all: d = 128, 8 x 2048 426 one after the other, 411 / 403 / 402; 32 x 512 187, 181 / 187 / 197; 16 x
// 8192 11.4 ms, 11.1 / 11.5 / 12.2; 32 x 4096 6.32 ms, 5.89 / 6.01 / 6.87.
__host__ __device__ __forceinline__ void prefill_place(int wg, int n_qblk, int slabs, int group, int* qb, int* slab) {
  if ((slabs & 7) == 0) {
    const int x = wg >> 3, own = slabs >> 3;
    const int first = x / n_qblk / group * group;                                // of this XCD's slabs
    const int level = own - first < group ? own - first : group;                 // workgroups per query block number
    const int r = x - first * n_qblk;
    *qb = n_qblk - 1 - r / level;
    *slab = (first + r % level) * 8 + (wg & 7);
  } else {
    *slab = wg % slabs;
    *qb = n_qblk - 1 - wg / slabs;
  }
}

// Compute units of a whole MI355X.  How a prefill launch is cut and dealt out goes by this number and not by the device's, so
// that the workspace it asks for is a function of the shape alone; a device with fewer (a partition) gets the same results.
constexpr int kChipUnits = 256;

// A prefill launch cut into key ranges.  The rows a query block sees, in a sequence of max_len rows, are cut
// into ranges of `per` 64-row tiles and what is left over: with causal visibility the early blocks of a
// long chunk have fewer ranges than the late ones, and a block of one range needs no partials.
struct PrefillCut {
  int max_len, n_new, tok_per_wg, n_qblk, per;
};
constexpr int kPrefillTile = 64;
__host__ __device__ __forceinline__ int prefill_ranges(const PrefillCut& c, int qb) {
  const int tokens = (qb + 1) * c.tok_per_wg < c.n_new ? (qb + 1) * c.tok_per_wg : c.n_new;
  const int rows = c.max_len - c.n_new + tokens;
  return rows <= 0 ? 1 : ((rows + kPrefillTile - 1) / kPrefillTile + c.per - 1) / c.per;
}
// Query blocks with more than k ranges: the last ones.
__host__ __device__ __forceinline__ int prefill_blocks_beyond(const PrefillCut& c, int k) {
  // new tokens that row k * per * 64 is hidden from
  const long long hidden = static_cast<long long>(k) * c.per * kPrefillTile - (c.max_len - c.n_new);
  if (k == 0 || hidden <= 0) return c.n_qblk;
  return hidden >= c.n_new ? 0 : c.n_qblk - static_cast<int>(hidden) / c.tok_per_wg;
}
// Workgroups of one slab of such a launch.
__host__ __device__ __forceinline__ int prefill_cut_wgs(const PrefillCut& c) {
  const int k_max = prefill_ranges(c, c.n_qblk - 1);
  int n = 0;
  for (int k = 0; k < k_max; ++k) n += prefill_blocks_beyond(c, k);
  return n;
}
// Range r of a slab, counted through the first ranges of all blocks, the heaviest block first, then the second ones.
__host__ __device__ __forceinline__ void prefill_range(int r, const PrefillCut& c, int* qb, int* k) {
  // ranges that every block has lie in front of the new tokens
  const int shift = c.max_len - c.n_new, common = shift > 0 ? shift / (c.per * kPrefillTile) + 1 : 1;
  int range = r / c.n_qblk < common ? r / c.n_qblk : common;
  r -= range * c.n_qblk;
  if (range == common)
    for (int n = prefill_blocks_beyond(c, range); r >= n; n = prefill_blocks_beyond(c, range)) {
      r -= n;
      ++range;
    }
  *qb = c.n_qblk - 1 - r;
  *k = range;
}
// Tiles of a range.
__host__ __device__ __forceinline__ int prefill_range_tiles(const PrefillCut& c, int qb, int k) {
  const int tokens = (qb + 1) * c.tok_per_wg < c.n_new ? (qb + 1) * c.tok_per_wg : c.n_new;
  const int tiles = (c.max_len - c.n_new + tokens + kPrefillTile - 1) / kPrefillTile - k * c.per;
  return tiles < c.per ? tiles : c.per;
}
// Which range (counted from the longest) and slab workgroup `wg` of n * slabs takes; a slab stays on one XCD where they
// number a multiple of eight.  At most 512 workgroups, two per compute unit, start together, and the hardware deals
// them out in turn, one to every unit and then a second one: those 256 apart share a unit, so the longest are to be
// alone or with the shortest.  The first `both` and the last `both` share, the longest of all lie between.  More
// workgroups than that start longest first.  32/8 heads, d = 90, longest first and so: 2048 tokens, 384 workgroups of up
// to 16 tiles, 92.2 -> 74.5 us; not cut, 4096 tokens, 512 workgroups, 193.9 -> 185.7.
// inv: ceil(2^22 / own slabs), own = slabs or, where an XCD keeps its slabs, an eighth of them (n * own * own < 2^22).
__host__ __device__ __forceinline__ uint32_t prefill_inv(int slabs) {
  const uint32_t own = (slabs & 7) == 0 ? slabs >> 3 : slabs;
  return ((1u << 22) + own - 1) / own;
}
__host__ __device__ __forceinline__ void prefill_place_cut(int wg, int n, int slabs, uint32_t inv, int* nth, int* slab) {
  const bool own_xcd = (slabs & 7) == 0;
  const int shift = own_xcd ? 3 : 0, own = slabs >> shift, all = n * own, units = kChipUnits >> shift;
  int x = wg >> shift;
  if (all > units && all <= 2 * units) {
    const int both = all - units;
    x = x < both ? units - both + x : x < units ? x - both : all - 1 - (x - units);
  }
  *nth = static_cast<int>(static_cast<uint32_t>(x) * inv >> 22);
  *slab = ((x - *nth * own) << shift) + (own_xcd ? wg & 7 : 0);
}

// Which bytes of a cache tile the prefill kernel loads.  A tile is up to kPrefillTile rows of `pitch`
// bytes, fetched in 16-byte pieces from the start of every row; piece c of a tile is piece
// c % per_row of row c / per_row.  With `repeat` (loads straight into LDS, where per_row counts the
// 16-byte slots of a padded LDS row) the slots behind a row take its last piece again, so that in a
// whole tile every slot has something to load; else a slot behind the row loads nothing.
constexpr int kNoPiece = 0x7fffffff;
__host__ __device__ __forceinline__ int prefill_piece_offset(int c, int per_row, int pitch, bool repeat) {
  const int row = c / per_row;
  int piece = c - row * per_row;
  if (repeat) piece = piece < (pitch - 1) >> 4 ? piece : (pitch - 1) >> 4;
  return row < kPrefillTile && 16 * piece < pitch ? row * pitch + 16 * piece : kNoPiece;
}
// Whether the piece at such an offset, inside a tile whose readable rows make `bytes` bytes, is read
// whole; else only what is left of those.  A row's last piece runs on into the next row, at the last
// readable row into the rows behind it: those exist, eight of them or sixteen for one-byte
// elements, unless the cache ends there (prefill_rows_follow).
__host__ __device__ __forceinline__ bool prefill_piece_whole(int off, int bytes, bool rows_follow) {
  return rows_follow || bytes - off >= 16;
}
// Readable rows and capacities are multiples of eight (sixteen), so one row more is as many more.
__host__ __device__ __forceinline__ bool prefill_rows_follow(long long first_row, int rows, long long all_rows) {
  return first_row + rows < all_rows;
}

}  // namespace rap
#endif  // RAP_ARITH_H_
