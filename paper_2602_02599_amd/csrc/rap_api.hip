// C ABI of librap: host-side validation, split planning and kernel dispatch.  See include/rap.h
// for the contract of every entry point.  Each exported function fills a request record and hands
// it to one of the two shared bodies below (append_impl, decode_impl); nothing here allocates,
// synchronises or keeps state between calls (rap_decode_attn_static remembers, per device, where
// its scratch array lives).
#include <math.h>
#include <string.h>

#include <algorithm>

#include "../../include/rap.h"
#include "rap_device.h"

namespace rap {
hipError_t launch_append(const AppendArgs& a, hipStream_t stream);
hipError_t launch_rope_queries(const AppendArgs& a, hipStream_t stream);
hipError_t launch_decode_valu(const DecodeArgs& a, hipStream_t stream);
hipError_t launch_decode_mfma(const DecodeArgs& a, hipStream_t stream);
hipError_t launch_merge(const DecodeArgs& a, hipStream_t stream);
hipError_t launch_prefill(const PrefillArgs& a, hipStream_t stream);
hipError_t launch_prefill_merge(const PrefillArgs& a, hipStream_t stream);
hipError_t launch_stream_read(const void* src, size_t bytes, void* sink, hipStream_t stream);
hipError_t launch_stream_copy(void* dst, const void* src, size_t bytes, hipStream_t stream);
hipError_t launch_validate(const int32_t* pos, long long n_pos, long long cap, const int32_t* keep, int n_kv, int n_pairs,
                           int half, const int32_t* seq_lens, int batch, long long max_len, uint32_t* flags, hipStream_t stream);
int mfma_lds_wave_bytes(int d_k, int d_v, bool q8, int cols, bool mx4);
}  // namespace rap

namespace {

constexpr int kCUs = 256;                          // MI355X; what is assumed when no device can be asked
constexpr float kLog2e = 1.4426950408889634f;
constexpr int64_t kInt32Max = 0x7fffffffLL;

bool misaligned(const void* p, uintptr_t bytes) { return (reinterpret_cast<uintptr_t>(p) & (bytes - 1)) != 0; }

rap_status_t hip_status(hipError_t e) { return e == hipSuccess ? RAP_OK : RAP_ERR_HIP; }

rap_status_t check_shape(const rap_shape_t* s) {
  if (!s) return RAP_ERR_NULL;
  if (s->batch < 0 || s->n_q_heads <= 0 || s->n_kv_heads <= 0 || s->d_head <= 0 || (s->d_head & 1) ||
      s->n_pairs <= 0 || s->d_v <= 0 || s->cache_cap <= 0 || !(s->rope_theta > 0.0))
    return RAP_ERR_SHAPE;
  if (s->n_q_heads % s->n_kv_heads != 0) return RAP_ERR_SHAPE;
  if (s->n_pairs > s->d_head / 2) return RAP_ERR_SHAPE;
  if (s->cache_cap % 8 != 0) return RAP_ERR_SHAPE;
  if (s->n_pairs > rap::kMaxPairs || s->d_v > rap::kMaxDv || s->n_q_heads / s->n_kv_heads > rap::kMaxGroupWide)
    return RAP_ERR_UNSUPPORTED;
  if (s->cache_cap > kInt32Max - 1024 || s->batch > 65535 || s->n_kv_heads > 65535) return RAP_ERR_UNSUPPORTED;
  return RAP_OK;
}

// Exponent of the rotation frequencies: theta_j = 2^(j * this), Eq. (rope).
double neg2_log2_theta_over_d(const rap_shape_t* s) {
  return -2.0 * log2(s->rope_theta) / static_cast<double>(s->d_head);
}

// A rotation needs either the kept pair indices or the caller's frequency table.
bool no_rotation_rule(const rap_shape_t* s, const int32_t* keep_pair_idx) {
  return !keep_pair_idx && !s->pair_inv_freq;
}

struct Plan {
  int rows_per_split;
  int n_split;
  int kernel;   // 1 vector ALU, 2 matrix core
  bool flat;    // ranges by length, where the call allows them
};

// Compute units of the current device, asked once per device (256 on MI355X, which is also the
// answer when no device can be asked: the workspace query is host-only arithmetic).
int device_cus() {
  static std::atomic<int> known[rap::kMaxDevicesRemembered];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= rap::kMaxDevicesRemembered) return kCUs;
  int n = known[dev].load(std::memory_order_relaxed);
  if (n > 0) return n;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return kCUs;
  known[dev].store(n, std::memory_order_relaxed);
  return n;
}

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Bytes of that many partials: accumulators, then (reference, sum); and of those of n_split ranges (with
// the extra slot).
size_t slot_bytes(size_t slots, int d_v) {
  return align_up(slots * d_v * sizeof(float), 256) + align_up(slots * 2 * sizeof(float), 256) + 256;
}
size_t partial_bytes(const rap_shape_t* s, int n_split, int n_tok) {
  return slot_bytes(static_cast<size_t>(s->batch) * n_tok * s->n_q_heads * (n_split + 1), s->d_v);
}

int64_t round_to_quantum(int64_t r) { return (r + rap::kSplitQuantum - 1) / rap::kSplitQuantum * rap::kSplitQuantum; }

// What the host picks: rows of a range, a function of the shape, max_seq_len, the tuning and the device.  Ranges of that many
// rows are what a call gets with rows_per_split set, with the plain rule's workspace, with one sequence or more than 64, and
// where they are below 768 rows (FlatPlan); a workgroup whose range starts at or beyond its sequence's length exits at
// once.  Else the number of ranges comes from here and the device cuts the sequences by their lengths (FlatPlan), which
// makes the order of a row's sums depend on the other sequences' lengths as well.  Measured on MI355X (bf16, d = 90, 8 KV
// heads unless said otherwise, attention call in a graph; "ragged": lengths spread evenly from
// max / 16 to max, which the host cannot see; all with fixed ranges):
//  * A launch takes 6.9 us with one 128-row step per workgroup and 1.25 us more for each further
//    step; cutting into ranges adds a combining launch, 2.7 us.  So while one range per compute unit
//    is at most 512 rows, that is the range, if it spares three steps or more (1 x 2048 rows: 14.0 us
//    in ranges of 512, 10.5 in 128; 1 x 8192: 15.0 in 512, 13.5 in 256; 16 x 512: 13.2 in 256, 12.0
//    whole; 14 x 790, seven steps or four: 17.0 us whole, 15.7 in 512); and with a slab for every
//    compute unit up to 1024 rows stay whole (32 x 1024: 23.4 us in two ranges, 22.1 in one).
//  * Beyond that the chip wants at least two workgroups per compute unit, of 512 rows or more.
//    Where the slabs leave more than a fifth of that number over, more and shorter ranges that come
//    out even are better: 24 x 8192 (192 slabs) 102 us with 2 ranges per slab, 95 with 4; 40 x 4096
//    (320 slabs) 92 us with one, 80 with 4.  With less left over they are not: 18 x 8192 (144 slabs)
//    72 us with 3 ranges, 75 with 7; 14 x 9738 at 16 query rows per slab 74 us with 4, 78 with 9.
//    From 257 slabs on, where rows would be whole, three or more ranges (from 2048 rows): two are good
//    for equal lengths only (whole / 2 / 3 ranges: 40 x 3000 69 / 65 / 63 us, ragged 45 / 49 / 42;
//    fp8, d = 128, 48 x 3000 66 / 60 / 68, ragged 57 / 68 / 53; 44 x 2600 67 / 64 / 65, ragged 49 / 49 / 41).
//  * Long ranges save a little on equal lengths and cost a lot on ragged ones, whose workgroups are
//    then few and unequal: an eighth of max_seq_len, no less than 2048 and no more than 4096 rows.
//    64 x 16384: 451 / 456 / 464 us in 8192 / 4096 / 2048 rows, ragged 327 / 274 / 265; 32 x 16384
//    230 / 231 / 232, ragged 159 / 145 / 141; fp8 32 x 16384 137 / 147 / 137, ragged 117 / 89 / 87;
//    64 x 32768 892 / 902 / 931, ragged 539 / 520 / 515.  What equal lengths lose is most where rows
//    were whole or ranges few: 64 x 8192 in 4 ranges 234 us, whole 229, ragged 138 and 160; fp8 at d = 64
//    93 and 81, ragged 63 and 69; fp8 28 x 8192 75 us in 4, 69 in 2, ragged 49 and 66.  Hence not for
//    the sake of a little (112 slabs of 9738 rows: 73 us in 2560, 81 in 2048), nor of two ranges where rows
//    are whole (64 x 4096: 115 us whole, 121 in two, ragged 83 and 94); and into equal ranges (64 x 5000:
//    153 us in three of 1792, 161 in 2048 with a short third; whole 147; ragged 99, 102 and 108).
//  * Up to 16 sequences keep the plain rule's ranges of up to 8192 rows where those bring the job into a
//    single round.  In 8192 / 4096 / 2048 rows: 4 x 131072 228 / 231 / 236 us, at d = 64 171 / 175 / 174, fp8 130
//    / 147 / 133; 8 x 65536 229 / 231 / 234, 16 x 32768 229 / 228 / 230, fp8 131 / 146 / 130.  That is for
//    equal lengths; ragged batches pay for it: 4 x 131072 154 / 149 / 135 us, at d = 64 162 / 127 / 111; 8 x
//    65536 160 / 147 / 138; 16 x 32768 157 / 145 / 139, fp8 117 / 86 / 86.
//  * The plan never takes more partials than the static scratch array holds where the plain rule
//    (two workgroups per compute unit, ranges of 512 to 4096 rows, up to 8192 where that avoids a
//    partly filled second round of workgroups) would not, so that what a caller with that much
//    scratch may ask for does not depend on any of the above (64 x 16384, 64 query heads, d = 128 keep 4096
//    rows, 673 us, ragged 424; in 2048, 18 MB: 702 and 406).  Every call has to bring a workspace for
//    the plain rule (`plain`) and gets its ranges if the plan's do not fit in it.
//  * Several query tokens go by the same rule, though their partials count as often: 5 tokens, 24 query
//    heads, 32 x 16384 266 us, in 8192 rows 249; ragged 162 and 169.
rap_status_t make_plan(const rap_shape_t* s, int64_t max_seq_len, const rap_tuning_t* t, Plan* p, bool plain = false) {
  const int rps = t ? t->rows_per_split : 0;
  if (rps < 0 || (rps % rap::kSplitQuantum) != 0) return RAP_ERR_SHAPE;
  const int kernel = t ? t->kernel : 0;
  if (kernel < 0 || kernel > 2) return RAP_ERR_SHAPE;
  p->kernel = kernel == 0 ? 2 : kernel;
  p->flat = false;
  auto ranges_of = [&](int64_t rows) { return static_cast<int>((max_seq_len + rows - 1) / rows); };
  if (rps != 0) {
    p->rows_per_split = rps;
    p->n_split = ranges_of(rps);
    return RAP_OK;
  }
  const int64_t cus = device_cus();
  const int64_t slabs = s->batch > 0 ? static_cast<int64_t>(s->batch) * s->n_kv_heads : 1;
  const int64_t k0 = 2 * cus / slabs > 1 ? 2 * cus / slabs : 1;                // ranges per slab, plain rule
  const int64_t halves = round_to_quantum((max_seq_len + k0 - 1) / k0);
  int64_t r = halves < 512 ? 512 : (halves > 4096 ? 4096 : halves);
  // workgroups the chip holds at once: three per compute unit up to d_k = 96, else two (narrow instantiations leave room for
  // four, decode_waves; the rule's figures are with three)
  const int64_t places = cus * (2 * s->n_pairs <= 96 ? 3 : 2);
  const int64_t n_wg = slabs * ((max_seq_len + r - 1) / r);
  const bool single_round = n_wg > places && n_wg < 2 * places && halves <= 8192;
  if (single_round) r = halves;
  p->rows_per_split = static_cast<int>(r);
  p->n_split = ranges_of(r);
  if (plain) return RAP_OK;

  const int64_t k1 = cus / slabs > 1 ? cus / slabs : 1;                        // ranges per slab with one workgroup per compute unit
  const int64_t per_cu = round_to_quantum((max_seq_len + k1 - 1) / k1);
  if (per_cu <= 512 && slabs <= cus) {
    r = round_to_quantum(max_seq_len) - per_cu >= 3 * rap::kSplitQuantum ? per_cu : round_to_quantum(max_seq_len);
  } else if (slabs >= cus && max_seq_len <= 1024) {
    r = round_to_quantum(max_seq_len);
  } else {
    auto rows_in = [&](int64_t c) { return round_to_quantum((max_seq_len + c - 1) / c); };
    // how evenly c ranges per slab fill the compute units, less a little for every further range
    auto evenness = [&](int64_t c) {
      const int64_t n = slabs * c, rounds = (n + cus - 1) / cus;
      return static_cast<double>(n) / static_cast<double>(rounds * cus) - 0.03 * static_cast<double>(c - k0) / static_cast<double>(k0);
    };
    int64_t k = k0;
    if (evenness(k0) < 0.78) {
      auto long_enough = [&](int64_t c) { return max_seq_len >= (k0 > 1 ? 1024 * c : c == 3 ? 2048 : 768 * c); };
      for (int64_t c = k0 == 1 ? 3 : k0 + 1; c <= 4 * k0 && long_enough(c); ++c)
        if (evenness(c) > evenness(k) + 0.02) k = c;
    }
    const int64_t eighth = round_to_quantum(max_seq_len / 8);
    const int64_t most = eighth < 2048 ? 2048 : (eighth > 4096 ? 4096 : eighth);
    r = rows_in(k);
    if (r > (k == 1 ? 2 * most : most + most / 2)) r = rows_in((max_seq_len + most - 1) / most);
    if (r < 512) r = 512;
    if (single_round && s->batch <= 16) r = halves;
  }
  if (ranges_of(r) > p->n_split && partial_bytes(s, ranges_of(r), 1) > RAP_STATIC_SCRATCH_BYTES) return RAP_OK;   // plain
  p->rows_per_split = static_cast<int>(r);
  p->n_split = ranges_of(r);
  p->flat = p->kernel == 2 && s->batch > 1 && s->batch <= rap::kWave;
  return RAP_OK;
}

// Workspace = accumulators [B, H_q, n_split + 1, d_v], then (reference, sum) pairs
// [B, H_q, n_split + 1, 2], fp32, each block rounded up to 256 bytes; the extra slot is the new
// token's in the one-call step.  (Ranges by length lay the same room out by KV head.)
// With n_tok query tokens per sequence there are n_tok times as many query rows.
size_t part_acc_bytes(const rap_shape_t* s, const Plan& p, int n_tok = 1) {
  return align_up(static_cast<size_t>(s->batch) * n_tok * s->n_q_heads * (p.n_split + 1) * s->d_v * sizeof(float), 256);
}
size_t workspace_need(const rap_shape_t* s, const Plan& p, int n_tok = 1) { return partial_bytes(s, p.n_split, n_tok); }

// What one call can use: the plan's partials, no less than the plain rule's, which every call has to
// bring; 0 for arguments that no call accepts.
size_t call_workspace_bytes(const rap_shape_t* shape, int64_t max_seq_len, const rap_tuning_t* tuning) {
  Plan p, base;
  if (check_shape(shape) != RAP_OK || max_seq_len < 1 || max_seq_len > shape->cache_cap) return 0;
  if (make_plan(shape, max_seq_len, tuning, &p) != RAP_OK || make_plan(shape, max_seq_len, tuning, &base, true) != RAP_OK) return 0;
  return std::max(workspace_need(shape, p), workspace_need(shape, base));
}

// page_rows a power of two in [32, 65536], table present, logical capacity consistent
rap_status_t check_paging(const rap_shape_t* s, const rap_paging_t* pg, int* shift) {
  if (!pg) return RAP_ERR_NULL;
  if (pg->page_rows < 32 || pg->page_rows > 65536 || (pg->page_rows & (pg->page_rows - 1)) != 0) return RAP_ERR_SHAPE;
  if (pg->n_pages <= 0 || pg->max_pages <= 0) return RAP_ERR_SHAPE;
  if (static_cast<int64_t>(pg->max_pages) * pg->page_rows != s->cache_cap) return RAP_ERR_SHAPE;
  if (s->batch > 0 && !pg->block_table) return RAP_ERR_NULL;
  int sh = 0;
  while ((1 << sh) < pg->page_rows) ++sh;
  *shift = sh;
  return RAP_OK;
}

// ---- append ---------------------------------------------------------------------------------

struct AppendRequest {
  const rap_shape_t* shape = nullptr;
  const rap_paging_t* paging = nullptr;    // paged pools instead of dense caches
  int32_t n_new = 0;
  const void* k_new = nullptr;
  const void* v_new = nullptr;
  const int32_t* pos = nullptr;
  const int32_t* keep_pair_idx = nullptr;
  void* k_cache = nullptr;
  void* v_cache = nullptr;
  bool fp8 = false;                        // caches hold E4M3 codes, scales required
  const float* k_scale = nullptr;
  const float* v_scale = nullptr;
  void* k_scales4 = nullptr;               // 4-bit caches: k_cache / v_cache hold the code blocks, these the scale bytes
  void* v_scales4 = nullptr;
  bool mx4 = false;
  void* stream = nullptr;
};

// Shared body of rap_rope_append and its paged, fp8 and 4-bit variants.
rap_status_t append_impl(const AppendRequest& r) {
  const rap_shape_t* shape = r.shape;
  rap_status_t st = check_shape(shape);
  if (st != RAP_OK) return st;
  int page_shift = 0;
  if (r.paging && (st = check_paging(shape, r.paging, &page_shift)) != RAP_OK) return st;
  if (r.n_new < 0) return RAP_ERR_SHAPE;
  if (r.n_new == 0 || shape->batch == 0) return RAP_OK;
  if (!r.k_new || !r.v_new || !r.pos || no_rotation_rule(shape, r.keep_pair_idx) || !r.k_cache || !r.v_cache)
    return RAP_ERR_NULL;
  if (static_cast<int64_t>(shape->batch) * r.n_new > kInt32Max) return RAP_ERR_UNSUPPORTED;
  if (misaligned(r.k_new, 4) || misaligned(r.v_new, 4) || misaligned(r.k_cache, 4) || misaligned(r.v_cache, 4))
    return RAP_ERR_SHAPE;
  rap::AppendArgs a;
  memset(&a, 0, sizeof(a));
  if (r.paging) {
    a.block_table = r.paging->block_table;
    a.page_shift = page_shift;
    a.n_pages = r.paging->n_pages;
    a.max_pages = r.paging->max_pages;
  }
  if (r.fp8) {
    if (!r.k_scale || !r.v_scale) return RAP_ERR_NULL;
    if (shape->cache_cap % 16 != 0) return RAP_ERR_SHAPE;
    a.k_scale = r.k_scale;
    a.v_scale = r.v_scale;
  }
  if (r.mx4) {
    if (!r.k_scales4 || !r.v_scales4) return RAP_ERR_NULL;
    if (r.paging || r.fp8) return RAP_ERR_UNSUPPORTED;
    if (misaligned(r.k_cache, 16) || misaligned(r.v_cache, 16) || misaligned(r.k_scales4, 4) || misaligned(r.v_scales4, 4))
      return RAP_ERR_SHAPE;
    a.k_scales4 = static_cast<uint8_t*>(r.k_scales4);
    a.v_scales4 = static_cast<uint8_t*>(r.v_scales4);
  }
  a.k_new = static_cast<const uint16_t*>(r.k_new);
  a.v_new = static_cast<const uint16_t*>(r.v_new);
  a.pos = r.pos;
  a.keep = r.keep_pair_idx;
  a.pair_freq = shape->pair_inv_freq;
  a.k_cache = static_cast<uint16_t*>(r.k_cache);
  a.v_cache = static_cast<uint16_t*>(r.v_cache);
  a.batch = shape->batch;
  a.n_new = r.n_new;
  a.n_kv = shape->n_kv_heads;
  a.d_head = shape->d_head;
  a.n_pairs = shape->n_pairs;
  a.d_v = shape->d_v;
  a.group = 1;
  a.cap = shape->cache_cap;
  a.neg2_log2_theta_over_d = neg2_log2_theta_over_d(shape);
  return hip_status(rap::launch_append(a, static_cast<hipStream_t>(r.stream)));
}

// ---- decode attention -------------------------------------------------------------------------

struct DecodeRequest {
  const rap_shape_t* shape = nullptr;
  const rap_paging_t* paging = nullptr;    // paged pools instead of dense caches
  const void* q = nullptr;
  const int32_t* q_pos = nullptr;          // non-null: q arrives un-rotated and is rotated in the prologue
  const int32_t* keep_pair_idx = nullptr;
  const void* k_cache = nullptr;
  const void* v_cache = nullptr;
  bool fp8 = false;                        // caches hold E4M3 codes, scales required
  const float* k_scale = nullptr;
  const float* v_scale = nullptr;
  const void* k_scales4 = nullptr;         // 4-bit caches: k_cache / v_cache hold the code blocks, these the scale bytes
  const void* v_scales4 = nullptr;
  bool mx4 = false;
  const void* k_new = nullptr;             // one-call step: the token to append first (with v_new, new_pos)
  const void* v_new = nullptr;
  const int32_t* new_pos = nullptr;
  int32_t n_tok = 1;                       // query tokens per sequence: the last n_tok rows, already appended
  const int32_t* seq_lens = nullptr;
  int64_t max_seq_len = 0;
  void* out = nullptr;
  float scale = 0.f;
  void* workspace = nullptr;
  size_t workspace_bytes = 0;
  const rap_tuning_t* tuning = nullptr;
  void* stream = nullptr;
};

// Shared body of rap_decode_attn, rap_decode_attn_rope, the paged and fp8 variants,
// rap_decode_step and rap_decode_attn_multi.
rap_status_t decode_impl(const DecodeRequest& r) {
  const rap_shape_t* shape = r.shape;
  rap_status_t st = check_shape(shape);
  if (st != RAP_OK) return st;
  int page_shift = 0;
  if (r.paging && (st = check_paging(shape, r.paging, &page_shift)) != RAP_OK) return st;
  if (r.max_seq_len < 1) return RAP_ERR_SHAPE;
  if (r.max_seq_len > shape->cache_cap) return RAP_ERR_CAPACITY;
  if (shape->batch == 0) return RAP_OK;
  const bool step = r.k_new || r.v_new || r.new_pos;
  const bool multi = r.n_tok > 1;
  if (r.n_tok < 1) return RAP_ERR_SHAPE;
  if (!r.q || !r.k_cache || !r.v_cache || !r.seq_lens || !r.out) return RAP_ERR_NULL;
  if (step && (!r.k_new || !r.v_new || !r.new_pos)) return RAP_ERR_NULL;
  if ((r.q_pos || step) && no_rotation_rule(shape, r.keep_pair_idx)) return RAP_ERR_NULL;
  if (misaligned(r.k_cache, 16) || misaligned(r.v_cache, 16) || misaligned(r.q, 4) || misaligned(r.out, 4))
    return RAP_ERR_SHAPE;
  Plan p;
  st = make_plan(shape, r.max_seq_len, r.tuning, &p);
  if (st != RAP_OK) return st;
  // the one-call step on the matrix-core kernel hands the new token to the combining kernel, which
  // therefore always runs
  const bool fused_step = step && p.kernel == 2;
  // several query tokens: their rows are the columns of the matrix instruction, 16 at most, and
  // the part among the tokens themselves is added by the combining kernel, which always runs
  if (multi && (p.kernel != 2 || step || r.q_pos ||
                static_cast<int64_t>(r.n_tok) * (shape->n_q_heads / shape->n_kv_heads) > 16))
    return RAP_ERR_UNSUPPORTED;
  // What a call must hand in is what the plain rule needs, so that whether it is accepted does not
  // hang on the plan; a workspace that holds no more than that gets the plain rule's ranges.
  Plan base;
  st = make_plan(shape, r.max_seq_len, r.tuning, &base, true);
  if (st != RAP_OK) return st;
  auto combines = [&](const Plan& q) { return q.n_split > 1 || fused_step || multi; };
  auto holds = [&](const Plan& q) {
    return r.workspace && !misaligned(r.workspace, 256) && r.workspace_bytes >= workspace_need(shape, q, r.n_tok);
  };
  if (combines(base) && !holds(base)) return RAP_ERR_WORKSPACE;
  if (combines(p) && !holds(p)) p = base;
  const bool combine = combines(p);
  if (p.n_split > 65535 || (static_cast<int64_t>(p.n_split) + 1) * shape->n_kv_heads * shape->batch > kInt32Max)
    return RAP_ERR_UNSUPPORTED;
  // combinations no kernel is built for
  if ((r.fp8 || r.paging) && p.kernel != 2) return RAP_ERR_UNSUPPORTED;   // the vector-ALU kernel reads dense bf16 caches only
  // more than 8 query heads per KV head: the matrix-core kernel with rotated queries only
  if (shape->n_q_heads / shape->n_kv_heads > rap::kMaxGroup && (p.kernel != 2 || step || r.q_pos)) return RAP_ERR_UNSUPPORTED;
  if (r.fp8) {
    if (shape->cache_cap % 16 != 0) return RAP_ERR_SHAPE;
    if (!r.k_scale || !r.v_scale) return RAP_ERR_NULL;
  }
  if (r.mx4) {
    // 4-bit caches: the plain attention call on the matrix-core kernel over dense caches
    if (!r.k_scales4 || !r.v_scales4) return RAP_ERR_NULL;
    if (p.kernel != 2 || r.fp8 || r.paging || step || multi || r.q_pos) return RAP_ERR_UNSUPPORTED;
    if (misaligned(r.k_scales4, 4) || misaligned(r.v_scales4, 4)) return RAP_ERR_SHAPE;
  }

  rap::DecodeArgs a;
  memset(&a, 0, sizeof(a));
  a.q = static_cast<const uint16_t*>(r.q);
  a.q_pos = r.q_pos;
  a.keep = r.keep_pair_idx;
  a.pair_freq = shape->pair_inv_freq;
  a.neg2_log2_theta_over_d = neg2_log2_theta_over_d(shape);
  a.d_head = shape->d_head;
  a.k_cache = static_cast<const uint16_t*>(r.k_cache);
  a.v_cache = static_cast<const uint16_t*>(r.v_cache);
  a.seq_lens = r.seq_lens;
  a.out = static_cast<float*>(r.out);
  a.part_acc = static_cast<float*>(r.workspace);
  a.part_ml = r.workspace ? reinterpret_cast<float*>(static_cast<char*>(r.workspace) + part_acc_bytes(shape, p, r.n_tok)) : nullptr;
  a.n_tok = r.n_tok;
  a.group_inv16 = (65536 + (shape->n_q_heads / shape->n_kv_heads) - 1) / (shape->n_q_heads / shape->n_kv_heads);
  a.batch = shape->batch;
  a.n_q = shape->n_q_heads;
  a.n_kv = shape->n_kv_heads;
  a.group = shape->n_q_heads / shape->n_kv_heads;
  a.n_pairs = shape->n_pairs;
  a.d_k = 2 * shape->n_pairs;
  a.d_v = shape->d_v;
  a.max_len = static_cast<int32_t>(r.max_seq_len);
  a.rows_per_split = p.rows_per_split;
  a.n_split = p.n_split;
  a.n_slots = fused_step ? p.n_split + 1 : p.n_split;
  a.cap = shape->cache_cap;
  a.scale_log2e = r.scale * kLog2e;
  a.lds_wave_bytes = rap::mfma_lds_wave_bytes(a.d_k, a.d_v, r.fp8, r.n_tok * a.group, r.mx4);
  a.k_scales4 = r.mx4 ? static_cast<const uint8_t*>(r.k_scales4) : nullptr;
  a.v_scales4 = r.mx4 ? static_cast<const uint8_t*>(r.v_scales4) : nullptr;
  a.k_scale = r.fp8 ? r.k_scale : nullptr;
  a.v_scale = r.fp8 ? r.v_scale : nullptr;
  if (r.paging) {
    a.block_table = r.paging->block_table;
    a.page_shift = page_shift;
    a.n_pages = r.paging->n_pages;
    a.max_pages = r.paging->max_pages;
  }
  a.direct_out = combine ? 0 : 1;
  if (fused_step) {
    a.k_new = static_cast<const uint16_t*>(r.k_new);
    a.v_new = static_cast<const uint16_t*>(r.v_new);
    a.new_pos = r.new_pos;
    a.k_cache_w = static_cast<uint16_t*>(const_cast<void*>(r.k_cache));
    a.v_cache_w = static_cast<uint16_t*>(const_cast<void*>(r.v_cache));
  }

  if (p.flat && combine) {
    const rap::FlatPlan f = rap::flat_plan(a.batch, a.n_kv, a.d_k, a.n_split, a.rows_per_split, a.max_len, a.n_tok, fused_step,
                                           a.k_scale != nullptr || a.k_scales4 != nullptr, device_cus());
    a.flat_wgs = f.wgs;
    a.flat_slots = f.slots;
    a.flat_full = f.full;
    a.flat_few = f.few;
  }
  hipStream_t s = static_cast<hipStream_t>(r.stream);
  if (step && !fused_step) {
    // vector-ALU kernel: the append is a launch of its own ahead of the attention
    AppendRequest ar;
    ar.shape = shape;
    ar.n_new = 1;
    ar.k_new = r.k_new;
    ar.v_new = r.v_new;
    ar.pos = r.new_pos;
    ar.keep_pair_idx = r.keep_pair_idx;
    ar.k_cache = const_cast<void*>(r.k_cache);
    ar.v_cache = const_cast<void*>(r.v_cache);
    ar.stream = r.stream;
    if ((st = append_impl(ar)) != RAP_OK) return st;
  }
  const rap_tuning_t* t = r.tuning;
  if (t && t->ev_main_start && hipEventRecord(static_cast<hipEvent_t>(t->ev_main_start), s) != hipSuccess)
    return RAP_ERR_HIP;
  const hipError_t e = p.kernel == 1 ? rap::launch_decode_valu(a, s) : rap::launch_decode_mfma(a, s);
  if (e != hipSuccess) return RAP_ERR_HIP;
  if (t && t->ev_main_stop && hipEventRecord(static_cast<hipEvent_t>(t->ev_main_stop), s) != hipSuccess)
    return RAP_ERR_HIP;
  if (combine && rap::launch_merge(a, s) != hipSuccess) return RAP_ERR_HIP;
  return RAP_OK;
}

// ---- scratch for the entry point that allocates nothing ------------------------------------------
// The array lives in the device image of the library: each GPU holds its own copy at its own
// address.  On the host its name is only a handle for hipGetSymbolAddress, never a device address;
// kernels get the looked-up pointer as an argument, like any caller's workspace.
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[RAP_STATIC_SCRATCH_BYTES];

std::atomic<void*> g_scratch_ptr[rap::kMaxDevicesRemembered];

// Address of `scratch` on the current device, looked up once per device.
rap_status_t static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= rap::kMaxDevicesRemembered) return RAP_ERR_HIP;
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (ptr == nullptr) {
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return RAP_ERR_HIP;
    g_scratch_ptr[dev].store(ptr, std::memory_order_release);   // a lost race between host threads repeats the lookup
  }
  *out = ptr;
  return RAP_OK;
}

// rap_decode_attn_rope and its relatives take q_pos and keep_pair_idx as a pair: an argument the
// call needs and does not get is RAP_ERR_NULL, but only once the shape itself has passed.
rap_status_t null_after_shape(const rap_shape_t* shape) {
  const rap_status_t st = check_shape(shape);
  return st != RAP_OK ? st : RAP_ERR_NULL;
}

bool live_call(const rap_shape_t* shape, int64_t max_seq_len) { return shape && shape->batch > 0 && max_seq_len >= 1; }

// ---- prefill attention ----------------------------------------------------------------------------

// Shared body of rap_prefill_attn, rap_prefill_attn_paged and rap_prefill_attn_ex (k_scale and
// v_scale non-null: the caches hold E4M3 codes).
// Workspace of the prefill attention with key ranges: partial accumulators [B * n_new * H_q,
// ranges, d_v] and (reference, sum) pairs, fp32, each block rounded up to 256 bytes; nothing
// when the launch is never split.  It has room for plan.slots ranges, of which a launch uses n_ksplit.
size_t prefill_part_acc_bytes(const rap_shape_t* s, int32_t n_new, int ranges) {
  return align_up(static_cast<size_t>(s->batch) * n_new * s->n_q_heads * ranges * s->d_v * sizeof(float), 256);
}
size_t prefill_workspace_need(const rap_shape_t* s, int32_t n_new, const rap::PrefillPlan& p) {
  if (p.slots <= 1) return 0;
  return prefill_part_acc_bytes(s, n_new, p.slots) +
         align_up(static_cast<size_t>(s->batch) * n_new * s->n_q_heads * p.slots * 2 * sizeof(float), 256) + 256;
}
rap::PrefillPlan prefill_plan_of(const rap_shape_t* s, int32_t n_new, int64_t max_seq_len) {
  return rap::prefill_plan(s->batch, s->n_kv_heads, s->n_q_heads / s->n_kv_heads, 2 * s->n_pairs, s->d_v, n_new,
                           static_cast<int>(max_seq_len));
}

// `split`: the caller offers a workspace, so a launch whose query blocks would not fill the chip
// is cut into key ranges as well and combined by a second launch.
rap_status_t prefill_impl(const rap_shape_t* shape, const rap_paging_t* paging, int32_t n_new, const void* q,
                          const void* k_cache, const void* v_cache, const int32_t* seq_lens, int64_t max_seq_len,
                          void* out, float scale, void* stream, const float* k_scale = nullptr,
                          const float* v_scale = nullptr, bool split = false, void* workspace = nullptr,
                          size_t workspace_bytes = 0) {
  rap_status_t st = check_shape(shape);
  if (st != RAP_OK) return st;
  if ((k_scale == nullptr) != (v_scale == nullptr)) return RAP_ERR_NULL;
  if (k_scale && shape->cache_cap % 16 != 0) return RAP_ERR_SHAPE;
  int page_shift = 0;
  if (paging) {
    if ((st = check_paging(shape, paging, &page_shift)) != RAP_OK) return st;
    if (paging->page_rows < 64) return RAP_ERR_UNSUPPORTED;     // a 64-row tile must not straddle pages
  }
  if (n_new < 0 || max_seq_len < 1) return RAP_ERR_SHAPE;
  if (max_seq_len > shape->cache_cap) return RAP_ERR_CAPACITY;
  if (n_new == 0 || shape->batch == 0) return RAP_OK;
  if (!q || !k_cache || !v_cache || !seq_lens || !out) return RAP_ERR_NULL;
  if (misaligned(k_cache, 16) || misaligned(v_cache, 16) || misaligned(q, 4) || misaligned(out, 4)) return RAP_ERR_SHAPE;
  if (static_cast<int64_t>(shape->batch) * n_new > kInt32Max) return RAP_ERR_UNSUPPORTED;
  rap::PrefillPlan plan = prefill_plan_of(shape, n_new, max_seq_len);
  if (!split) plan.slots = plan.n_ksplit = 1;
  if (plan.slots > 1) {
    if (!workspace || workspace_bytes < prefill_workspace_need(shape, n_new, plan) || misaligned(workspace, 256))
      return RAP_ERR_WORKSPACE;
    if (static_cast<int64_t>(shape->batch) * n_new * shape->n_q_heads > kInt32Max) return RAP_ERR_UNSUPPORTED;
  }
  rap::PrefillArgs a;
  memset(&a, 0, sizeof(a));
  a.q = static_cast<const uint16_t*>(q);
  a.k_cache = static_cast<const uint16_t*>(k_cache);
  a.v_cache = static_cast<const uint16_t*>(v_cache);
  a.seq_lens = seq_lens;
  a.out = static_cast<float*>(out);
  a.batch = shape->batch;
  a.n_new = n_new;
  a.n_q = shape->n_q_heads;
  a.n_kv = shape->n_kv_heads;
  a.group = shape->n_q_heads / shape->n_kv_heads;
  a.d_k = 2 * shape->n_pairs;
  a.d_v = shape->d_v;
  a.max_len = static_cast<int32_t>(max_seq_len);
  a.cap = shape->cache_cap;
  a.scale_log2e = scale * kLog2e;
  a.k_scale = k_scale;
  a.v_scale = v_scale;
  if (paging) {
    a.block_table = paging->block_table;
    a.page_shift = page_shift;
    a.n_pages = paging->n_pages;
    a.max_pages = paging->max_pages;
  }
  if (plan.slots > 1)
    rap::prefill_cut_plan(&plan, a.n_kv * a.batch, a.group, a.d_k, a.d_v, n_new, a.max_len, a.order);
  a.n_ksplit = plan.n_ksplit;
  a.as_combined = plan.slots > 1;
  if (plan.n_ksplit > 1) {
    a.n_ranges = plan.n_ranges;
    a.tiles_per_split = plan.tiles_per_split;
    a.tok_per_wg = plan.tok_per_wg;
    a.n_qblk = plan.n_qblk;
    a.part_acc = static_cast<float*>(workspace);
    a.part_ml = reinterpret_cast<float*>(static_cast<char*>(workspace) + prefill_part_acc_bytes(shape, n_new, plan.n_ksplit));
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (rap::launch_prefill(a, s) != hipSuccess) return RAP_ERR_HIP;
  if (plan.n_ksplit > 1) {
    if (rap::launch_prefill_merge(a, s) != hipSuccess) return RAP_ERR_HIP;
  }
  return RAP_OK;
}

}  // namespace

extern "C" {

rap_status_t rap_rope_append(const rap_shape_t* shape, int32_t n_new, const void* k_new, const void* v_new,
                             const int32_t* pos, const int32_t* keep_pair_idx, void* k_cache, void* v_cache,
                             void* stream) {
  AppendRequest r;
  r.shape = shape;
  r.n_new = n_new;
  r.k_new = k_new;
  r.v_new = v_new;
  r.pos = pos;
  r.keep_pair_idx = keep_pair_idx;
  r.k_cache = k_cache;
  r.v_cache = v_cache;
  r.stream = stream;
  return append_impl(r);
}

rap_status_t rap_rope_append_paged(const rap_shape_t* shape, const rap_paging_t* paging, int32_t n_new,
                                   const void* k_new, const void* v_new, const int32_t* pos,
                                   const int32_t* keep_pair_idx, void* k_pool, void* v_pool, void* stream) {
  if (!paging) return RAP_ERR_NULL;
  AppendRequest r;
  r.shape = shape;
  r.paging = paging;
  r.n_new = n_new;
  r.k_new = k_new;
  r.v_new = v_new;
  r.pos = pos;
  r.keep_pair_idx = keep_pair_idx;
  r.k_cache = k_pool;
  r.v_cache = v_pool;
  r.stream = stream;
  return append_impl(r);
}

rap_status_t rap_rope_append_q8(const rap_shape_t* shape, int32_t n_new, const void* k_new, const void* v_new,
                                const int32_t* pos, const int32_t* keep_pair_idx, void* k_cache8, void* v_cache8,
                                const float* k_scale, const float* v_scale, void* stream) {
  AppendRequest r;
  r.shape = shape;
  r.n_new = n_new;
  r.k_new = k_new;
  r.v_new = v_new;
  r.pos = pos;
  r.keep_pair_idx = keep_pair_idx;
  r.k_cache = k_cache8;
  r.v_cache = v_cache8;
  r.fp8 = true;
  r.k_scale = k_scale;
  r.v_scale = v_scale;
  r.stream = stream;
  return append_impl(r);
}

rap_status_t rap_rope_append_mx4(const rap_shape_t* shape, int32_t n_new, const void* k_new, const void* v_new,
                                 const int32_t* pos, const int32_t* keep_pair_idx, void* k_codes, void* k_scales,
                                 void* v_codes, void* v_scales, void* stream) {
  AppendRequest r;
  r.shape = shape;
  r.n_new = n_new;
  r.k_new = k_new;
  r.v_new = v_new;
  r.pos = pos;
  r.keep_pair_idx = keep_pair_idx;
  r.k_cache = k_codes;
  r.v_cache = v_codes;
  r.mx4 = true;
  r.k_scales4 = k_scales;
  r.v_scales4 = v_scales;
  r.stream = stream;
  return append_impl(r);
}

rap_status_t rap_decode_attn_mx4(const rap_shape_t* shape, const void* q, const void* k_codes, const void* k_scales,
                                 const void* v_codes, const void* v_scales, const int32_t* seq_lens,
                                 int64_t max_seq_len, void* out, float scale, void* workspace, size_t workspace_bytes,
                                 const rap_tuning_t* tuning, void* stream) {
  DecodeRequest r;
  r.shape = shape;
  r.q = q;
  r.k_cache = k_codes;
  r.v_cache = v_codes;
  r.mx4 = true;
  r.k_scales4 = k_scales;
  r.v_scales4 = v_scales;
  r.seq_lens = seq_lens;
  r.max_seq_len = max_seq_len;
  r.out = out;
  r.scale = scale;
  r.workspace = workspace;
  r.workspace_bytes = workspace_bytes;
  r.tuning = tuning;
  r.stream = stream;
  return decode_impl(r);
}

rap_status_t rap_rope_queries(const rap_shape_t* shape, int32_t n_new, const void* q, const int32_t* pos,
                              const int32_t* keep_pair_idx, void* q_out, void* stream) {
  rap_status_t st = check_shape(shape);
  if (st != RAP_OK) return st;
  if (n_new < 0) return RAP_ERR_SHAPE;
  if (n_new == 0 || shape->batch == 0) return RAP_OK;
  if (!q || !pos || no_rotation_rule(shape, keep_pair_idx) || !q_out) return RAP_ERR_NULL;
  if (static_cast<int64_t>(shape->batch) * n_new > kInt32Max) return RAP_ERR_UNSUPPORTED;
  if (misaligned(q, 4) || misaligned(q_out, 4)) return RAP_ERR_SHAPE;
  // the append kernel walking query rows: no V, no cache layout, G query heads per row of kept pairs
  rap::AppendArgs a;
  memset(&a, 0, sizeof(a));
  a.k_new = static_cast<const uint16_t*>(q);
  a.pos = pos;
  a.keep = keep_pair_idx;
  a.pair_freq = shape->pair_inv_freq;
  a.k_cache = static_cast<uint16_t*>(q_out);
  a.batch = shape->batch;
  a.n_new = n_new;
  a.n_kv = shape->n_q_heads;          // heads per token row of the input
  a.d_head = shape->d_head;
  a.n_pairs = shape->n_pairs;
  a.d_v = 0;
  a.group = shape->n_q_heads / shape->n_kv_heads;
  a.cap = shape->cache_cap;
  a.neg2_log2_theta_over_d = neg2_log2_theta_over_d(shape);
  return hip_status(rap::launch_rope_queries(a, static_cast<hipStream_t>(stream)));
}

size_t rap_decode_attn_workspace_bytes(const rap_shape_t* shape, int64_t max_seq_len, const rap_tuning_t* tuning) {
  const size_t need = call_workspace_bytes(shape, max_seq_len, tuning);
  if (need == 0 || (tuning && tuning->rows_per_split != 0)) return need;
  // The array also serves smaller batches and shorter sequences, which the plain rule may cut into
  // more ranges (32 x 2200 rows: two, 33: one): a slab then has at most two ranges per compute unit's
  // share, none shorter than 512 rows, or as many as 4096 rows give it.
  const int64_t b = shape->batch, cuts = 2LL * device_cus() / shape->n_kv_heads;
  const int64_t by_512 = b * ((max_seq_len + 511) / 512), by_4096 = b * ((max_seq_len + 4095) / 4096);
  const int64_t ranges = std::max(std::min(cuts, by_512), by_4096);
  return std::max(need, slot_bytes(static_cast<size_t>(ranges + b) * shape->n_q_heads, shape->d_v));
}

rap_status_t rap_decode_attn(const rap_shape_t* shape, const void* q, const void* k_cache, const void* v_cache,
                             const int32_t* seq_lens, int64_t max_seq_len, void* out, float scale, void* workspace,
                             size_t workspace_bytes, const rap_tuning_t* tuning, void* stream) {
  DecodeRequest r;
  r.shape = shape;
  r.q = q;
  r.k_cache = k_cache;
  r.v_cache = v_cache;
  r.seq_lens = seq_lens;
  r.max_seq_len = max_seq_len;
  r.out = out;
  r.scale = scale;
  r.workspace = workspace;
  r.workspace_bytes = workspace_bytes;
  r.tuning = tuning;
  r.stream = stream;
  return decode_impl(r);
}

rap_status_t rap_decode_attn_static(const rap_shape_t* shape, const void* q, const void* k_cache, const void* v_cache,
                                    const int32_t* seq_lens, int64_t max_seq_len, void* out, float scale,
                                    const rap_tuning_t* tuning, void* stream) {
  DecodeRequest r;
  r.shape = shape;
  r.q = q;
  r.k_cache = k_cache;
  r.v_cache = v_cache;
  r.seq_lens = seq_lens;
  r.max_seq_len = max_seq_len;
  r.out = out;
  r.scale = scale;
  r.tuning = tuning;
  r.stream = stream;
  // an invalid shape, length or tuning gives 0 here and its own error from decode_impl below
  const size_t need = call_workspace_bytes(shape, max_seq_len, tuning);
  if (need > RAP_STATIC_SCRATCH_BYTES) return RAP_ERR_STATIC_LIMIT;
  if (need > 0 && shape->batch > 0) {
    void* ptr = nullptr;
    const rap_status_t st = static_scratch(&ptr);
    if (st != RAP_OK) return st;
    r.workspace = ptr;
    r.workspace_bytes = RAP_STATIC_SCRATCH_BYTES;
  }
  return decode_impl(r);
}

rap_status_t rap_decode_attn_rope(const rap_shape_t* shape, const void* q, const int32_t* q_pos,
                                  const int32_t* keep_pair_idx, const void* k_cache, const void* v_cache,
                                  const int32_t* seq_lens, int64_t max_seq_len, void* out, float scale,
                                  void* workspace, size_t workspace_bytes, const rap_tuning_t* tuning, void* stream) {
  if (live_call(shape, max_seq_len) && (!q_pos || no_rotation_rule(shape, keep_pair_idx))) return null_after_shape(shape);
  DecodeRequest r;
  r.shape = shape;
  r.q = q;
  r.q_pos = q_pos;
  r.keep_pair_idx = keep_pair_idx;
  r.k_cache = k_cache;
  r.v_cache = v_cache;
  r.seq_lens = seq_lens;
  r.max_seq_len = max_seq_len;
  r.out = out;
  r.scale = scale;
  r.workspace = workspace;
  r.workspace_bytes = workspace_bytes;
  r.tuning = tuning;
  r.stream = stream;
  return decode_impl(r);
}

rap_status_t rap_decode_step(const rap_shape_t* shape, const void* k_new, const void* v_new, const int32_t* pos,
                             const int32_t* keep_pair_idx, const void* q, int32_t q_is_rotated, void* k_cache,
                             void* v_cache, const int32_t* seq_lens, int64_t max_seq_len, void* out, float scale,
                             void* workspace, size_t workspace_bytes, const rap_tuning_t* tuning, void* stream) {
  if (live_call(shape, max_seq_len) && (!k_new || !v_new || !pos || no_rotation_rule(shape, keep_pair_idx)))
    return null_after_shape(shape);
  DecodeRequest r;
  r.shape = shape;
  r.q = q;
  r.q_pos = q_is_rotated ? nullptr : pos;
  r.keep_pair_idx = keep_pair_idx;
  r.k_cache = k_cache;
  r.v_cache = v_cache;
  r.k_new = k_new;
  r.v_new = v_new;
  r.new_pos = pos;
  r.seq_lens = seq_lens;
  r.max_seq_len = max_seq_len;
  r.out = out;
  r.scale = scale;
  r.workspace = workspace;
  r.workspace_bytes = workspace_bytes;
  r.tuning = tuning;
  r.stream = stream;
  return decode_impl(r);
}

rap_status_t rap_decode_step_ex(const rap_shape_t* shape, const rap_kv_cache_t* cache, const void* k_new,
                                const void* v_new, const int32_t* pos, const int32_t* keep_pair_idx, const void* q,
                                int32_t q_is_rotated, const int32_t* seq_lens, int64_t max_seq_len, void* out, float scale,
                                void* workspace, size_t workspace_bytes, const rap_tuning_t* tuning, void* stream) {
  if (!cache) return RAP_ERR_NULL;
  if ((cache->k_scale == nullptr) != (cache->v_scale == nullptr)) return null_after_shape(shape);
  if (live_call(shape, max_seq_len) && (!k_new || !v_new || !pos || no_rotation_rule(shape, keep_pair_idx)))
    return null_after_shape(shape);
  DecodeRequest r;
  r.shape = shape;
  r.paging = cache->paging;
  r.q = q;
  r.q_pos = q_is_rotated ? nullptr : pos;
  r.keep_pair_idx = keep_pair_idx;
  r.k_cache = cache->k;
  r.v_cache = cache->v;
  r.fp8 = cache->k_scale != nullptr;
  r.k_scale = cache->k_scale;
  r.v_scale = cache->v_scale;
  r.k_new = k_new;
  r.v_new = v_new;
  r.new_pos = pos;
  r.seq_lens = seq_lens;
  r.max_seq_len = max_seq_len;
  r.out = out;
  r.scale = scale;
  r.workspace = workspace;
  r.workspace_bytes = workspace_bytes;
  r.tuning = tuning;
  r.stream = stream;
  return decode_impl(r);
}

rap_status_t rap_decode_attn_multi(const rap_shape_t* shape, const rap_kv_cache_t* cache, int32_t n_tok, const void* q,
                                   const int32_t* seq_lens, int64_t max_seq_len, void* out, float scale,
                                   void* workspace, size_t workspace_bytes, const rap_tuning_t* tuning, void* stream) {
  if (!cache) return RAP_ERR_NULL;
  if ((cache->k_scale == nullptr) != (cache->v_scale == nullptr)) return null_after_shape(shape);
  DecodeRequest r;
  r.shape = shape;
  r.paging = cache->paging;
  r.q = q;
  r.k_cache = cache->k;
  r.v_cache = cache->v;
  r.fp8 = cache->k_scale != nullptr;
  r.k_scale = cache->k_scale;
  r.v_scale = cache->v_scale;
  r.n_tok = n_tok;
  r.seq_lens = seq_lens;
  r.max_seq_len = max_seq_len;
  r.out = out;
  r.scale = scale;
  r.workspace = workspace;
  r.workspace_bytes = workspace_bytes;
  r.tuning = tuning;
  r.stream = stream;
  return decode_impl(r);
}

rap_status_t rap_decode_attn_q8(const rap_shape_t* shape, const void* q, const int32_t* q_pos,
                                const int32_t* keep_pair_idx, const void* k_cache8, const void* v_cache8,
                                const float* k_scale, const float* v_scale, const int32_t* seq_lens,
                                int64_t max_seq_len, void* out, float scale, void* workspace, size_t workspace_bytes,
                                const rap_tuning_t* tuning, void* stream) {
  if (live_call(shape, max_seq_len) && q_pos && no_rotation_rule(shape, keep_pair_idx)) return null_after_shape(shape);
  DecodeRequest r;
  r.shape = shape;
  r.q = q;
  r.q_pos = q_pos;
  r.keep_pair_idx = keep_pair_idx;
  r.k_cache = k_cache8;
  r.v_cache = v_cache8;
  r.fp8 = true;
  r.k_scale = k_scale;
  r.v_scale = v_scale;
  r.seq_lens = seq_lens;
  r.max_seq_len = max_seq_len;
  r.out = out;
  r.scale = scale;
  r.workspace = workspace;
  r.workspace_bytes = workspace_bytes;
  r.tuning = tuning;
  r.stream = stream;
  return decode_impl(r);
}

rap_status_t rap_decode_attn_paged(const rap_shape_t* shape, const rap_paging_t* paging, const void* q,
                                   const int32_t* q_pos, const int32_t* keep_pair_idx, const void* k_pool,
                                   const void* v_pool, const int32_t* seq_lens, int64_t max_seq_len, void* out,
                                   float scale, void* workspace, size_t workspace_bytes, const rap_tuning_t* tuning,
                                   void* stream) {
  if (!paging) return RAP_ERR_NULL;
  if (live_call(shape, max_seq_len) && q_pos && no_rotation_rule(shape, keep_pair_idx)) return null_after_shape(shape);
  DecodeRequest r;
  r.shape = shape;
  r.paging = paging;
  r.q = q;
  r.q_pos = q_pos;
  r.keep_pair_idx = keep_pair_idx;
  r.k_cache = k_pool;
  r.v_cache = v_pool;
  r.seq_lens = seq_lens;
  r.max_seq_len = max_seq_len;
  r.out = out;
  r.scale = scale;
  r.workspace = workspace;
  r.workspace_bytes = workspace_bytes;
  r.tuning = tuning;
  r.stream = stream;
  return decode_impl(r);
}

rap_status_t rap_rope_append_paged_q8(const rap_shape_t* shape, const rap_paging_t* paging, int32_t n_new,
                                      const void* k_new, const void* v_new, const int32_t* pos,
                                      const int32_t* keep_pair_idx, void* k_pool8, void* v_pool8, const float* k_scale,
                                      const float* v_scale, void* stream) {
  if (!paging) return RAP_ERR_NULL;
  AppendRequest r;
  r.shape = shape;
  r.paging = paging;
  r.n_new = n_new;
  r.k_new = k_new;
  r.v_new = v_new;
  r.pos = pos;
  r.keep_pair_idx = keep_pair_idx;
  r.k_cache = k_pool8;
  r.v_cache = v_pool8;
  r.fp8 = true;
  r.k_scale = k_scale;
  r.v_scale = v_scale;
  r.stream = stream;
  return append_impl(r);
}

rap_status_t rap_decode_attn_paged_q8(const rap_shape_t* shape, const rap_paging_t* paging, const void* q,
                                      const int32_t* q_pos, const int32_t* keep_pair_idx, const void* k_pool8,
                                      const void* v_pool8, const float* k_scale, const float* v_scale,
                                      const int32_t* seq_lens, int64_t max_seq_len, void* out, float scale,
                                      void* workspace, size_t workspace_bytes, const rap_tuning_t* tuning, void* stream) {
  if (!paging) return RAP_ERR_NULL;
  if (live_call(shape, max_seq_len) && q_pos && no_rotation_rule(shape, keep_pair_idx)) return null_after_shape(shape);
  DecodeRequest r;
  r.shape = shape;
  r.paging = paging;
  r.q = q;
  r.q_pos = q_pos;
  r.keep_pair_idx = keep_pair_idx;
  r.k_cache = k_pool8;
  r.v_cache = v_pool8;
  r.fp8 = true;
  r.k_scale = k_scale;
  r.v_scale = v_scale;
  r.seq_lens = seq_lens;
  r.max_seq_len = max_seq_len;
  r.out = out;
  r.scale = scale;
  r.workspace = workspace;
  r.workspace_bytes = workspace_bytes;
  r.tuning = tuning;
  r.stream = stream;
  return decode_impl(r);
}

rap_status_t rap_prefill_attn(const rap_shape_t* shape, int32_t n_new, const void* q, const void* k_cache,
                              const void* v_cache, const int32_t* seq_lens, int64_t max_seq_len, void* out, float scale,
                              void* stream) {
  return prefill_impl(shape, nullptr, n_new, q, k_cache, v_cache, seq_lens, max_seq_len, out, scale, stream);
}

rap_status_t rap_prefill_attn_ex(const rap_shape_t* shape, const rap_kv_cache_t* cache, int32_t n_new, const void* q,
                                 const int32_t* seq_lens, int64_t max_seq_len, void* out, float scale, void* stream) {
  if (!cache) return RAP_ERR_NULL;
  return prefill_impl(shape, cache->paging, n_new, q, cache->k, cache->v, seq_lens, max_seq_len, out, scale, stream,
                      cache->k_scale, cache->v_scale);
}

size_t rap_prefill_attn_split_workspace_bytes(const rap_shape_t* shape, int32_t n_new, int64_t max_seq_len) {
  if (check_shape(shape) != RAP_OK || n_new < 1 || max_seq_len < 1 || max_seq_len > shape->cache_cap) return 0;
  if (shape->batch == 0) return 0;
  return prefill_workspace_need(shape, n_new, prefill_plan_of(shape, n_new, max_seq_len));
}

rap_status_t rap_prefill_attn_split(const rap_shape_t* shape, const rap_kv_cache_t* cache, int32_t n_new, const void* q,
                                    const int32_t* seq_lens, int64_t max_seq_len, void* out, float scale,
                                    void* workspace, size_t workspace_bytes, void* stream) {
  if (!cache) return RAP_ERR_NULL;
  return prefill_impl(shape, cache->paging, n_new, q, cache->k, cache->v, seq_lens, max_seq_len, out, scale, stream,
                      cache->k_scale, cache->v_scale, true, workspace, workspace_bytes);
}

rap_status_t rap_prefill_attn_paged(const rap_shape_t* shape, const rap_paging_t* paging, int32_t n_new, const void* q,
                                    const void* k_pool, const void* v_pool, const int32_t* seq_lens, int64_t max_seq_len,
                                    void* out, float scale, void* stream) {
  if (!paging) return RAP_ERR_NULL;
  return prefill_impl(shape, paging, n_new, q, k_pool, v_pool, seq_lens, max_seq_len, out, scale, stream);
}

rap_status_t rap_check_inputs(const rap_shape_t* shape, int32_t n_new, const int32_t* pos, const int32_t* keep_pair_idx,
                              const int32_t* seq_lens, int64_t max_seq_len, uint32_t* flags, void* stream) {
  const rap_status_t st = check_shape(shape);
  if (st != RAP_OK) return st;
  if (!flags) return RAP_ERR_NULL;
  if (n_new < 0 || max_seq_len < 0 || max_seq_len > shape->cache_cap) return RAP_ERR_SHAPE;
  if (misaligned(flags, 4)) return RAP_ERR_SHAPE;
  const long long n_pos = pos ? static_cast<long long>(shape->batch) * n_new : 0;
  if (n_pos > kInt32Max) return RAP_ERR_UNSUPPORTED;
  return hip_status(rap::launch_validate(pos, n_pos, shape->cache_cap, keep_pair_idx, shape->n_kv_heads, shape->n_pairs,
                                         shape->d_head / 2, seq_lens, shape->batch, max_seq_len, flags,
                                         static_cast<hipStream_t>(stream)));
}

rap_status_t rap_stream_read(const void* src, size_t bytes, void* sink, void* stream) {
  if (!src || !sink) return RAP_ERR_NULL;
  if ((bytes & 15) || misaligned(src, 16) || misaligned(sink, 16)) return RAP_ERR_SHAPE;
  return hip_status(rap::launch_stream_read(src, bytes, sink, static_cast<hipStream_t>(stream)));
}

rap_status_t rap_stream_copy(void* dst, const void* src, size_t bytes, void* stream) {
  if (!src || !dst) return RAP_ERR_NULL;
  if ((bytes & 15) || misaligned(src, 16) || misaligned(dst, 16)) return RAP_ERR_SHAPE;
  return hip_status(rap::launch_stream_copy(dst, src, bytes, static_cast<hipStream_t>(stream)));
}

const char* rap_status_str(rap_status_t status) {
  switch (status) {
    case RAP_OK: return "ok";
    case RAP_ERR_NULL: return "null pointer";
    case RAP_ERR_SHAPE: return "inconsistent shape or argument";
    case RAP_ERR_UNSUPPORTED: return "shape outside the supported range";
    case RAP_ERR_CAPACITY: return "max_seq_len exceeds cache capacity";
    case RAP_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case RAP_ERR_HIP: return "HIP runtime error";
    case RAP_ERR_STATIC_LIMIT: return "shape needs more scratch than the static array of rap_decode_attn_static holds";
  }
  return "unknown status";
}

int32_t rap_version(void) { return 1000; }

}  // extern "C"
