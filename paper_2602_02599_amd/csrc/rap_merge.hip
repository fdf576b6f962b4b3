// Second stage of split decode attention: combine the per-range partials of one query head.
//
// A range s leaves (m_s, l_s, acc_s[d_v]) with m_s the running maximum of the scaled scores in
// log2 units, l_s = sum_i 2^(x_i - m_s) and acc_s = sum_i 2^(x_i - m_s) V[i].  Softmax over the
// whole sequence is then
//   out = sum_s 2^(m_s - m*) acc_s / sum_s 2^(m_s - m*) l_s,   m* = max_s m_s,
// which is Eq. (attn) regrouped by row ranges.  Only the ranges that hold rows of this sequence
// (ceil(len / rows_per_split) of them) were written by the first stage and only those are read.
// In the one-call decode step there is one more slot behind the ranges, always written: the new
// token on its own (m = its score, l = 1, acc = its V row, or m = -inf when it is not attended).
// MULTI, several query tokens per sequence: the ranges stop in front of the new tokens' rows, and
// the causal part among the tokens themselves (token t attends the new rows 0 .. t, at most 16) is
// worked out here, by the workgroup of the query row: each thread multiplies one element of the
// query row with the same element of the new K rows, the products are summed over the workgroup,
// and the weighted new V rows enter the combination like one more range.
//
// Latency is all there is to this kernel (a few MB at most): the partials miss L2, they were written
// through other XCDs, so one round trip for everything is the floor.  Eight slots per thread are
// requested together, before the sequence length is known, and GRP groups of 128 threads take
// eight slots each side by side, so that up to 8 GRP ranges cost one round trip; the groups meet in
// LDS.  64 ranges (one sequence of 32768 rows, 32 query heads): 11.3 us with one group, 3.9 us with
// eight.  Up to eight ranges one group is enough, and its smaller workgroup starts faster.
#include "rap_device.h"

namespace rap {

constexpr int kMaxTok = 16;
constexpr int kMergeSlots = 8;                     // slots a thread has in flight
typedef __attribute__((ext_vector_type(4))) float f32x4;

// MT: 0 for one query token, else an upper bound of n_tok, to which the loops over new tokens are
// unrolled: four, eight or sixteen.  Unrolled to sixteen, five to eight tokens cost 2 to 4 us more (attention
// of 5 tokens, 16 x 8192 rows, 24 query heads: 73.9 us, to eight 70.1; fp8 50.0 and 46.4; 9 tokens 71.3).
// FLAT: ranges by length (DecodeArgs); an instantiation of its own, because what it takes costs the other form up to 1.5 us.
template <int MT, int GRP, bool FLAT>
__global__ __launch_bounds__(128 * GRP) void merge_kernel(DecodeArgs a) {
  constexpr bool MULTI = MT > 0;
  const long long hq = blockIdx.x;                 // query row: (b * n_tok + token) * n_q + query head
  // (FLAT: 32 bits, because the first slots' addresses wait for what is left over)
  const uint32_t n_q = a.n_q, in_batch = FLAT ? blockIdx.x / (n_q * a.n_tok) : 0;
  const int b = FLAT ? in_batch : static_cast<int>(hq / (static_cast<long long>(a.n_q) * a.n_tok));
  const int c = threadIdx.x & 127;
  const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x >> 7);
  const bool live = c < a.d_v;
  // This query row's slots: one behind the other, or (FLAT) `stride` rows apart among those of its KV head, from slot0 on.
  const int stride = FLAT ? a.n_tok * a.group : 1;
  long long row0 = hq * a.n_slots;
  if constexpr (FLAT) {
    const uint32_t in_seq = blockIdx.x - in_batch * n_q * a.n_tok, qt = MULTI ? in_seq / n_q : 0, qh = in_seq - qt * n_q;
    const uint32_t kv = qh / static_cast<uint32_t>(a.group);
    row0 = static_cast<long long>(kv) * a.flat_slots * stride + qt * a.group + (qh - kv * a.group);
  }
  int slot0 = FLAT ? b * a.flat_full : 0;
  const float* ml = a.part_ml + row0 * 2;
  const float* accc = a.part_acc + row0 * a.d_v + (live ? c : 0);
  // All slots of a query head are allocated, whatever they hold, so this group's first eight are
  // requested before anything else is known (FLAT: those that are right where all sequences are as long as they may be).
  float m[kMergeSlots], l[kMergeSlots], v[kMergeSlots];
  auto request = [&](int s0) {
#pragma unroll
    for (int u = 0; u < kMergeSlots; ++u) {
      const bool have = FLAT ? slot0 + s0 + u < a.flat_slots : s0 + u < a.n_split;
      const int at = (slot0 + s0 + u) * stride;
      m[u] = have ? ml[2 * at] : -INFINITY;
      l[u] = have ? ml[2 * at + 1] : 0.f;
      v[u] = have ? accc[static_cast<long long>(at) * a.d_v] : 0.f;
    }
  };
  request(kMergeSlots * grp);
  const bool tok = grp == 0 && a.n_slots > a.n_split;   // the slot behind the ranges is in use
  const int tok_at = FLAT ? (a.flat_slots - a.batch + b) * stride : a.n_split;
  float m_tok = tok ? ml[2 * tok_at] : -INFINITY;
  float l_tok = tok ? ml[2 * tok_at + 1] : 0.f;
  float v_tok = tok ? accc[static_cast<long long>(tok_at) * a.d_v] : 0.f;
  FlatLens f;
  if constexpr (FLAT) f = flat_lens(a, threadIdx.x & (kWave - 1));
  const int t_new = a.new_pos != nullptr ? a.new_pos[b] : -1;
  int len = a.seq_lens[b];
  len = len < 0 ? 0 : (len > a.max_len ? a.max_len : len);
  if constexpr (MULTI) {
    __shared__ float s_dot[2][MT > 0 ? MT : 1];
    const int T = a.n_tok, G = a.group;
    const int t = static_cast<int>((hq / a.n_q) % T);           // this query row's token
    const int h = static_cast<int>(hq % a.n_q) / G;             // and KV head
    const int p0 = len - T;                                     // position of new token 0, may be negative
    const bool q8 = a.k_scale != nullptr;
    // row of the cache (dense) or of the pool (paged) that holds position pos >= 0
    auto row_of = [&](int pos) -> long long {
      if (a.block_table == nullptr) return (static_cast<long long>(b) * a.n_kv + h) * a.cap + pos;
      int pg = a.block_table[static_cast<long long>(b) * a.max_pages + (pos >> a.page_shift)];
      pg = pg < 0 ? 0 : (pg >= a.n_pages ? a.n_pages - 1 : pg);
      return ((static_cast<long long>(pg) * a.n_kv + h) << a.page_shift) + (pos & ((1 << a.page_shift) - 1));
    };
    const bool have_k = c < a.d_k;
    const float qv = have_k ? bf16_to_f32(a.q[hq * a.d_k + c]) : 0.f;
    float prod[MT], vnew[MT];
    // The loads of all slots are issued first and used afterwards, so that they travel together:
    // slot j beyond this token's own row repeats that row, a position in front of the sequence
    // reads row 0; what such a slot holds is dropped below by a select.
    const int ck = have_k ? c : 0, cv = live ? c : 0;
    if (grp == 0) {
      uint32_t kraw[MT], vraw[MT];
#pragma unroll
      for (int j = 0; j < MT; ++j) {
        const int pos = p0 + (j < t ? j : t);
        const long long row = row_of(pos < 0 ? 0 : pos);
        if (q8) {
          kraw[j] = reinterpret_cast<const uint8_t*>(a.k_cache)[row * a.d_k + ck];
          vraw[j] = reinterpret_cast<const uint8_t*>(a.v_cache)[row * a.d_v + cv];
        } else {
          kraw[j] = a.k_cache[row * a.d_k + ck];
          vraw[j] = a.v_cache[row * a.d_v + cv];
        }
      }
#pragma unroll
      for (int j = 0; j < MT; ++j) {
        const float kf = q8 ? e4m3_to_f32(static_cast<uint8_t>(kraw[j])) : bf16_to_f32(static_cast<uint16_t>(kraw[j]));
        vnew[j] = q8 ? e4m3_to_f32(static_cast<uint8_t>(vraw[j])) : bf16_to_f32(static_cast<uint16_t>(vraw[j]));
        prod[j] = have_k ? qv * kf : 0.f;
      }
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) {
#pragma unroll
        for (int j = 0; j < MT; ++j) prod[j] += __shfl_xor(prod[j], o);
      }
      if ((c & 63) == 0) {
#pragma unroll
        for (int j = 0; j < MT; ++j) s_dot[c >> 6][j] = prod[j];
      }
    }
    __syncthreads();
    if (grp == 0) {
      const float sc = q8 ? a.scale_log2e * a.k_scale[h] : a.scale_log2e;
      float x[MT];
      m_tok = -INFINITY;
#pragma unroll
      for (int j = 0; j < MT; ++j) {
        x[j] = (j <= t && p0 + j >= 0) ? (s_dot[0][j] + s_dot[1][j]) * sc : -INFINITY;
        m_tok = fmaxf(m_tok, x[j]);
      }
      l_tok = 0.f;
      v_tok = 0.f;
      if (m_tok > -INFINITY) {
#pragma unroll
        for (int j = 0; j < MT; ++j) {
          const bool in = j <= t && p0 + j >= 0;
          const float pj = in ? exp2f(x[j] - m_tok) : 0.f;
          l_tok += pj;
          v_tok = fmaf(pj, in ? vnew[j] : 0.f, v_tok);          // a left-out slot may hold NaN or inf
        }
        if (q8) v_tok *= a.v_scale[h];
      }
    }
  }
  int n;                                           // ranges that hold rows
  if constexpr (FLAT) {
    int first;
    if (f.alike > 0) {
      n = min(f.alike, __builtin_amdgcn_readlane(f.units, b));
      first = b * f.alike;
    } else {
      int n_of, n_to;
      flat_counts(a, f, &n_of, &n_to);
      n = __builtin_amdgcn_readlane(n_of, b);
      first = __builtin_amdgcn_readlane(n_to, b) - n;
    }
    if (first != slot0) {
      slot0 = first;
      if (kMergeSlots * grp < n) request(kMergeSlots * grp);
    }
  } else {
    if (len > 0 && t_new == len - 1) len -= 1;     // the first stage stopped before the new token's row
    if (a.n_tok > 1) len = len > a.n_tok ? len - a.n_tok : 0;   // or before the new tokens' rows
    n = (len + a.rows_per_split - 1) / a.rows_per_split;
  }
  float mstar = m_tok, den = 0.f, num = 0.f;
  if (m_tok > -INFINITY) {
    den = l_tok;
    num = v_tok;
  }
  // slots beyond the ranges that hold rows are dropped by a select, not multiplied
  for (int s0 = kMergeSlots * grp; s0 < n; s0 += kMergeSlots * GRP) {
    if (s0 != kMergeSlots * grp) request(s0);
    float gmax = -INFINITY;
#pragma unroll
    for (int u = 0; u < kMergeSlots; ++u) {
      if (s0 + u >= n) {                           // unwritten slot: any bits, NaN included
        m[u] = -INFINITY;
        l[u] = 0.f;
        v[u] = 0.f;
      }
      gmax = fmaxf(gmax, m[u]);
    }
    if (gmax > mstar) {                            // the reference follows the running maximum
      const float r = mstar > -INFINITY ? exp2f(mstar - gmax) : 0.f;
      den *= r;
      num *= r;
      mstar = gmax;
    }
#pragma unroll
    for (int u = 0; u < kMergeSlots; ++u) {
      const bool has = m[u] > -INFINITY;           // an empty range leaves only its reference and sum
      const float w = has ? exp2f(m[u] - mstar) : 0.f;
      den = fmaf(w, l[u], den);
      num = fmaf(w, has ? v[u] : 0.f, num);
    }
  }
  if constexpr (GRP > 1) {
    __shared__ float s_m[GRP], s_den[GRP], s_num[GRP][128];
    if (c == 0) {
      s_m[grp] = mstar;
      s_den[grp] = den;
    }
    s_num[grp][c] = num;
    __syncthreads();
    if (grp != 0) return;
#pragma unroll
    for (int g = 1; g < GRP; ++g) mstar = fmaxf(mstar, s_m[g]);
    den = 0.f;
    num = 0.f;
#pragma unroll
    for (int g = 0; g < GRP; ++g) {
      const float w = s_m[g] > -INFINITY ? exp2f(s_m[g] - mstar) : 0.f;
      den = fmaf(w, s_den[g], den);
      num = fmaf(w, s_num[g][c], num);
    }
  }
  if (live) a.out[hq * a.d_v + c] = den > 0.f ? num / den : 0.f;
}

// The same for a prefill launch in key ranges, whose query rows are many and whose ranges are few, so that reading the partials is what bounds it: 32 lanes per query row, four
// channels per lane in 16-byte loads (where d_v is no multiple of four the last lane repeats channels of its
// neighbour), eight rows per workgroup.  Up to eight ranges are one round trip; more are shared by 2, 4 or 8 sets
// of lanes, which meet in LDS.  One workgroup of 128 threads per query row, as above, spends its time on starting
// workgroups: 72336 rows of 2 ranges, d_v = 56, 42.9 us, so 17.2; 16384 rows of 8, d_v = 90 (48 MB), 14.9 and 9.5;
// 1800 rows of 10, d_v = 74, 4.7 and 4.0.  Rows of one range
// were stored by the attention kernel itself: the launch begins at the first token whose block has several.
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_dw;
template <int GRP>
__global__ __launch_bounds__(256) void prefill_merge_kernel(PrefillMergeArgs a) {
  constexpr int ROWS = 8 / GRP;                    // per workgroup
  const int lane = threadIdx.x & 31, set = threadIdx.x >> 5;
  const int grp = set % GRP;
  const int tok0 = a.tok0;
  const int in_seq = static_cast<int>(blockIdx.x) * ROWS + set / GRP;
  const bool live = in_seq < (a.cut.n_new - tok0) * a.n_q;
  const int row = (static_cast<int>(blockIdx.y) * a.cut.n_new + tok0) * a.n_q + in_seq;
  const int dv = a.d_v;
  const int c = dv < 4 ? 0 : (4 * lane < dv - 4 ? 4 * lane : dv - 4);
  const bool has = 4 * lane < dv;
  const float2* ml = reinterpret_cast<const float2*>(a.part_ml) + static_cast<long long>(row) * a.n_ksplit;
  const float* acc = a.part_acc + static_cast<long long>(row) * a.n_ksplit * dv + c;
  float mstar = -INFINITY, den = 0.f;
  f32x4_dw num = {0.f, 0.f, 0.f, 0.f};
  // the first slots are requested, whatever they hold, before it is known how many this row's block wrote
  float m[kMergeSlots], l[kMergeSlots];
  f32x4_dw v[kMergeSlots];
  auto request = [&](int s0) {
#pragma unroll
    for (int u = 0; u < kMergeSlots; ++u) {
      const bool have = live && s0 + u < a.n_ksplit;
      const float2 x = have ? ml[s0 + u] : make_float2(-INFINITY, 0.f);
      m[u] = x.x;
      l[u] = x.y;
      v[u] = f32x4_dw{0.f, 0.f, 0.f, 0.f};
      if (have && has) {
        const float* p = acc + (s0 + u) * dv;
        if (dv >= 4) {
          v[u] = *reinterpret_cast<const f32x4_dw*>(p);
        } else {
#pragma unroll
          for (int e = 0; e < 3; ++e) v[u][e] = e < dv ? p[e] : 0.f;
        }
      }
    }
  };
  request(kMergeSlots * grp);
  const int n = live ? prefill_ranges(a.cut, (tok0 + in_seq / a.n_q) / a.cut.tok_per_wg) : 0;
  for (int s0 = kMergeSlots * grp; s0 < n; s0 += kMergeSlots * GRP) {
    if (s0 != kMergeSlots * grp) request(s0);
#pragma unroll
    for (int u = 0; u < kMergeSlots; ++u) m[u] = s0 + u < n ? m[u] : -INFINITY;      // unwritten: any bits
    float gmax = m[0];
#pragma unroll
    for (int u = 1; u < kMergeSlots; ++u) gmax = fmaxf(gmax, m[u]);
    if (gmax > mstar) {                            // the reference follows the running maximum
      const float r = mstar > -INFINITY ? exp2f(mstar - gmax) : 0.f;
      den *= r;
#pragma unroll
      for (int e = 0; e < 4; ++e) num[e] *= r;
      mstar = gmax;
    }
#pragma unroll
    for (int u = 0; u < kMergeSlots; ++u) {
      const bool some = m[u] > -INFINITY;          // an empty range leaves only its reference and sum
      const float w = some ? exp2f(m[u] - mstar) : 0.f;
      den = fmaf(w, some ? l[u] : 0.f, den);
#pragma unroll
      for (int e = 0; e < 4; ++e) num[e] = fmaf(w, some ? v[u][e] : 0.f, num[e]);
    }
  }
  if constexpr (GRP > 1) {
    __shared__ float s_m[8], s_den[8];
    __shared__ f32x4 s_num[8][32];
    if (lane == 0) {
      s_m[set] = mstar;
      s_den[set] = den;
    }
    s_num[set][lane] = f32x4{num[0], num[1], num[2], num[3]};
    __syncthreads();
    if (grp != 0) return;
#pragma unroll
    for (int g = 1; g < GRP; ++g) mstar = fmaxf(mstar, s_m[set + g]);
    den = 0.f;
    num = f32x4_dw{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < GRP; ++g) {
      const float w = s_m[set + g] > -INFINITY ? exp2f(s_m[set + g] - mstar) : 0.f;
      den = fmaf(w, s_den[set + g], den);
#pragma unroll
      for (int e = 0; e < 4; ++e) num[e] = fmaf(w, s_num[set + g][lane][e], num[e]);
    }
  }
  if (!live || !has || n <= 1) return;
#pragma unroll
  for (int e = 0; e < 4; ++e) num[e] = den > 0.f ? num[e] / den : 0.f;
  float* dst = a.out + static_cast<long long>(row) * dv + c;
  if (dv >= 4) {
    *reinterpret_cast<f32x4_dw*>(dst) = num;
  } else {
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (e < dv) dst[e] = num[e];
  }
}

namespace {

// Groups of 128 threads per query row: as many as the slots of a row need, eight for each.  FLAT: a long sequence among
// short ones has more ranges than n_split, up to flat_most; its rows get groups for them while all rows' groups number no
// more than three per compute unit, beyond which idle groups cost the other rows more than they save.  Attention
// calls with 1 / 2 / 4 / 8 groups, one sequence long and the others a 32nd: 8 x 65536, 256 rows, 47.4 / 45.6 / 44.9 / 45.2 us, equal
// lengths 225.2 / 225.6 / 225.4 / 226.2; 8 x 16384 20.3 / 19.2 / 19.1 / 19.6 and 63.9 / 64.0 / 64.3 / 64.8; 4 x 131072, 160 rows, 60.2 /
// 57.4 / 56.4 / 56.8 and 165.0 / 164.3 / 164.4 / 164.8; 24 x 8192, 768 rows, 15.9 / 16.3 / 17.5 / 20.3 and 91.8 / 92.4 / 93.4 / 96.0; 64 x
// 16384, 2048 rows, 34.2 / 35.3 / 38.7 / 47.1 and 459 / 461 / 464 / 472.
template <int MT, bool FLAT>
void launch_groups(const DecodeArgs& a, hipStream_t stream) {
  dim3 grid(static_cast<unsigned>(a.batch) * a.n_tok * a.n_q);
  int slots = a.n_split;
  if constexpr (FLAT) {
    const FlatPlan p = {a.flat_wgs, a.flat_slots, a.flat_full, a.flat_few};
    const int most = flat_most(p, (a.max_len + kSplitQuantum - 1) / kSplitQuantum);
    const int each = 3 * kChipUnits / static_cast<int>(grid.x), groups = each >= 8 ? 8 : each >= 4 ? 4 : each >= 2 ? 2 : 1;
    const int wanted = most < groups * kMergeSlots ? most : groups * kMergeSlots;
    if (wanted > slots) slots = wanted;
  }
  // a launch holds fewer than 2^32 threads: from 4 M query rows on, fewer groups walk the ranges in turn
  auto fits = [&](unsigned threads) { return static_cast<unsigned long long>(grid.x) * threads < (1ull << 32); };
  if (slots <= kMergeSlots || !fits(256)) hipLaunchKernelGGL((merge_kernel<MT, 1, FLAT>), grid, dim3(128), 0, stream, a);
  else if (slots <= 2 * kMergeSlots || !fits(512)) hipLaunchKernelGGL((merge_kernel<MT, 2, FLAT>), grid, dim3(256), 0, stream, a);
  else if (slots <= 4 * kMergeSlots || !fits(1024)) hipLaunchKernelGGL((merge_kernel<MT, 4, FLAT>), grid, dim3(512), 0, stream, a);
  else hipLaunchKernelGGL((merge_kernel<MT, 8, FLAT>), grid, dim3(1024), 0, stream, a);
}

template <bool FLAT>
hipError_t launch_merge_form(const DecodeArgs& a, hipStream_t stream) {
  if (a.n_tok <= 1) launch_groups<0, FLAT>(a, stream);
  else if (a.n_tok <= 4) launch_groups<4, FLAT>(a, stream);
  else if (a.n_tok <= 8) launch_groups<8, FLAT>(a, stream);
  else launch_groups<kMaxTok, FLAT>(a, stream);
  return hipGetLastError();
}

template <int GRP>
hipError_t launch_prefill_groups(const PrefillMergeArgs& a, hipStream_t stream) {
  // fewer than 384 query blocks are cut, so the rows are few enough for any arithmetic here
  const int per_seq = (a.cut.n_new - a.tok0) * a.n_q;
  hipLaunchKernelGGL((prefill_merge_kernel<GRP>), dim3((per_seq * GRP + 7) / 8, a.batch), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

// `a` as the attention launch had it, tok_per_wg and n_qblk included.
hipError_t launch_prefill_merge(const PrefillArgs& p, hipStream_t stream) {
  const PrefillCut c = prefill_cut_of(p);
  const int tok0 = (c.n_qblk - prefill_blocks_beyond(c, 1)) * c.tok_per_wg;
  const PrefillMergeArgs a = {p.part_acc, p.part_ml, p.out, c, p.batch, p.n_q, p.d_v, p.n_ksplit, tok0};
  if (p.n_ksplit <= kMergeSlots) return launch_prefill_groups<1>(a, stream);
  if (p.n_ksplit <= 2 * kMergeSlots) return launch_prefill_groups<2>(a, stream);
  if (p.n_ksplit <= 4 * kMergeSlots) return launch_prefill_groups<4>(a, stream);
  return launch_prefill_groups<8>(a, stream);
}

hipError_t launch_merge(const DecodeArgs& a, hipStream_t stream) {
  return a.flat_wgs > 0 ? launch_merge_form<true>(a, stream) : launch_merge_form<false>(a, stream);
}

}  // namespace rap
