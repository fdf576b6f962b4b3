// Causal prefill attention over the compact cache: rap_prefill_attn.  The kernel and its table of
// instantiations, included by one source file per score width (rap_prefill_k1.hip .. _k4.hip) so
// that they compile side by side.
//
// Eq. (attn) for the last n_new tokens of every sequence at once, each token seeing the cache rows
// up to and including its own (the decoder-only rule), at the pruned widths d_k = 2P and d_v.
// Unlike the decode step this is a dense contraction (n_new x len scores per head), so it is
// bound by the matrix cores and by the vector instructions of the softmax beside them; the design
// is about keeping both busy at once:
//
//  * A workgroup takes a block of consecutive query tokens of one (sequence, KV head) together
//    with all G query heads of that KV head: its 64 NB "columns" are (token, head) pairs, so a K
//    or V tile staged in LDS once serves G times as many scores as it would per head.
//  * Everything is computed transposed, on v_mfma_f32_16x16x32_bf16: S^T[key][column] = K . q with
//    the K rows as the A operand from LDS and the query columns, resident in registers, as the B
//    operand; out^T[channel][column] = V^T . P^T with the probabilities as the B operand.  A lane
//    holds eight keys of ONE column in the result of the first product, and these are exactly the
//    contraction slots of the second when those are numbered accordingly: probabilities, the
//    softmax reference, the accumulators and their rescaling never leave the lane.  A K or V^T
//    fragment read from LDS serves all NB column blocks of the wavefront.
//  * The V^T operand (one channel, eight keys per lane) comes out of the row-major V tile by the
//    transposing LDS read (ds_read_b64_tr_b16), two per operand and no byte permutes.
//  * Tiles of 64 keys are staged by the whole workgroup one tile ahead into the other buffer, one
//    barrier per tile, in rows whose pitch is a constant of the instantiation, chosen so that the
//    16-byte K reads and the transposing V reads spread over all banks.  bf16 rows of even width
//    are loaded straight into LDS (a lane's destination is fixed, its source address is not: 16
//    bytes from any dword-aligned address); odd bf16 rows and one-byte codes go through registers,
//    codes being widened to bf16 (exactly) on the way, once per workgroup.
//  * Online softmax in the log2 domain against a per-column reference that moves only when a
//    score outgrows it by 2^64; the causal mask is applied only on the groups that straddle the
//    diagonal of the wavefront's columns, later groups are skipped by the wavefront.
//
// What bounds it, and what this form bought (32/8 heads, 8 x 8192 tokens, one launch):
//  * d = 90 4.31 -> 4.12 ms, d = 64 3.55 -> 3.27, d = 116 5.65 -> 5.12, d = 128 6.39 -> 5.40 ms, and
//    2 x 4001 tokens at widths 116/115 over one-byte codes 0.64 -> 0.41 ms, against the same
//    arithmetic with flat tile copies in LDS, V operands gathered by 4- (bf16), 2- or 1-byte reads
//    and byte permutes, and codes widened by every wavefront for itself.  The sums are the same,
//    bit for bit.
//  * The two streams of a key group at d = 90, 72 matrix instructions and 165 vector ones per
//    wavefront, take 0.69 us per SIMD and pair of wavefronts by themselves, the kernel 0.99 us.
//    On random operands the chip lowers its clock: matrix instructions alone then run at 1.9
//    PFLOP/s in this shape and at 1.7 as 32x32x16, which halves the instructions but moves more
//    accumulator words per product.  A version on 32x32x16, software-pipelined over three key groups
//    with every instruction placed, took 4.7 ms at d = 90 (32 columns per wavefront), so the
//    instructions are not what is short; with 64 columns 4.27 ms.
//  * Without the tile loads the kernel takes 0.19 ms less at d = 90, without the exponentials
//    0.35 ms, without its barriers the same; P.V of a block written between the vector
//    instructions of the next: the same.
//
// Paged caches: with a block table the caches are pools of pages of at least 64 rows, a staged
// tile never straddles two pages, and only its start address changes (looked up a tile ahead).
//
// Garbage safety: rows at or beyond the sequence length may hold any bits; their scores are never
// visible (a select to -inf), their V rows are cleared in LDS, K fragments are masked beyond d_k.
// A 16-byte piece may run past the end of its row into the next row of the cache (its bytes are
// masked, or belong to channels that are never stored), but never past the end of the cache.
#ifndef RAP_PREFILL_KERNEL_H_
#define RAP_PREFILL_KERNEL_H_

#include <utility>

#include "rap_device.h"

namespace rap {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((address_space(3))) const void* lds_ptr_t;
typedef __attribute__((address_space(3))) s16x4* lds_s16x4_t;
// four dwords at any byte address / any dword address
struct __attribute__((packed, aligned(1))) Bytes16 { uint32_t w[4]; };
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_dw;

// Maximum of three floats, NaNs left out: one instruction (v_max3_f32).  Not written as the
// instruction, because the compiler puts no wait between a matrix instruction and inline code that
// reads its result, which takes eight wait states; and not as fmaxf, which is asked to quiet a
// signalling NaN and passes every operand through a max(x, x) of its own first.
__device__ __forceinline__ float max3(float a, float b, float c) {
  return __builtin_elementwise_maximumnum(__builtin_elementwise_maximumnum(a, b), c);
}

// 16 bytes per lane from base + off (any dword-aligned address) straight into LDS: lane i's land at
// lane0_slot + 16 i.  Written as the instruction because the compiler, which cannot tell the buffer
// being filled from the one being read, waits for every outstanding load of the builtin's form in
// front of the next LDS read: the whole latency of a tile's loads, once per tile.  The caller waits
// (s_waitcnt, then the workgroup barrier) before anybody reads the slots.  The LDS address goes in
// m0, which the compiler sets and keeps track of.  It does not see a load in here: the s_nop is the
// five wait states that one needs after a vector instruction has written its base address
// (v_readlane, v_readfirstlane), and covers the one it needs after a move to m0.
__device__ __forceinline__ void load_to_lds(const unsigned char* base, int off, uint32_t lane0_slot) {
  asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "{m0}"(lane0_slot) : "memory");
}

// f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>): a loop whose index is a
// constant inside the body (register arrays must never be indexed by a run-time value)
template <int... Is, class F>
__device__ __forceinline__ void static_for_seq(std::integer_sequence<int, Is...>, F&& f) {
  (f(std::integral_constant<int, Is>()), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_seq(std::make_integer_sequence<int, N>(), f);
}

constexpr float kHeadroomP = 64.f;   // log2 units a score may exceed the reference before a rescale

// KS = ceil(d_k / 32) contraction steps of the scores, CT = ceil(d_v / 16) channel tiles, NB blocks
// of 16 query columns per wavefront.  ONES: d_v leaves a spare channel slot in the last tile, which
// carries the constant 1 so that the row sums of the probabilities come out of P.V.  MODE: how
// tiles reach LDS.
template <int KS, int CT, int MODE, bool ONES, int NB>
__global__ __launch_bounds__(256, 2) void prefill_kernel(PrefillArgs a) {
  constexpr int NW = kPrefillWaves;
  constexpr bool Q8 = MODE == kTilesCodes;
  constexpr bool K_DIRECT = !Q8, V_DIRECT = MODE == kTilesDirect;
  constexpr int EB = Q8 ? 1 : 2;                       // bytes per cache element
  constexpr int NT = 64 * NW;                          // threads
  constexpr int LPK = prefill_k_pitch(KS), LPV = prefill_v_pitch(CT);
  constexpr int KBUF = kPrefillTile * LPK, VBUF = kPrefillTile * LPV;
  // 16-byte LDS slots per row and loads per thread: direct loads walk whole padded rows (the slots
  // of the gap load nothing), loads through registers only the pieces that hold elements
  constexpr int SLK = LPK / 16, SLV = LPV / 16;
  constexpr int PCK = 2 * KS, PCV = Q8 ? CT : 2 * CT;   // pieces per row through registers (16 codes, or 8 bf16)
  constexpr int NLK = K_DIRECT ? (kPrefillTile * SLK + NT - 1) / NT : (kPrefillTile * PCK + NT - 1) / NT;
  constexpr int NLV = V_DIRECT ? (kPrefillTile * SLV + NT - 1) / NT : (kPrefillTile * PCV + NT - 1) / NT;
  extern __shared__ __align__(16) unsigned char smem[];   // K tile 0, K tile 1, V tile 0, V tile 1

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15;
  const int lg = lane >> 4;

  int qb, slab_id, ks = 0;
  const bool cut = a.n_ksplit > 1;
  bool in_ranges = false;                          // this block's rows are shared with other workgroups
  if (a.n_ranges > 0) {                            // cut, or all workgroups start together
    int nth;
    prefill_place_cut(static_cast<int>(blockIdx.x), a.n_ranges, a.n_kv * a.batch, a.slab_inv, &nth, &slab_id);
    if (!cut) {
      qb = a.n_qblk - 1 - nth;
    } else if (a.n_ranges <= kMaxOrdered) {
      const uint32_t r = a.order[nth];
      qb = r & 0x1ff;
      ks = (r >> 9) & 0x3fffff;
      in_ranges = (r >> 31) != 0;
    } else {
      const PrefillCut c = prefill_cut_of(a);
      prefill_range(nth, c, &qb, &ks);
      in_ranges = prefill_ranges(c, qb) > 1;
    }
  } else {
    prefill_place(static_cast<int>(blockIdx.x), a.n_qblk, a.n_kv * a.batch, prefill_slabs(KS, CT), &qb, &slab_id);
  }
  const int h = slab_id % a.n_kv;
  const int b = slab_id / a.n_kv;

  int len = a.seq_lens[b];
  len = len < 0 ? 0 : (len > a.max_len ? a.max_len : len);
  const int G = a.group;
  const int dk = a.d_k, dv = a.d_v;
  const int BT = a.tok_per_wg;
  const int i0 = qb * BT;
  const int i_end = min(a.n_new, i0 + BT);
  const int shift = len - a.n_new;                 // position of token i is shift + i
  const int n_keys = min(len, shift + i_end);      // rows the block's last token sees
  const long long out_row0 = (static_cast<long long>(b) * a.n_new) * a.n_q + h * G;   // + i * n_q + g

  const int n_tiles_all = (n_keys + kPrefillTile - 1) / kPrefillTile;
  const int t_first = ks * a.tiles_per_split;                       // key range of this workgroup, in tiles
  const int n_tiles = in_ranges ? min(n_tiles_all, t_first + a.tiles_per_split) : n_tiles_all;
  if (in_ranges && t_first >= n_tiles) {
    // nothing of this range is visible to the block (or the block lies before the start of its
    // sequence): empty partials, which the combining kernel drops
    for (int r = tid; r < (i_end - i0) * G; r += NT) {
      const int g = r % G, i = i0 + r / G;
      const long long slot = (out_row0 + static_cast<long long>(i) * a.n_q + g) * a.n_ksplit + ks;
      a.part_ml[slot * 2 + 0] = -INFINITY;
      a.part_ml[slot * 2 + 1] = 0.f;
    }
    return;
  }
  if (n_keys <= 0) {
    // every token of this block lies before the start of its sequence: zero rows
    for (int e = tid; e < (i_end - i0) * G * dv; e += NT) {
      const int c = e % dv, r = e / dv;
      const int g = r % G, i = i0 + r / G;
      a.out[(out_row0 + static_cast<long long>(i) * a.n_q + g) * dv + c] = 0.f;
    }
    return;
  }

  const int pitch_k = EB * dk, pitch_v = EB * dv;  // bytes, in the cache
  const float scale_l2e = Q8 ? a.scale_log2e * a.k_scale[h] : a.scale_log2e;
  const long long slab = static_cast<long long>(b) * a.n_kv + h;
  const bool paged = a.block_table != nullptr;
  const unsigned char* kcache = reinterpret_cast<const unsigned char*>(a.k_cache);
  const unsigned char* vcache = reinterpret_cast<const unsigned char*>(a.v_cache);
  // row of the cache (all slabs, or all pages, counted through) where logical row `row` lies; a
  // page number outside the pool is clamped into it
  auto tile_row = [&](int row) -> long long {
    if (!paged) return slab * a.cap + row;
    int pg = a.block_table[static_cast<long long>(b) * a.max_pages + (row >> a.page_shift)];
    pg = pg < 0 ? 0 : (pg >= a.n_pages ? a.n_pages - 1 : pg);
    return ((static_cast<long long>(pg) * a.n_kv + h) << a.page_shift) + (row & ((1 << a.page_shift) - 1));
  };
  const long long all_rows = paged ? (static_cast<long long>(a.n_pages) * a.n_kv) << a.page_shift
                                   : static_cast<long long>(a.batch) * a.n_kv * a.cap;
  // rows below len8 are readable: <= cache_cap, a multiple of 8 (of 16 for one-byte elements)
  const int len8 = Q8 ? (len + 15) & ~15 : (len + 7) & ~7;

  // ---- tile loads.  A thread's load j covers 16-byte slot (or piece) c = j * NT + tid of the tile:
  // offset of its source inside the cache tile, or beyond any tile where there is nothing to load.
  int kgo[NLK], vgo[NLV];
#pragma unroll
  for (int j = 0; j < NLK; ++j) kgo[j] = prefill_piece_offset(j * NT + tid, K_DIRECT ? SLK : PCK, pitch_k, K_DIRECT);
#pragma unroll
  for (int j = 0; j < NLV; ++j) vgo[j] = prefill_piece_offset(j * NT + tid, V_DIRECT ? SLV : PCV, pitch_v, V_DIRECT);
  // LDS address of this wavefront's first slot
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_ptr_t)smem))) + 1024 * wave;
  // one tile straight into LDS at `area`: `src` its first byte, `rows` those that are readable, `follow`:
  // more rows of the cache come behind them
  auto load_direct = [&](const int* off, auto n_loads, auto wave_loads, const unsigned char* src, int rows, int pitch, bool follow, int area) {
    const int bytes = rows * pitch;
    if (follow && rows == kPrefillTile) {
      static_for<decltype(n_loads)::value>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if (j * NW + NW <= decltype(wave_loads)::value || j * NW + wave < decltype(wave_loads)::value)
          load_to_lds(src, off[j], lds0 + area + j * NT * 16);
      });
    } else {
      static_for<decltype(n_loads)::value>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const int o = off[j];
        if (o < bytes && prefill_piece_whole(o, bytes, follow)) load_to_lds(src, o, lds0 + area + j * NT * 16);
        if (o < bytes && !prefill_piece_whole(o, bytes, follow))          // the cache ends inside this piece (whole dwords)
          for (int i = 0; i < bytes - o; i += 4)
            *reinterpret_cast<uint32_t*>(smem + area + (j * NT + tid) * 16 + i) = *reinterpret_cast<const uint32_t*>(src + o + i);
      });
    }
  };
  auto load_regs = [&](const int* off, auto n_loads, const unsigned char* src, int bytes, bool follow, uint4* st) {
    static_for<decltype(n_loads)::value>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      const int o = off[j];
      if (o < bytes) {
        if (prefill_piece_whole(o, bytes, follow)) {
          const Bytes16 v = *reinterpret_cast<const Bytes16*>(src + o);
          st[j] = make_uint4(v.w[0], v.w[1], v.w[2], v.w[3]);
        } else {
          uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (i < bytes - o) w[i >> 2] |= static_cast<uint32_t>(src[o + i]) << (8 * (i & 3));
          st[j] = make_uint4(w[0], w[1], w[2], w[3]);
        }
      }
    });
  };
  // register pieces to their LDS rows (codes widened)
  auto park = [&](auto n_loads, auto pieces, auto pitch, const uint4* st, unsigned char* area) {
    constexpr int PC = decltype(pieces)::value, LP = decltype(pitch)::value;
    static_for<decltype(n_loads)::value>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      const int c = j * NT + tid, row = c / PC, piece = c - row * PC;
      if (row < kPrefillTile) {
        if constexpr (Q8) {
          uint4* dst = reinterpret_cast<uint4*>(area + row * LP + 32 * piece);
          dst[0] = widen_e4m3x8(st[j].x, st[j].y);
          dst[1] = widen_e4m3x8(st[j].z, st[j].w);
        } else {
          *reinterpret_cast<uint4*>(area + row * LP + 16 * piece) = st[j];
        }
      }
    });
  };
  uint4 kst[K_DIRECT ? 1 : NLK], vst[V_DIRECT ? 1 : NLV];
  if constexpr (!K_DIRECT) static_for<NLK>([&](auto j) { kst[decltype(j)::value] = make_uint4(0, 0, 0, 0); });
  if constexpr (!V_DIRECT) static_for<NLV>([&](auto j) { vst[decltype(j)::value] = make_uint4(0, 0, 0, 0); });
  auto issue_k = [&](int t, long long trow) {
    const int rows = min(kPrefillTile, len8 - t * kPrefillTile);
    const bool follow = prefill_rows_follow(trow, rows, all_rows);
    if constexpr (K_DIRECT) load_direct(kgo, std::integral_constant<int, NLK>(), std::integral_constant<int, SLK>(), kcache + trow * pitch_k, rows, pitch_k, follow, (t & 1) * KBUF);
    else load_regs(kgo, std::integral_constant<int, NLK>(), kcache + trow * pitch_k, rows * pitch_k, follow, kst);
  };
  auto issue_v = [&](int t, long long trow) {
    const int rows = min(kPrefillTile, len8 - t * kPrefillTile);
    const bool follow = prefill_rows_follow(trow, rows, all_rows);
    if constexpr (V_DIRECT) load_direct(vgo, std::integral_constant<int, NLV>(), std::integral_constant<int, SLV>(), vcache + trow * pitch_v, rows, pitch_v, follow, 2 * KBUF + (t & 1) * VBUF);
    else load_regs(vgo, std::integral_constant<int, NLV>(), vcache + trow * pitch_v, rows * pitch_v, follow, vst);
  };
  // start row of a tile, looked up (paged) one tile ahead of its loads
  auto row_of_tile = [&](int t) -> long long { return t < n_tiles ? tile_row(t * kPrefillTile) : 0; };
  {
    const long long trow = row_of_tile(t_first);
    issue_k(t_first, trow);
    issue_v(t_first, trow);
  }
  long long trow_next = row_of_tile(t_first + 1);

  // ---- this lane's columns: (token, head) pairs, and their positions
  int pos_col[NB];
  bool col_valid[NB];
  int wmin = 0x7fffffff, wmax = -1;
  bf16x8 qf[NB][KS];                       // query columns as the B operand: lane (l16 = column, lg = k sub-chunk)
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int cw = (wave * NB + nb) * 16 + l16;
    const int tl = cw / G, g = cw - (cw / G) * G;
    const int i = i0 + tl;
    col_valid[nb] = tl < BT && i < a.n_new && shift + i >= 0;
    pos_col[nb] = col_valid[nb] ? shift + i : 0;
    wmin = min(wmin, col_valid[nb] ? pos_col[nb] : 0x7fffffff);
    wmax = max(wmax, col_valid[nb] ? pos_col[nb] : -1);
    const uint32_t* qrow = reinterpret_cast<const uint32_t*>(a.q) +
                           ((static_cast<long long>(b) * a.n_new + (col_valid[nb] ? i : 0)) * a.n_q + h * G +
                            (col_valid[nb] ? g : 0)) * (dk / 2);
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      uint32_t w[4];
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        const int e = 32 * kk + 8 * lg + 2 * e2;
        w[e2] = (col_valid[nb] && e < dk) ? qrow[e >> 1] : 0u;
      }
      qf[nb][kk] = __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
    }
  }
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    wmin = min(wmin, __shfl_xor(wmin, o));
    wmax = max(wmax, __shfl_xor(wmax, o));
  }
  wmin = __builtin_amdgcn_readfirstlane(wmin);
  wmax = __builtin_amdgcn_readfirstlane(wmax);

  f32x4 acc[NB][CT];
  float m_run[NB], l_run[NB];
  float nref[NB];      // minus the reference as the exponent's addend: kept beside m_run, 0 while that is -inf
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    m_run[nb] = -INFINITY;
    nref[nb] = 0.f;
    l_run[nb] = 0.f;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[nb][ct][r] = 0.f;
  }

  // elements of this lane's last K fragment that exist
  const int klim = dk - 32 * (KS - 1) - 8 * lg;
  const bool one_slot = ONES && l16 == 15;
  const int koff = l16 * LPK + 16 * lg;
  const int voff = 2 * KBUF + (4 * lg + (l16 >> 2)) * LPV + 8 * (l16 & 3);

  // rows 16 rt .. + 15, elements 32 kk .. + 31 of the key group that starts `base` bytes into smem
  auto k_frag = [&](int base, auto rc, auto kc) -> bf16x8 {
    constexpr int rt = decltype(rc)::value, kk = decltype(kc)::value;
    uint4 w = *reinterpret_cast<const uint4*>(smem + base + koff + 16 * rt * LPK + 64 * kk);
    if constexpr (kk == KS - 1) {                         // beyond d_k lies the next row (or stale LDS)
      w.x = klim > 0 ? w.x : 0u;
      w.y = klim > 2 ? w.y : 0u;
      w.z = klim > 4 ? w.z : 0u;
      w.w = klim > 6 ? w.w : 0u;
    }
    return __builtin_bit_cast(bf16x8, w);
  };
  // V^T operand: channels 16 ct .. + 15 of the group's 32 keys
  auto v_frag = [&](int base, auto cc) -> bf16x8 {
    constexpr int ct = decltype(cc)::value;
    unsigned char* p = smem + base + voff + 32 * ct;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t)(p + 16 * LPV));
    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
  };
  // the spare channel's lanes of the last tile's operand become 1
  auto with_ones = [&](bf16x8 v) -> bf16x8 {
    uint4 w = __builtin_bit_cast(uint4, v);
    w.x = one_slot ? 0x3f803f80u : w.x;
    w.y = one_slot ? 0x3f803f80u : w.y;
    w.z = one_slot ? 0x3f803f80u : w.z;
    w.w = one_slot ? 0x3f803f80u : w.w;
    return __builtin_bit_cast(bf16x8, w);
  };

  for (int t = t_first; t < n_tiles; ++t) {
    const int kbase0 = (t & 1) * KBUF, vbase0 = (t & 1) * VBUF;
    __builtin_amdgcn_s_waitcnt(0);         // this wavefront's share of tile t has landed
    if constexpr (!K_DIRECT) park(std::integral_constant<int, NLK>(), std::integral_constant<int, PCK>(), std::integral_constant<int, LPK>(), kst, smem + kbase0);
    if constexpr (!V_DIRECT) park(std::integral_constant<int, NLV>(), std::integral_constant<int, PCV>(), std::integral_constant<int, LPV>(), vst, smem + 2 * KBUF + vbase0);
    __syncthreads();                       // everybody's has, and nobody still reads the other buffer
    if (t + 1 < n_tiles) {
      issue_k(t + 1, trow_next);
      issue_v(t + 1, trow_next);
    }
    trow_next = row_of_tile(t + 2);
    if ((t + 1) * kPrefillTile > len) {
      // The V rows at or beyond the sequence length may hold anything (NaN included) and a zero
      // probability does not silence a NaN: in the one tile that holds the end of the sequence
      // they are cleared in LDS before use.
      for (int o = (len - t * kPrefillTile) * LPV + 16 * tid; o < VBUF; o += 16 * NT)
        *reinterpret_cast<uint4*>(smem + 2 * KBUF + vbase0 + o) = make_uint4(0, 0, 0, 0);
      __syncthreads();
    }
#pragma unroll 1
    for (int sub = 0; sub < kPrefillTile / 32; ++sub) {
      const int sbase = t * kPrefillTile + 32 * sub;
      if (sbase > wmax || sbase >= n_keys) break;   // nothing of this or any later key group is visible here
      const int kbase = kbase0 + sub * 32 * LPK, vbase = vbase0 + sub * 32 * LPV;

      // ---- A. scores S[nb][rt][r] = column (nb, l16) . K[sbase + 16 rt + 4 lg + r]
      f32x4 S[NB][2];
      static_for<2>([&](auto rt) {
        static_for<KS>([&](auto kk) {
          const bf16x8 kf = k_frag(kbase, rt, kk);
          static_for<NB>([&](auto nb) {
            constexpr int n = decltype(nb)::value, r = decltype(rt)::value, k = decltype(kk)::value;
            S[n][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[n][k], k == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : S[n][r], 0, 0, 0);
          });
        });
      });
      // ---- B. the visibility test where the group straddles the diagonal of this wavefront's
      // columns, block maxima, and the rare move of a reference.  With all 32 keys visible and a
      // non-negative scale the raw scores stay as they are: scale and reference then fold into
      // one multiply-add per score (mul), and the maximum is scaled instead of the scores.
      const bool no_mask = sbase + 31 <= wmin;
      const bool raw = no_mask && scale_l2e >= 0.f;
      const float mul = raw ? scale_l2e : 1.f;
      if (!raw) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const int rel = (no_mask ? 32 : pos_col[nb] - sbase) - 4 * lg;   // keys 0 .. rel + 4 lg of the group are visible to this column
#pragma unroll
          for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) S[nb][rt][r] = (16 * rt + r) <= rel ? S[nb][rt][r] * scale_l2e : -INFINITY;
        }
      }
      float tmax[NB];
      bool grow = false;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        tmax[nb] = max3(max3(S[nb][0][0], S[nb][0][1], S[nb][0][2]), max3(S[nb][0][3], S[nb][1][0], S[nb][1][1]),
                        max3(S[nb][1][2], S[nb][1][3], S[nb][1][3])) * mul;
        grow = grow || tmax[nb] > m_run[nb] + kHeadroomP;
      }
      if (__any(grow)) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          float tm = fmaxf(tmax[nb], __shfl_xor(tmax[nb], 16));   // the column's other keys
          tm = fmaxf(tm, __shfl_xor(tm, 32));
          const float m_new = fmaxf(m_run[nb], tm);
          // a column that has seen nothing yet and sees nothing here keeps its -inf reference
          const float alpha = m_new > -INFINITY ? __builtin_amdgcn_exp2f(m_run[nb] - m_new) : 0.f;
          l_run[nb] *= alpha;
#pragma unroll
          for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[nb][ct][r] *= alpha;
          m_run[nb] = m_new;
          nref[nb] = m_new > -INFINITY ? -m_new : 0.f;      // -inf - -inf would be NaN
        }
      }

      // ---- C. numerators, packed straight into the P.V operand: a bf16 head and a bf16 remainder
      // of every probability (16 significant bits).  The remainder is p minus the head widened
      // back (a shift or a mask, then a subtraction: exact).
      uint4 p_hi[NB], p_lo[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        float pr[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) pr[j] = __builtin_amdgcn_exp2f(fmaf(S[nb][j >> 2][j & 3], mul, nref[nb]));
        if constexpr (!ONES)                         // otherwise the sum comes out of the P.V product
          l_run[nb] += ((pr[0] + pr[1]) + (pr[2] + pr[3])) + ((pr[4] + pr[5]) + (pr[6] + pr[7]));
        uint32_t* ph = reinterpret_cast<uint32_t*>(&p_hi[nb]);
        uint32_t* pl = reinterpret_cast<uint32_t*>(&p_lo[nb]);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const uint32_t hh = pack_bf16(pr[2 * d], pr[2 * d + 1]);
          ph[d] = hh;
          pl[d] = pack_bf16(pr[2 * d] - bf16_lo(hh), pr[2 * d + 1] - bf16_hi(hh));
        }
      }

      // ---- D. P.V: acc[nb][ct][r] is channel 16 ct + 4 lg + r of column (nb, l16).  Heads of all
      // column blocks first, remainders after: an accumulator's two instructions then lie NB apart.
      static_for<CT>([&](auto cc) {
        constexpr int ct = decltype(cc)::value;
        bf16x8 vf = v_frag(vbase, cc);
        if constexpr (ONES && ct == CT - 1) vf = with_ones(vf);
        static_for<NB>([&](auto nb) {
          constexpr int n = decltype(nb)::value;
          acc[n][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8, p_hi[n]), acc[n][ct], 0, 0, 0);
        });
        static_for<NB>([&](auto nb) {
          constexpr int n = decltype(nb)::value;
          acc[n][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8, p_lo[n]), acc[n][ct], 0, 0, 0);
        });
      });
    }
  }

  // ---- normalise and store: register r of lane (l16, lg) is channel 4 lg + r of the tile, of column
  // l16: four adjacent channels
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int cw = (wave * NB + nb) * 16 + l16;
    const int tl = cw / G, g = cw - (cw / G) * G;
    const int i = i0 + tl;
    float l = l_run[nb];
    if constexpr (ONES) {
      l = __shfl(acc[nb][CT - 1][3], l16 + 48);      // the spare slot
    } else {
      l += __shfl_xor(l, 16);
      l += __shfl_xor(l, 32);
    }
    if (tl < BT && i < a.n_new) {
      const long long row = out_row0 + static_cast<long long>(i) * a.n_q + g;
      float mul;
      float* dst;
      bool live = true;
      if (in_ranges) {
        // partial of this key range: reference (log2 units), sum, un-normalised accumulators
        live = shift + i >= 0 && m_run[nb] > -INFINITY;
        const long long slot = row * a.n_ksplit + ks;
        if (lg == 0) {
          a.part_ml[slot * 2 + 0] = live ? m_run[nb] : -INFINITY;
          a.part_ml[slot * 2 + 1] = live ? l : 0.f;
        }
        mul = 1.f;
        dst = a.part_acc + slot * dv;
      } else {
        // a token in front of its sequence is zeros; for one that exists a sum that is not a number
        // has made the accumulators so too, and they are multiplied, not replaced, so that it shows
        // (in a call that may be cut all rows are as the combining kernel leaves them, which stores zeros there)
        live = shift + i >= 0 && (!a.as_combined || l > 0.f);
        mul = l > 0.f ? 1.f / l : 0.f;
        dst = a.out + row * dv;
      }
      if constexpr (Q8) mul *= a.v_scale[h];       // codes -> values
      static_for<CT>([&](auto cc) {
        constexpr int ct = decltype(cc)::value;
        const int c = 16 * ct + 4 * lg;
        f32x4_dw v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = live ? acc[nb][ct][e] * mul : 0.f;
        if (c + 3 < dv) {
          *reinterpret_cast<f32x4_dw*>(dst + c) = v;
        } else {
#pragma unroll
          for (int e = 0; e < 3; ++e)
            if (c + e < dv) dst[c + e] = v[e];
        }
      });
    }
  }
}

template <int KS, int CT, int MODE, bool ONES>
hipError_t launch_prefill_inst(PrefillArgs a, hipStream_t stream) {
  constexpr int NB = prefill_blocks(KS, CT);
  // key ranges were planned for a block size: it has to be this instantiation's
  if (a.n_ksplit > 1 && a.tok_per_wg != prefill_tokens_per_wg(KS, CT, a.group)) return hipErrorInvalidValue;
  a.tok_per_wg = prefill_tokens_per_wg(KS, CT, a.group);
  a.n_qblk = (a.n_new + a.tok_per_wg - 1) / a.tok_per_wg;
  constexpr size_t lds = 2 * static_cast<size_t>(kPrefillTile) * (prefill_k_pitch(KS) + prefill_v_pitch(CT));
  const long long slabs = static_cast<long long>(a.n_kv) * a.batch;
  if (a.n_ksplit <= 1) a.n_ranges = a.n_qblk * slabs <= 2 * kChipUnits ? a.n_qblk : 0;
  if (a.n_ranges > 0) a.slab_inv = prefill_inv(static_cast<int>(slabs));
  const long long n_wg = slabs * (a.n_ranges > 0 ? a.n_ranges : a.n_qblk);
  if (n_wg > 0x7fffffffLL) return hipErrorInvalidValue;
  if (lds > 64 * 1024) {
    const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(&prefill_kernel<KS, CT, MODE, ONES, NB>), static_cast<int>(lds));
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((prefill_kernel<KS, CT, MODE, ONES, NB>), dim3(static_cast<unsigned>(n_wg)), dim3(64 * kPrefillWaves), lds, stream, a);
  return hipGetLastError();
}

template <int KS, int CT>
hipError_t launch_prefill_ct(const PrefillArgs& a, hipStream_t stream) {
  const bool ones = (a.d_v & 15) != 0;              // a spare channel slot
  if (a.k_scale != nullptr)
    return ones ? launch_prefill_inst<KS, CT, kTilesCodes, true>(a, stream) : launch_prefill_inst<KS, CT, kTilesCodes, false>(a, stream);
  // rows of odd width start at odd multiples of two bytes, which the loads into LDS do not take
  // (and always leave a spare slot)
  if ((a.d_v & 1) != 0) return launch_prefill_inst<KS, CT, kTilesOddV, true>(a, stream);
  return ones ? launch_prefill_inst<KS, CT, kTilesDirect, true>(a, stream) : launch_prefill_inst<KS, CT, kTilesDirect, false>(a, stream);
}

template <int KS>
hipError_t launch_prefill_k(const PrefillArgs& a, hipStream_t stream) {
  switch ((a.d_v + 15) / 16) {
    case 1: return launch_prefill_ct<KS, 1>(a, stream);
    case 2: return launch_prefill_ct<KS, 2>(a, stream);
    case 3: return launch_prefill_ct<KS, 3>(a, stream);
    case 4: return launch_prefill_ct<KS, 4>(a, stream);
    case 5: return launch_prefill_ct<KS, 5>(a, stream);
    case 6: return launch_prefill_ct<KS, 6>(a, stream);
    case 7: return launch_prefill_ct<KS, 7>(a, stream);
    case 8: return launch_prefill_ct<KS, 8>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

}  // namespace rap

#endif  // RAP_PREFILL_KERNEL_H_
