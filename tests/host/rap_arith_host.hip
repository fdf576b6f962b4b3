// Host-side harness for the CPU tests: runs librap's own arithmetic and indexing helpers
// (paper_2602_02599_amd/csrc/rap_arith.h, the code the kernels compile) on the host, so that
// pytest can compare them with the float64 oracle and with long-double library routines, under the
// host sanitizers.  Built with hipcc's host pass only; nothing here touches a GPU.
//
//   rap_arith_host bf16      stdin: float64[n]  -> stdout: uint16[n]   f64_to_bf16_rne
//   rap_arith_host sincos    stdin: float64[n]  -> stdout: float64[2n] sincos_f64 (sin, cos)
//   rap_arith_host odd448    stdin: float64[n]  -> stdout: uint32[n]   bits of f64_to_f32_odd_clamped448
//   rap_arith_host mx4       stdin: float64[32 n] (n blocks) -> stdout: per block one byte
//                               mx_shared_exponent + 127 and 32 bytes f64_to_e2m1(x * pow2_neg(e))
//   rap_arith_host loadplan  -> text, one line per (kind, width, element size): what the decode
//                               kernel's tile loads touch; exit status 1 if any load leaves its tile,
//                               or any tile byte is fetched twice or not at all
//   rap_arith_host loadplan-trim1  the same with only the LAST load of a run trimmed (a planted
//                               mistake: bf16 K tiles whose width needs an odd number of loads
//                               then read past the tile; the tests expect this one to fail)
//   rap_arith_host place     -> text, one line per (ranges, KV heads, sequences): whether every
//                               (sequence, range, head) is placed once, and on how many of eight
//                               neighbouring compute units the first ranges of eight following
//                               sequences lie, at least; exit status 1 if placed wrongly or on fewer than 4
//   rap_arith_host place-rotated  the same with every number of ranges rotated by the sequence (a
//                               planted mistake: odd numbers then pile up)
//   rap_arith_host flat      -> text, one line per (sequences, KV heads, width, rows, range, several tokens or the one-call
//                               step, pattern of lengths): whether ranges by length cover every sequence once inside
//                               the partials' room, and the rows on the fullest of 256 compute units, in units of 128,
//                               against those of full sequences
//   rap_arith_host flat-one-length  the same with one range length for all sequences that are not equal (a planted
//                               mistake: nearly equal lengths then fill the chip worse than equal ones)
//   rap_arith_host prefill-place -> text, one line per (query blocks, slabs, key ranges, group): whether every
//                               (block, slab, range) is placed once, on how many XCDs a slab lies, and how
//                               often a query block follows a lighter one within a group of slabs
//   rap_arith_host prefill-cut -> text, one line per shape of a prefill launch in key ranges: whether every
//                               (slab, block, range) is taken once and a block's ranges make up its rows, and
//                               how often a range follows a shorter one
//   rap_arith_host pieceplan -> text, one line per (kind, element size, width): what the prefill
//                               kernel's tile loads touch, in the middle of a cache and at its end; exit
//                               status 1 if any leaves the cache, or misses a byte of a readable row
//   rap_arith_host pieceplan-whole  the same with every piece read whole (a planted mistake: the
//                               last row's last piece then runs past the end of the cache)
#include <stdio.h>
#include <string.h>

#include <vector>

#include "../../paper_2602_02599_amd/csrc/rap_prefill.hip"   // the plan; it brings rap_arith.h

// what the plan's file dispatches to
namespace rap {
hipError_t launch_prefill_ks1(const PrefillArgs&, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_prefill_ks2(const PrefillArgs&, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_prefill_ks3(const PrefillArgs&, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_prefill_ks4(const PrefillArgs&, hipStream_t) { return hipErrorInvalidValue; }
}  // namespace rap

namespace {

std::vector<double> read_doubles() {
  std::vector<double> v;
  double buf[4096];
  size_t n;
  while ((n = fread(buf, sizeof(double), 4096, stdin)) > 0) v.insert(v.end(), buf, buf + n);
  return v;
}

// One line per tile shape: the highest byte (exclusive) any issued load touches and the number of
// tile bytes no load covers, for the full tile and for every partial tile of 8 k (16 k) rows.
int loadplan(bool trim_one_only) {
  int bad = 0;
  for (int q8 = 0; q8 < 2; ++q8) {
    const int eb = q8 ? 1 : 2, row_quantum = q8 ? 16 : 8;
    for (int kind = 0; kind < 2; ++kind) {            // 0: K tile (even widths), 1: V tile
      for (int d = kind == 0 ? 2 : 1; d <= 128; d += kind == 0 ? 2 : 1) {
        const int n_ld = kind == 0 ? rap::k_tile_loads((d + 31) / 32, q8 != 0) : rap::v_tile_loads(rap::decode_v_tiles(d, q8 != 0), q8 != 0);
        const int n_trim = trim_one_only ? 1 : (kind == 0 ? rap::k_tile_trimmed(q8 != 0) : rap::v_tile_trimmed(q8 != 0));
        const int pitch = eb * d;
        for (int rows = row_quantum; rows <= 32; rows += row_quantum) {
          const bool whole = rows == 32;
          const int bytes = rows * pitch;
          std::vector<char> hit(static_cast<size_t>(1024) * n_ld + 16, 0);
          int top = 0;
          for (int j = 0; j < n_ld; ++j)
            for (int lane = 0; lane < 64; ++lane)
              if (rap::tile_load_issued(j, lane, n_ld, n_trim, bytes, whole)) {
                const int at = 1024 * j + 16 * lane;
                for (int i = 0; i < 16; ++i) hit[at + i] += 1;
                top = at + 16 > top ? at + 16 : top;
              }
          int missed = 0, twice = 0;
          for (int i = 0; i < bytes; ++i) {
            missed += hit[i] == 0;
            twice += hit[i] > 1;
          }
          printf("%s q8=%d d=%d rows=%d n_ld=%d bytes=%d top=%d missed=%d twice=%d\n", kind == 0 ? "K" : "V", q8, d, rows, n_ld,
                 bytes, top, missed, twice);
          bad += top > bytes || missed != 0 || twice != 0;
        }
      }
    }
  }
  return bad;
}

int prefill_placed() {
  int bad = 0;
  for (int slabs : {1, 3, 8, 10, 16, 24, 64, 72, 128})
    for (int n_qblk : {1, 2, 5, 10, 16, 25, 80})
      for (int group : {1, 4, 8}) {
        const int n = slabs * n_qblk;
        std::vector<int> hit(n, 0), last(static_cast<size_t>(8) * slabs, n_qblk), xcd(slabs, 0);
        int lighter = 0, wrong = 0;
        for (int wg = 0; wg < n; ++wg) {
          int qb, slab;
          rap::prefill_place(wg, n_qblk, slabs, group, &qb, &slab);
          if (qb < 0 || qb >= n_qblk || slab < 0 || slab >= slabs) return 1000000;
          hit[slab * n_qblk + qb] += 1;
          xcd[slab] |= 1 << (wg & 7);
          int& before = last[(slabs & 7) == 0 ? (wg & 7) * slabs + (slab >> 3) / group : 0];   // the group's blocks so far
          lighter += qb > before;
          before = qb;
        }
        for (int x : hit) wrong += x != 1;
        int spread = 1;
        for (int x : xcd) spread = __builtin_popcount(x) > spread ? __builtin_popcount(x) : spread;
        printf("blocks=%d slabs=%d group=%d wrong=%d xcds=%d lighter=%d\n", n_qblk, slabs, group, wrong, spread, lighter);
        bad += wrong != 0 || lighter != 0 || ((slabs & 7) == 0 && spread != 1);
      }
  return bad;
}

// The ranges of cut prefill launches: every (block, range) of every slab is taken by one workgroup, the ranges of a block
// make up its tiles, there are no more than the workspace holds, and they come longest first.
int prefill_cut_up() {
  int bad = 0;
  for (int slabs : {1, 2, 3, 4, 7, 8, 12, 16, 24, 40, 56, 64, 96, 128, 200, 383})
    for (int group : {1, 3, 4, 8, 16})
      for (int d : {32, 90, 104, 128})
        for (int n_new : {1, 5, 60, 64, 65, 300, 1000, 5000, 20000})
          for (int max_len : {3, 449, 512, 700, 2048, 5001, 32768, 100000}) {
            rap::PrefillPlan p = rap::prefill_plan(slabs, 1, group, d, d, n_new, max_len);
            if (p.slots <= 1) continue;
            std::vector<uint32_t> order(rap::kMaxOrdered, 0xffffffffu);
            rap::prefill_cut_plan(&p, slabs, group, d, d, n_new, max_len, order.data());
            const rap::PrefillCut c = {max_len, n_new, p.tok_per_wg, p.n_qblk, p.tiles_per_split};
            const uint32_t inv = rap::prefill_inv(slabs);
            int wrong = p.n_ksplit > p.slots || p.tiles_per_split < 4, unordered = 0, spread = 1;
            if (p.n_ksplit == 1) {
              wrong += p.n_ranges != p.n_qblk;
            }
            std::vector<int> hit(static_cast<size_t>(slabs) * p.n_qblk * p.n_ksplit, 0), xcd(slabs, 0);
            int before = 1 << 30;
            for (int wg = 0; wg < p.n_ranges * slabs; ++wg) {
              int nth, slab, qb, k;
              rap::prefill_place_cut(wg, p.n_ranges, slabs, inv, &nth, &slab);
              if (nth < 0 || nth >= p.n_ranges || slab < 0 || slab >= slabs) return 1000000;
              rap::prefill_range(nth, c, &qb, &k);
              if (p.n_ranges <= rap::kMaxOrdered) {
                qb = order[nth] & 0x1ff;
                k = (order[nth] >> 9) & 0x3fffff;
                if (qb < c.n_qblk) wrong += (order[nth] >> 31) != (rap::prefill_ranges(c, qb) > 1);
              }
              if (qb < 0 || qb >= c.n_qblk || k < 0 || k >= p.n_ksplit) return 1000000;
              hit[(static_cast<size_t>(slab) * c.n_qblk + qb) * p.n_ksplit + k] += 1;
              xcd[slab] |= 1 << (wg & 7);
              if (p.n_ranges <= rap::kMaxOrdered && p.n_ranges * slabs > 512) {
                const int tiles = rap::prefill_range_tiles(c, qb, k) / (c.per / 256 + 1);
                unordered += tiles > before;
                before = tiles;
              }
            }
            for (int qb = 0; qb < c.n_qblk; ++qb) {
              const int n = rap::prefill_ranges(c, qb), tokens = (qb + 1) * c.tok_per_wg < n_new ? (qb + 1) * c.tok_per_wg : n_new;
              const int rows = max_len - n_new + tokens;
              int tiles = 0;
              for (int k = 0; k < p.n_ksplit; ++k) {
                for (int s = 0; s < slabs; ++s) wrong += hit[(static_cast<size_t>(s) * c.n_qblk + qb) * p.n_ksplit + k] != (k < n);
                if (k < n && rows > 0) tiles += rap::prefill_range_tiles(c, qb, k);
                wrong += rap::prefill_blocks_beyond(c, k) < c.n_qblk - qb && k < n;
              }
              wrong += rows > 0 && tiles != (rows + 63) / 64;
            }
            for (int x : xcd) spread = __builtin_popcount(x) > spread ? __builtin_popcount(x) : spread;
            printf("slabs=%d group=%d d=%d new=%d rows=%d ranges=%d of=%d wrong=%d unordered=%d xcds=%d\n", slabs, group, d, n_new, max_len,
                   p.n_ranges, p.n_ksplit, wrong, unordered, spread);
            bad += wrong != 0 || unordered != 0 || ((slabs & 7) == 0 && spread != 1);
          }
  return bad;
}

// Prefill launches that are not cut and whose workgroups all start together: every query block of every slab is taken by one
// workgroup, and with a multiple of eight slabs a slab stays on one XCD.  Beyond 256 of them the unit that has the most
// work, counted in the blocks' places from the shortest, has no more than the longest and the shortest together.
int prefill_dealt() {
  int bad = 0;
  for (int slabs = 1; slabs <= 512; ++slabs)
    for (int n_qblk = 1; n_qblk * slabs <= 512; ++n_qblk) {
      const int n = slabs * n_qblk;
      const uint32_t inv = rap::prefill_inv(slabs);
      std::vector<int> hit(n, 0), xcd(slabs, 0), unit(256, 0);
      int wrong = 0, most = 0, spread = 1;
      for (int wg = 0; wg < n; ++wg) {
        int nth, slab;
        rap::prefill_place_cut(wg, n_qblk, slabs, inv, &nth, &slab);
        if (nth < 0 || nth >= n_qblk || slab < 0 || slab >= slabs) return 1000000;
        hit[nth * slabs + slab] += 1;
        xcd[slab] |= 1 << (wg & 7);
        unit[wg & 255] += n_qblk - nth;
      }
      for (int x : hit) wrong += x != 1;
      for (int x : xcd) spread = __builtin_popcount(x) > spread ? __builtin_popcount(x) : spread;
      for (int x : unit) most = x > most ? x : most;
      const bool uneven = n > 256 && most > n_qblk + 1;
      printf("slabs=%d blocks=%d wrong=%d xcds=%d most=%d uneven=%d\n", slabs, n_qblk, wrong, spread, most, uneven);
      bad += wrong != 0 || ((slabs & 7) == 0 && spread != 1) || uneven;
    }
  return bad;
}

// The division by an inverse that is off by a unit in the last place either way, next to every multiple of the divisor.
int flat_divided() {
  int bad = 0;
  for (int b = 1; b < rap::kFlatDivLimit; b += b < 3000 ? 1 : 1 + b / 977) {
    const float inv = rap::flat_inverse(b);
    for (float f : {std::nextafterf(inv, 0.f), inv, std::nextafterf(inv, 2.f)})
      for (long long m = 0; m <= rap::kFlatDivLimit; m += b * (1 + rap::kFlatDivLimit / b / 700))
        for (long long a = m - 1; a <= m + 1; ++a)
          if (a >= 0 && a < rap::kFlatDivLimit) bad += rap::flat_div(static_cast<int>(a), f) != a / b;
  }
  printf("division wrong=%d\n", bad);
  return bad;
}

int flat(bool one_length) {
  const int cus = 256;
  int bad = 0;
  for (int batch : {2, 3, 7, 9, 16, 22, 24, 33, 36, 40, 48, 64})
    for (int n_kv : {1, 3, 4, 8})
      for (int d_k : {90, 116})
        for (int max_len : {2500, 4096, 8192, 16384, 50001, 131072})
          for (int rows : {512, 768, 1024, 1408, 2048, 2816, 4096, 8192})
            for (int how = 0; how < 3; ++how) {             // plain, five tokens, the one-call step
              const int n_split = (max_len + rows - 1) / rows, n_tok = how == 1 ? 5 : 1;
              const rap::FlatPlan p = rap::flat_plan(batch, n_kv, d_k, n_split, rows, max_len, n_tok, how == 2, false, cus);
              // over codes the same, or ranges of a fixed length where short ones take more than one round
              const rap::FlatPlan q = rap::flat_plan(batch, n_kv, d_k, n_split, rows, max_len, n_tok, how == 2, true, cus);
              const bool rounds = batch * n_kv * n_split > cus * (d_k <= 96 ? 3 : 2);
              bad += q.wgs != (rows < 2048 && rounds ? 0 : p.wgs);
              if (p.wgs == 0) continue;
              const int most = (max_len - (how == 2 ? 1 : how == 1 ? 5 : 0) + rap::kSplitQuantum - 1) / rap::kSplitQuantum;
              const int scan_slots = p.slots - (how == 2 ? batch : 0);
              int equal = 0;                                // rows on the fullest unit where all sequences are full
              for (int pattern = 0; pattern < 9; ++pattern) {
                std::vector<int> units(batch, 0);
                int total = 0, longest = 0;
                for (int b = 0; b < batch; ++b) {
                  const int at[] = {most, b == 0 ? most - 1 : most, most - (b * 7 % 11) * most / 110, most - most * b / (4 * batch),
                                    most / 16 + (most - most / 16) * b / batch, b == 0 ? most : 1, b % 3 == 0 ? 0 : most, most / 5, 0};
                  units[b] = at[pattern];
                  total += units[b];
                  longest = units[b] > longest ? units[b] : longest;
                }
                const bool alike = rap::flat_alike(total, longest, batch) && !(one_length && pattern != 0);
                const int r = alike ? 0 : rap::flat_length(total, batch, p.wgs, [&](int len) {
                  int n = 0;
                  for (int u : units) n += (u + len - 1) / len;
                  return n;
                });
                int at = 0, wrong = 0, ranges = 0, longest_range = 0;
                for (int b = 0; b < batch; ++b) {
                  const int n = alike ? rap::flat_alike_ranges(longest, p.full, p.few) : (units[b] + r - 1) / r;
                  int from = 0;
                  for (int i = 0; i < n; ++i) {
                    const int begin = rap::flat_begin(i, n, units[b]), end = rap::flat_begin(i + 1, n, units[b]);
                    // those that hold rows come first: the combining kernel reads the first min(n, units)
                    wrong += begin != from || end < begin || (end > begin) != (i < units[b]) || (!alike && end - begin > r);
                    from = end;
                    ranges += end > begin;
                    longest_range = end - begin > longest_range ? end - begin : longest_range;
                  }
                  wrong += from != units[b] || (n < units[b] ? n : units[b]) > rap::flat_most(p, most);
                  at += n;
                }
                wrong += at > scan_slots || p.slots > batch * (n_split + 1);
                const int fullest = (ranges * n_kv + cus - 1) / cus * longest_range;
                if (pattern == 0) equal = fullest;
                // lengths within a tenth of each other: no more on any unit than with full ones (the chip is full with both)
                const bool near = pattern <= 2;
                printf("sequences=%d heads=%d d_k=%d rows=%d range=%d how=%d pattern=%d ranges=%d of=%d wrong=%d fullest=%d equal=%d\n", batch, n_kv,
                       d_k, max_len, rows, how, pattern, ranges, scan_slots, wrong, fullest, equal);
                bad += wrong != 0 || (near && fullest > equal);
              }
            }
  return bad;
}

int place(bool always_rotated) {
  int bad = 0;
  for (int n_kv = 1; n_kv <= 16; n_kv = n_kv < 8 ? n_kv + 1 : n_kv + 8)
    for (int n_split = 1; n_split <= 33; ++n_split)
      for (int batch : {1, 3, 8, 9, 12, 24, 64}) {
        std::vector<int> hit(static_cast<size_t>(batch) * n_split * n_kv, 0), first(batch, 0);
        for (int wg = 0; wg < batch * n_split * n_kv; ++wg) {
          int b, split, h;
          rap::decode_place(wg, n_split, n_kv, batch, &b, &split, &h);
          if (always_rotated && (n_split & 1) != 0) split = (split + b) % n_split;
          if (b < 0 || b >= batch || split < 0 || split >= n_split || h < 0 || h >= n_kv) return 1000000;
          hit[(static_cast<size_t>(b) * n_split + split) * n_kv + h] += 1;
          if (split == 0 && h == 0) first[b] = wg / n_kv;         // its turn among the workgroups of an XCD
        }
        int wrong = 0, units = 8;
        for (int x : hit) wrong += x != 1;
        for (int b = 0; batch > 8 && n_split >= 4 && b + 8 <= batch; ++b) {
          unsigned seen = 0;
          for (int i = 0; i < 8; ++i) seen |= 1u << (first[b + i] & 7);
          units = __builtin_popcount(seen) < units ? __builtin_popcount(seen) : units;
        }
        printf("ranges=%d heads=%d sequences=%d wrong=%d units=%d\n", n_split, n_kv, batch, wrong, units);
        bad += wrong != 0 || units < 4;
      }
  return bad;
}

// The pieces of a tile as prefill_kernel walks them: straight into LDS (slots of padded rows: bf16,
// even widths) or through registers.  `over`: bytes read beyond what exists behind the tile, `missed`:
// bytes of readable rows that no piece covers, `idle`: slots of a whole tile, loaded without a lane
// mask, that have nothing to load.
int pieceplan(bool read_whole) {
  int bad = 0;
  for (int eb = 1; eb <= 2; ++eb) {
    const int quantum = eb == 1 ? 16 : 8;                         // rows come in such groups, and so do capacities
    for (int kind = 0; kind < 2; ++kind) {                        // 0: K tile (even widths), 1: V tile
      for (int d = kind == 0 ? 2 : 1; d <= 128; d += kind == 0 ? 2 : 1) {
        const int pitch = eb * d;
        const bool direct = eb == 2 && (d & 1) == 0;
        const int per_row = kind == 0 ? (direct ? 4 * ((d + 31) / 32) + 1 : 2 * ((d + 31) / 32))
                                      : (direct ? 2 * ((d + 15) / 16 | 1) : (eb == 1 ? 1 : 2) * ((d + 15) / 16));
        int over = 0, missed = 0, idle = 0;
        for (int rows = quantum; rows <= rap::kPrefillTile; rows += quantum) {
          for (int groups_behind = 0; groups_behind < 2; ++groups_behind) {
            const bool follow = rap::prefill_rows_follow(1000 * quantum, rows, 1000 * quantum + rows + groups_behind * quantum);
            const int bytes = rows * pitch, exist = bytes + groups_behind * quantum * pitch;
            std::vector<char> hit(static_cast<size_t>(rap::kPrefillTile) * pitch + 64, 0);
            const int slots = (rap::kPrefillTile * per_row + 255) / 256 * 256;
            for (int c = 0; c < slots; ++c) {
              const int o = rap::prefill_piece_offset(c, per_row, pitch, direct);
              if (direct && rows == rap::kPrefillTile && follow) idle += c < rap::kPrefillTile * per_row && o == rap::kNoPiece;
              const int n = o >= bytes ? 0 : read_whole || rap::prefill_piece_whole(o, bytes, follow) ? 16 : bytes - o;
              if (n > 0 && o + n - exist > over) over = o + n - exist;
              for (int i = 0; i < n; ++i) hit[o + i] = 1;
            }
            for (int i = 0; i < bytes; ++i) missed += hit[i] == 0;
          }
        }
        printf("%s eb=%d d=%d direct=%d over=%d missed=%d idle=%d\n", kind == 0 ? "K" : "V", eb, d, direct, over, missed, idle);
        bad += over > 0 || missed != 0 || idle != 0;
      }
    }
  }
  return bad;
}

}  // namespace

int main(int argc, char** argv) {
  if (argc != 2) {
    fprintf(stderr, "usage: rap_arith_host bf16|sincos|odd448|mx4|loadplan|loadplan-trim1|pieceplan|pieceplan-whole|place|place-rotated|flat|flat-div|flat-one-length|prefill-place|prefill-cut|prefill-deal\n");
    return 2;
  }
  if (strcmp(argv[1], "loadplan") == 0) return loadplan(false) == 0 ? 0 : 1;
  if (strcmp(argv[1], "loadplan-trim1") == 0) return loadplan(true) == 0 ? 0 : 1;
  if (strcmp(argv[1], "flat-div") == 0) return flat_divided() == 0 ? 0 : 1;
  if (strcmp(argv[1], "flat") == 0) return flat(false) == 0 ? 0 : 1;
  if (strcmp(argv[1], "flat-one-length") == 0) return flat(true) == 0 ? 0 : 1;
  if (strcmp(argv[1], "prefill-place") == 0) return prefill_placed() == 0 ? 0 : 1;
  if (strcmp(argv[1], "prefill-cut") == 0) return prefill_cut_up() == 0 ? 0 : 1;
  if (strcmp(argv[1], "prefill-deal") == 0) return prefill_dealt() == 0 ? 0 : 1;
  if (strcmp(argv[1], "place") == 0) return place(false) == 0 ? 0 : 1;
  if (strcmp(argv[1], "place-rotated") == 0) return place(true) == 0 ? 0 : 1;
  if (strcmp(argv[1], "pieceplan") == 0) return pieceplan(false) == 0 ? 0 : 1;
  if (strcmp(argv[1], "pieceplan-whole") == 0) return pieceplan(true) == 0 ? 0 : 1;
  const std::vector<double> in = read_doubles();
  if (strcmp(argv[1], "bf16") == 0) {
    std::vector<uint16_t> out(in.size());
    for (size_t i = 0; i < in.size(); ++i) out[i] = rap::f64_to_bf16_rne(in[i]);
    fwrite(out.data(), sizeof(uint16_t), out.size(), stdout);
  } else if (strcmp(argv[1], "sincos") == 0) {
    std::vector<double> out(2 * in.size());
    for (size_t i = 0; i < in.size(); ++i) rap::sincos_f64(in[i], &out[2 * i], &out[2 * i + 1]);
    fwrite(out.data(), sizeof(double), out.size(), stdout);
  } else if (strcmp(argv[1], "odd448") == 0) {
    std::vector<uint32_t> out(in.size());
    for (size_t i = 0; i < in.size(); ++i) out[i] = rap::f32_bits(rap::f64_to_f32_odd_clamped448(in[i]));
    fwrite(out.data(), sizeof(uint32_t), out.size(), stdout);
  } else if (strcmp(argv[1], "mx4") == 0) {
    std::vector<uint8_t> out;
    for (size_t b = 0; b + 32 <= in.size(); b += 32) {
      double amax = 0.0;
      for (int i = 0; i < 32; ++i) {
        const double m = in[b + i] < 0 ? -in[b + i] : in[b + i];
        amax = m > amax ? m : amax;
      }
      const int e = rap::mx_shared_exponent(amax);
      out.push_back(static_cast<uint8_t>(e + 127));
      for (int i = 0; i < 32; ++i) out.push_back(static_cast<uint8_t>(rap::f64_to_e2m1(in[b + i] * rap::pow2_neg(e))));
    }
    fwrite(out.data(), 1, out.size(), stdout);
  } else {
    fprintf(stderr, "unknown command %s\n", argv[1]);
    return 2;
  }
  return 0;
}
