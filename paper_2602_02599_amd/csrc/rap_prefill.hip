// Causal prefill attention over the compact cache: the host-side plan of key ranges and the
// dispatch on the score width; the kernel is in rap_prefill_kernel.h.
#include "rap_device.h"

namespace rap {

hipError_t launch_prefill_ks1(const PrefillArgs& a, hipStream_t stream);
hipError_t launch_prefill_ks2(const PrefillArgs& a, hipStream_t stream);
hipError_t launch_prefill_ks3(const PrefillArgs& a, hipStream_t stream);
hipError_t launch_prefill_ks4(const PrefillArgs& a, hipStream_t stream);

// Query blocks from which on no launch is cut.
constexpr int kMostBlocks = 3 * kChipUnits / 2;

// How a call with a workspace is cut.  Nothing is cut while the query blocks number at least one and a half per
// compute unit or the context is short; else the workspace has room for about 512 workgroups, in ranges of no less than four
// tiles, which is what callers have to bring.  prefill_cut_plan then picks, within that, the ranges it expects to be
// done first.
PrefillPlan prefill_plan(int batch, int n_kv, int group, int d_k, int d_v, int n_new, int max_len) {
  PrefillPlan p;
  p.tok_per_wg = prefill_tokens_per_wg((d_k + 31) / 32, (d_v + 15) / 16, group);
  p.n_qblk = (n_new + p.tok_per_wg - 1) / p.tok_per_wg;
  p.slots = p.n_ksplit = 1;
  p.tiles_per_split = 0;
  const long long base = static_cast<long long>(p.n_qblk) * n_kv * batch;
  const int tiles = (max_len + kPrefillTile - 1) / kPrefillTile;
  if (base > 0 && base < kMostBlocks && tiles >= 8) {
    const int want = static_cast<int>((2 * kChipUnits + base - 1) / base);
    int per = (tiles + want - 1) / want;
    if (per < 4) per = 4;
    p.slots = (tiles + per - 1) / per;
    p.tiles_per_split = per;
  }
  return p;
}

namespace {

// Ranges of a slab by length, the longest first: `full` ranges of `per` tiles, then the last range of every
// block, `block` saying whose (where the launch can be told their order; else as they are counted, which is from
// the longest to the shortest for a chunk that is short beside its context).
struct CutLengths {
  int per, full, n;
  bool ordered;
  int tiles[kMostBlocks];
  uint16_t block[kMostBlocks];
  int length(int nth) const { return nth < full ? per : tiles[nth - full]; }
};
void cut_lengths(const PrefillCut& c, CutLengths* out) {
  const int ranges = prefill_ranges(c, c.n_qblk - 1);
  out->per = c.per;
  out->full = 0;
  for (int k = 1; k < ranges; ++k) out->full += prefill_blocks_beyond(c, k);
  out->n = out->full + c.n_qblk;
  out->ordered = out->n <= kMaxOrdered;
  constexpr int kClasses = 256;                    // counting sort; longer ranges than that in classes
  int first[kClasses + 1] = {0}, tiles[kMostBlocks];
  const int step = c.per / kClasses + 1;
  for (int qb = 0; qb < c.n_qblk; ++qb) {
    const int t = prefill_range_tiles(c, qb, prefill_ranges(c, qb) - 1);
    tiles[qb] = t > 0 ? t : 0;
    first[kClasses - tiles[qb] / step]++;
  }
  int at = 0;
  for (int s = 0; s <= kClasses; ++s) {
    const int m = first[s];
    first[s] = at;
    at += m;
  }
  for (int qb = c.n_qblk - 1; qb >= 0; --qb) {
    const int to = first[kClasses - tiles[qb] / step]++;
    out->tiles[to] = tiles[qb];
    out->block[to] = static_cast<uint16_t>(qb);
  }
}

// How long a launch takes, in tiles of a compute unit that holds two workgroups: `slabs` times those ranges, placed by
// prefill_place_cut.  A workgroup alone on its unit runs at 1 / alone of what two of them do together: 1.22 with four
// column blocks (4 x 512 tokens at 8192 rows: 356 us in 256 workgroups, 294 in 512 of half the rows), 1.5 with three
// (360 tokens at 6677 rows, 112/93: 87 us in 264 workgroups of 26 tiles, 74 in 512 of 14).
double slowest_unit(const CutLengths& l, int slabs, double alone) {
  const int all = l.n * slabs;
  double worst = alone * l.length(0);
  if (all <= kChipUnits) return worst;
  if (all <= 2 * kChipUnits) {
    for (int j = 0; j < all - kChipUnits; j += slabs < 8 ? 1 : 8) {
      const double t = l.length((2 * kChipUnits - all + j) / slabs) + l.length((all - 1 - j) / slabs);
      worst = t > worst ? t : worst;
    }
    return worst;
  }
  // more than fit: each of the places takes the longest that is left when it is free; places in groups
  // that are free at the same time
  struct Group { double t; int n; };
  constexpr int kGroups = 64;
  Group free_[kGroups];
  int lo = 0, hi = 1;
  free_[0] = {0.0, 2 * kChipUnits};
  worst = 0.0;
  for (int i = 0; i < l.n;) {
    const int tiles = l.length(i);
    int j = i;
    while (j < l.n && l.length(j) == tiles) ++j;
    for (int left = (j - i) * slabs; left > 0 && lo < hi;) {
      const int k = left < free_[lo].n ? left : free_[lo].n;
      const double done = free_[lo].t + 2.0 * tiles;
      worst = done > worst ? done : worst;
      left -= k;
      free_[lo].n -= k;
      if (free_[lo].n == 0) ++lo;
      if (hi < kGroups) {
        int at = hi++;
        for (; at > lo && free_[at - 1].t > done; --at) free_[at] = free_[at - 1];
        free_[at] = {done, k};
      }
    }
    i = j;
  }
  return worst;
}

}  // namespace

// What to cut into: of a few range lengths the one with the least time for its slowest unit and its partials.
// Ranges as long as the workspace allows them to be many (512 workgroups or a few more, rounded up) leave a second round of a
// few: attention calls so and as picked here (tiles of the first ranges, 32/8 heads unless said): 5 x 48 tokens at 14901
// rows, d = 86, 18 tiles 145 us, 20: 106; 3 x 512 at 8192 43 tiles 290, 52 and a last range of 24: 241; 5 x 448 at 4096 32
// tiles 228, 43 and 21: 205; 9 x 200 at 6000, 20/4 heads, 24 tiles 174, 27 and 13: 142.  Chunks as long as their context: 2 x 3014
// tokens, 12/4 heads, d = 56, 97 -> 78 us, 2048 tokens 92 -> 74, 4 x 600 tokens (left whole) 49 -> 41.
// The ten or so lengths tried cost the host 1.5 us a call, 8 where there are 370 query blocks (6000 of 6000 tokens over 4 KV heads, a
// call of 200 us on the device, 100 us less than in the first length that the workspace allows); nothing is kept from
// one call for the next.
void prefill_cut_plan(PrefillPlan* p, int slabs, int group, int d_k, int d_v, int n_new, int max_len, uint32_t* order) {
  const int ks = (d_k + 31) / 32, ct = (d_v + 15) / 16;
  const int tiles = (max_len + kPrefillTile - 1) / kPrefillTile, least = p->tiles_per_split, most = p->slots;
  PrefillCut c{max_len, n_new, p->tok_per_wg, p->n_qblk, 0};
  const double us_per_tile = 0.064 * prefill_blocks(ks, ct) * (ks + ct);
  const double alone = prefill_blocks(ks, ct) == 4 ? 1.22 : 1.5;
  // partials, written and read once (512 tokens, 32 query heads, 8 ranges: 48 MB, combined in 9.5 us)
  const double us_per_range = static_cast<double>(n_new) * group / p->n_qblk * (d_v + 2) * sizeof(float) / 4e6;
  CutLengths l, best_l;
  double best = 1e30;
  auto consider = [&](int per) {
    if (per < least || per > tiles) return;
    c.per = per;
    cut_lengths(c, &l);
    const int in_parts = prefill_blocks_beyond(c, 1);
    const double t = us_per_tile * slowest_unit(l, slabs, alone) + (in_parts > 0 ? 2.5 + us_per_range * slabs * (l.full + in_parts) : 0.0);
    if (t < best) {
      best = t;
      best_l = l;
    }
  };
  int last = 0;
  auto try_once = [&](int per) {
    if (per != last) consider(per);
    last = per;
  };
  for (int k = most; k > 0 && k > most - 3; --k) try_once((tiles + k - 1) / k);               // equal ranges
  for (int r = 2; r <= 3; ++r) try_once((tiles * r + r * (most - 1)) / (r * (most - 1) + 1)); // a short last one: r of them in the time of the others
  for (int e = 9; e <= 15; e += 2) try_once(least * e / 8);
  try_once(tiles);
  p->tiles_per_split = best_l.per;
  p->n_ranges = best_l.n;
  p->n_ksplit = (tiles + best_l.per - 1) / best_l.per;
  if (!best_l.ordered) return;
  c.per = best_l.per;
  int at = 0;
  for (int k = 0; k + 1 < p->n_ksplit; ++k)
    for (int i = prefill_blocks_beyond(c, k + 1), qb = c.n_qblk - 1; i > 0; --i, --qb) order[at++] = qb | k << 9 | 1u << 31;
  for (int i = 0; i < c.n_qblk; ++i) {
    const int k = prefill_ranges(c, best_l.block[i]) - 1;
    order[at++] = best_l.block[i] | k << 9 | (k > 0 ? 1u << 31 : 0u);
  }
}

hipError_t launch_prefill(const PrefillArgs& a, hipStream_t stream) {
  switch ((a.d_k + 31) / 32) {
    case 1: return launch_prefill_ks1(a, stream);
    case 2: return launch_prefill_ks2(a, stream);
    case 3: return launch_prefill_ks3(a, stream);
    case 4: return launch_prefill_ks4(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace rap
