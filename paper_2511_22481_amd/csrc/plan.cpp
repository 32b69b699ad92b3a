// Work partition for sparse MLA decode (host only, no HIP calls).
#include "plan.h"

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <functional>
#include <utility>

namespace omniattn {

namespace {

// What a partition costs with one of the kernels (measured on MI355X):
//   head_block  head rows per work unit;
//   tile_us  a KV tile in the long loop when all compute units work;
//   seg      a segment (page-table entries, query block, first tile, last PV, result rows), in tiles;
//   combine  the second launch that merges partial rows, with the gap in front of it (6 us), in tiles;
//   slots_per_tile  partial rows of how many slots are written and read back in a tile's time by
//            the whole chip (131 KB each per 128 rows, both ways, at 5 TB/s).
struct KernelCost {
  int head_block;
  double tile_us;
  int seg;
  double combine;
  double slots_per_tile;
};
// The kernels for blocks of 128 rows: 9 us and 13 us a segment.
constexpr KernelCost kWideBf16 = {4 * kHeadsPerWave, 1.8, 5, 3.3, 36.0};
constexpr KernelCost kWideFp8 = {4 * kHeadsPerWave, 3.5, 4, 1.8, 65.0};
// Blocks of 64 (fp8 cache) and 32 rows: every tile passes through once per block.  Fitted to nine shapes
// from 4 to 256 sequences, each timed with each kernel forced; the estimates are within 12 % of those times.
constexpr KernelCost kMidFp8 = {kHeadBlockFp8, 1.7, 8, 2.4, 65.0};
constexpr KernelCost kNarrowBf16 = {kHeadsPerWave, 1.4, 4, 4.3, 112.0};
constexpr KernelCost kNarrowFp8 = {kHeadsPerWave, 1.5, 7, 2.7, 114.0};
// Do not leave slivers shorter than this many tiles unless the item itself is shorter.
constexpr int kMinSegTiles = 2;

// Deals the items (sequence b, head block hb) in order to units of capacity `cap` (tiles plus `seg` per
// segment), cutting an item where a unit is full.  emit(b, hb, tile_lo, tile_hi, unit) for every segment;
// returns the number of units used.
template <typename Emit>
int fill_units(const std::vector<int32_t>& tiles, int n_hb, int cap, int seg, Emit emit) {
  int load = 0, unit = 0;
  auto close_unit = [&]() {
    if (load > 0) {
      ++unit;
      load = 0;
    }
  };
  for (int b = 0; b < (int)tiles.size(); ++b)
    for (int hb = 0; hb < n_hb; ++hb) {
      const int ntiles = tiles[b];
      if (ntiles == 0) {  // empty retained set: one segment that only writes zeros / -inf
        if (load + seg > cap) close_unit();
        emit(b, hb, 0, 0, unit);
        load += seg;
        continue;
      }
      int done = 0;
      while (done < ntiles) {
        const int rem = ntiles - done;
        int room = cap - load - seg;
        const int need = std::min(rem, kMinSegTiles);
        if (room < need) {
          if (load == 0) room = need;  // capacity smaller than one minimal segment
          else { close_unit(); continue; }
        }
        int take = std::min(std::min(rem, room), kMaxSegTiles);
        // avoid leaving a sliver behind
        if (rem - take > 0 && rem - take < kMinSegTiles) take = std::max(1, rem - kMinSegTiles);
        emit(b, hb, done, done + take, unit);
        done += take;
        load += take + seg;
        if (load >= cap) close_unit();
      }
    }
  close_unit();
  return unit;
}

// Work partition over `num_cus` compute units that all start together: the launch lasts as long
// as its longest unit, and one more launch follows if any item was cut.  Three shapes are
// estimated with the costs above and the cheapest is taken:
//   whole  items dealt whole, largest first, to the unit with the least work: nothing to merge.
//          Wins when items of one size come close to a multiple of the unit count (256 sequences
//          of 133 tiles on 256 units: 137 against 143 + merge);
//   even   every item cut into equal pieces, one piece per unit: wins for a few equal items (32
//          sequences of 130 tiles: eight pieces of 16 or 17, where filling units to the brim
//          leaves some with the ends of two sequences, which cost them a second start);
//   fill   units filled one after the other to the same load, items cut wherever that falls: wins
//          when the item count is not near a multiple or divisor of the unit count.
//
// The estimates come first and only the partition that is taken is laid out: a serving loop plans again
// for every decode step, and searching the fill of three kernels to the end took 30 us of host time
// (40 sequences) where this takes 5.
struct Shape {
  enum { kFill, kWhole, kEven } kind = kFill;
  int size = 0;                  // kFill: capacity of a unit; kEven: tiles of a piece
  int64_t slots = 0;             // partial rows it leaves
  double us = INFINITY;
  std::vector<int32_t> unit_of;  // kWhole: unit of every item (empty: one item to a unit)
};

// `tiles`: per sequence; every sequence is n_hb items of that many.  `most_slots`: partial slots that fit
// the built-in scratch buffer; even pieces are not cut so short that omniattn_decode_static would refuse
// the plan.  Returns an estimate of `limit_us` or more when nothing below it exists.
Shape choose_shape(const std::vector<int32_t>& tiles, int n_hb, int num_cus, const KernelCost& cost, int most_slots,
                   double limit_us) {
  Shape r;
  const int n = (int)tiles.size() * n_hb;
  int64_t sum = 0;
  int n_max = 0;
  for (int t : tiles) {
    sum += t;
    n_max = std::max(n_max, t);
  }
  sum *= n_hb;
  auto merge_cost = [&](int64_t slots) { return slots ? cost.combine + slots / cost.slots_per_tile : 0.0; };
  // Tile counts with how often they occur: windows make most sequences alike, and the sums over all items
  // below are then sums over a few entries.
  std::vector<std::pair<int32_t, int32_t>> counts;
  counts.reserve(tiles.size());
  for (int t : tiles) {
    const size_t known = std::min<size_t>(counts.size(), 16);
    size_t k = 0;
    while (k < known && counts[k].first != t) ++k;
    if (k < known) ++counts[k].second;
    else counts.emplace_back(t, 1);
  }
  auto pieces_at = [&](int p) {  // pieces of at most p tiles
    int64_t k = 0;
    for (const auto& c : counts) k += (int64_t)(c.first > p ? (c.first + p - 1) / p : 1) * c.second;
    return k * n_hb;
  };
  auto cut_pieces_at = [&](int p) {  // those of items that are cut
    int64_t k = 0;
    for (const auto& c : counts)
      if (c.first > p) k += (int64_t)((c.first + p - 1) / p) * c.second;
    return k * n_hb;
  };
  double best = limit_us / cost.tile_us;  // in tiles, as all below
  bool found = false;
  auto take = [&](double t) {
    if (t >= best) return false;
    best = t;
    return found = true;
  };
  // (some unit has at least the average tiles, and a segment)
  if ((double)sum / num_cus + cost.seg >= best) return r;

  // whole (a segment's tile table holds kMaxSegTiles)
  if (n_max <= kMaxSegTiles) {
    if (n <= num_cus) {
      if (take(n_max + cost.seg)) r.kind = Shape::kWhole;
    } else if ((double)(sum + (int64_t)n * cost.seg) / num_cus < best && n_max + cost.seg < best) {
      std::vector<int32_t> order(n), unit_of(n);
      for (int i = 0; i < n; ++i) order[i] = i;
      std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return tiles[a / n_hb] > tiles[b / n_hb]; });
      std::vector<std::pair<int32_t, int32_t>> heap;  // (load, unit), least loaded on top
      heap.reserve(num_cus);
      const auto later = std::greater<std::pair<int32_t, int32_t>>();
      int longest = 0;
      for (int i = 0; i < n && longest < best; ++i) {
        const int cost_i = tiles[order[i] / n_hb] + cost.seg;
        int unit = i, load = cost_i;
        if (i < num_cus) {
          heap.emplace_back(load, unit);
          if (i == num_cus - 1) std::make_heap(heap.begin(), heap.end(), later);
        } else {
          std::pop_heap(heap.begin(), heap.end(), later);
          unit = heap.back().second;
          load = heap.back().first += cost_i;
          std::push_heap(heap.begin(), heap.end(), later);
        }
        unit_of[order[i]] = unit;
        longest = std::max(longest, load);
      }
      if (take(longest)) {
        r.kind = Shape::kWhole;
        r.unit_of = std::move(unit_of);
      }
    }
  }
  // even: the smallest piece that needs no more pieces than there are units
  if (n <= num_cus && n_max > 1) {
    int bad = (int)((sum - 1) / num_cus), good = n_max;  // (shorter pieces than the average are too many; one piece per item fits)
    while (good - bad > 1) {
      const int mid = bad + (good - bad) / 2;
      (pieces_at(mid) > num_cus ? bad : good) = mid;
    }
    // (with few items the shortest pieces give more partial rows than they save tiles: sum / p
    // slots cost sum / p / slots_per_tile, which balances p at the square root below)
    const int balanced = (int)std::sqrt((double)sum / cost.slots_per_tile);
    for (int p : {good, std::max(good, balanced), 2 * good}) {
      p = std::min({p, n_max, kMaxSegTiles});
      if (p + cost.seg >= best || pieces_at(p) > num_cus) continue;
      const int64_t slots = cut_pieces_at(p);
      if (slots <= most_slots && take(p + cost.seg + merge_cost(slots))) {
        r.kind = Shape::kEven;
        r.size = p;
        r.slots = slots;
      }
    }
  }
  // fill: the smallest capacity that needs no more units than there are, if one can win at all
  auto units_at = [&](int cap) { return fill_units(tiles, n_hb, cap, cost.seg, [](int, int, int, int, int) {}); };
  int lo = (int)std::min<int64_t>((sum + (int64_t)n * cost.seg + num_cus - 1) / num_cus, INT32_MAX / 2);
  lo = std::max(lo, cost.seg + 1);
  // (a capacity that gives no more than whole items may come without a merge; then `whole` is as good)
  const double cap_max = found || best < INFINITY ? best - cost.combine : INFINITY;
  // (a capacity c gives segments of at most c - seg tiles: at least that many of them, and slots)
  bool worth_it = cap_max == INFINITY;
  for (int c = lo; !worth_it && c < cap_max; ++c) {
    if (sum + cost.seg * pieces_at(c - cost.seg) > (int64_t)num_cus * c) {
      if (c == lo) ++lo;
      continue;
    }
    worth_it = c + merge_cost(cut_pieces_at(c - cost.seg)) < best;
  }
  int cap = 0;
  if (worth_it) {  // upwards from the bound, which is close, then back to the smallest
    int bad = lo - 1, step = 1;
    while (lo < cap_max && step < (1 << 28) && units_at(lo) > num_cus) {
      bad = lo;
      lo += step;
      step *= 2;
    }
    if (lo < cap_max) {
      cap = lo;
      while (cap - bad > 1) {
        const int mid = bad + (cap - bad) / 2;
        (units_at(mid) > num_cus ? bad : cap) = mid;
      }
    }
  }
  if (cap > 0) {
    int64_t slots = 0;
    int longest = 0, load = 0, last_unit = -1;
    fill_units(tiles, n_hb, cap, cost.seg, [&](int b, int, int lo_t, int hi_t, int unit) {
      if (hi_t - lo_t < tiles[b]) ++slots;
      load = (unit == last_unit ? load : 0) + hi_t - lo_t + cost.seg;
      last_unit = unit;
      longest = std::max(longest, load);
    });
    if (take(longest + merge_cost(slots))) {
      r.kind = Shape::kFill;
      r.size = cap;
      r.slots = slots;
    }
  }
  if (found) r.us = best * cost.tile_us;
  return r;
}

void lay_out(const Shape& shape, const std::vector<int32_t>& tiles, int n_hb, int num_cus, const KernelCost& cost,
             std::vector<Segment>& segs, std::vector<int32_t>& unit_seg) {
  segs.clear();
  segs.reserve(2 * (size_t)num_cus + tiles.size() * n_hb);
  unit_seg.reserve(num_cus + 1);
  unit_seg.assign(1, 0);
  auto add = [&](int b, int hb, int lo, int hi, int unit) {
    while ((int)unit_seg.size() <= unit) unit_seg.push_back((int32_t)segs.size());
    segs.push_back({b, hb, lo, hi, -1, unit, 0, tiles[b]});
  };
  const int batch = (int)tiles.size(), n = batch * n_hb;
  if (shape.kind == Shape::kFill) {
    fill_units(tiles, n_hb, shape.size, cost.seg, add);
  } else if (shape.kind == Shape::kEven) {
    int unit = 0;
    for (int b = 0; b < batch; ++b) {
      const int t = tiles[b], k = std::max(1, (t + shape.size - 1) / shape.size);
      for (int hb = 0; hb < n_hb; ++hb)
        for (int s = 0; s < k; ++s) add(b, hb, (int)((int64_t)t * s / k), (int)((int64_t)t * (s + 1) / k), unit++);
    }
  } else if (shape.unit_of.empty()) {
    for (int i = 0; i < n; ++i) add(i / n_hb, i % n_hb, 0, tiles[i / n_hb], i);
  } else {
    // units in order, each with its items
    std::vector<int32_t> first(num_cus + 1, 0), at(n);
    for (int i = 0; i < n; ++i) ++first[shape.unit_of[i] + 1];
    for (int u = 0; u < num_cus; ++u) first[u + 1] += first[u];
    std::vector<int32_t> next(first.begin(), first.end() - 1);
    for (int i = 0; i < n; ++i) at[next[shape.unit_of[i]]++] = i;
    for (int u = 0; u < num_cus; ++u)
      for (int k = first[u]; k < first[u + 1]; ++k) add(at[k] / n_hb, at[k] % n_hb, 0, tiles[at[k] / n_hb], u);
  }
  unit_seg.push_back((int32_t)segs.size());
}

}  // namespace

int build_host_plan(HostPlan& hp, const omniattn_problem_t& prob, const int32_t* seq_lens,
                    int num_cus) {
  if (!seq_lens) return OMNIATTN_EINVAL;
  if (prob.batch < 1 || prob.num_heads < 1 || prob.sink < 0 || prob.window < 0 ||
      prob.max_pages_per_seq < 1 || prob.num_pages < 1 || prob.num_splits_hint < 0 || num_cus < 1)
    return OMNIATTN_EINVAL;
  if (prob.qk_dim != kQK || prob.v_dim != kV || prob.page_size != kPage) return OMNIATTN_EUNSUPPORTED;
  if (prob.kv_dtype != OMNIATTN_BF16 && prob.kv_dtype != OMNIATTN_FP8_E4M3) return OMNIATTN_EUNSUPPORTED;
  if (prob.out_dtype != OMNIATTN_BF16 && prob.out_dtype != OMNIATTN_FP32) return OMNIATTN_EUNSUPPORTED;
  if (!(prob.softmax_scale == prob.softmax_scale)) return OMNIATTN_EINVAL;  // NaN
  if (prob.q_len < 0 || prob.q_len > 64) return OMNIATTN_EINVAL;
  const int q_len = prob.q_len > 1 ? prob.q_len : 1;
  if ((int64_t)prob.num_heads * q_len > (1 << 20)) return OMNIATTN_EUNSUPPORTED;
  for (int b = 0; b < prob.batch; ++b) {
    int64_t L = seq_lens[b];
    if (L < 0) return OMNIATTN_EINVAL;
    if (L > 0 && L < q_len) return OMNIATTN_EINVAL;  // every query needs its own token in the cache
    if ((L + kPage - 1) / kPage > prob.max_pages_per_seq) return OMNIATTN_EINVAL;
  }

  hp.prob = prob;
  hp.num_cus = num_cus;
  hp.seq_lens.assign(seq_lens, seq_lens + prob.batch);
  hp.q_len = q_len;
  hp.tile = prob.kv_dtype == OMNIATTN_FP8_E4M3 ? kTileFp8 : kTile;
  hp.heads_total = prob.num_heads * q_len;
  // Several causal queries: query t keeps [0, S) and the W positions ending at its own token.
  // Over all queries that is [0, S) and (for W > 0) the W + q_len - 1 positions ending at L:
  // tiles are laid out for that union, the kernel masks per query.
  hp.window_union = prob.window > 0 ? (int)std::min<int64_t>((int64_t)prob.window + q_len - 1, INT32_MAX) : 0;
  const size_t elt = prob.out_dtype == OMNIATTN_FP32 ? 4 : 2;
  std::vector<int32_t> tiles(prob.batch);
  int64_t sum_tiles = 0;
  hp.retained_tokens = 0;
  for (int b = 0; b < prob.batch; ++b) {
    int L = seq_lens[b];
    int64_t sink_end = std::min<int64_t>(prob.sink, L);
    int64_t win_lo = std::max<int64_t>((int64_t)L - hp.window_union, 0);
    hp.retained_tokens += (win_lo <= sink_end) ? L : sink_end + (L - win_lo);
    tiles[b] = tile_layout(L, prob.sink, hp.window_union, hp.tile).count();
    sum_tiles += tiles[b];
  }
  // (segments are listed sequence-major: the head blocks of one sequence read the same tiles; as
  // neighbours they land on one XCD (see the unit mapping in the kernel) and share its L2)
  auto blocks_of = [&](int head_block) { return (hp.heads_total + head_block - 1) / head_block; };

  // The kernels that this problem can run on.  One block of 32 rows: only the narrow kernel, which does
  // the same work in fewer instructions whatever the lengths (128 sequences of 2176 kept tokens, 16
  // heads: 88 -> 62 us, fp8 94 -> 43 us).
  const bool fp8 = prob.kv_dtype == OMNIATTN_FP8_E4M3;
  const KernelCost& wide = fp8 ? kWideFp8 : kWideBf16;
  std::vector<const KernelCost*> kernels;
  if (hp.heads_total > kHeadsPerWave) {
    kernels.push_back(&wide);
    if (fp8) kernels.push_back(&kMidFp8);
  }
  kernels.push_back(fp8 ? &kNarrowFp8 : &kNarrowBf16);
  if (prob.num_splits_hint > 0) {
    // forced splits: the smallest block that takes all rows, or the largest
    int block = kernels[0]->head_block;
    for (const KernelCost* k : kernels)
      if (hp.heads_total <= k->head_block) block = k->head_block;
    hp.head_block = block;
    hp.segs.clear();
    hp.unit_seg.assign(1, 0);
    for (int b = 0; b < prob.batch; ++b)
      for (int hb = 0; hb < blocks_of(block); ++hb) {
        int pieces = std::max(1, std::min(prob.num_splits_hint, tiles[b]));
        pieces = std::max(pieces, (tiles[b] + kMaxSegTiles - 1) / kMaxSegTiles);
        for (int s = 0; s < pieces; ++s) {
          int lo = (int)((int64_t)tiles[b] * s / pieces);
          int hi = (int)((int64_t)tiles[b] * (s + 1) / pieces);
          hp.segs.push_back({b, hb, lo, hi, -1, (int32_t)hp.unit_seg.size() - 1, 0, tiles[b]});
          hp.unit_seg.push_back((int32_t)hp.segs.size());
        }
      }
  } else {
    // The kernel with the smallest estimate is taken.  Narrow: few sequences, whose pieces would be short
    // (one sequence of 2176 kept tokens, 128 heads: 69 pieces of one tile and 69 partial rows to merge, or
    // 4 x 17 pieces of four tiles: 24.1 -> 15.4 us).  64 rows, fp8: most of the rest (32 sequences of 8320
    // tokens, 128 heads: 83 -> 73 us; 128 of 2176, 64 heads: 87 -> 56).  128 rows: bf16, and fp8 with many short
    // sequences (256 of 1024 tokens: 76 against 93 us).
    const auto most_slots = [&](int head_block) {  // (+ 1: room for alignment)
      return (int)(OMNIATTN_STATIC_SCRATCH_BYTES / ((size_t)head_block * (sizeof(float) + kV * elt) + 1));
    };
    Shape best;
    KernelCost kernel{};
    for (const KernelCost* k : kernels) {
      const int n_hb = blocks_of(k->head_block);
      Shape s = choose_shape(tiles, n_hb, num_cus, *k, most_slots(k->head_block), best.us);
      if (s.us >= best.us) continue;
      // (not at the price of a plan that omniattn_decode_static would refuse)
      if (k != kernels[0] && s.slots > most_slots(k->head_block)) continue;
      best = std::move(s);
      kernel = *k;
    }
    // Units filled by tiles alone: a segment that costs as much as several tiles moves the cuts, and now and then
    // (two of 3000 random problems) that makes a few partial rows more than the built-in scratch buffer holds.
    // Then the cuts stay where one tile a segment puts them, if those fit.
    if (best.slots > most_slots(kernel.head_block)) {
      const int n_hb = blocks_of(wide.head_block), n = prob.batch * n_hb;
      int cap = std::max((int)std::min<int64_t>((sum_tiles * n_hb + n + num_cus - 1) / num_cus, INT32_MAX / 2), 2);
      for (int i = 0; i < 64 && fill_units(tiles, n_hb, cap, 1, [](int, int, int, int, int) {}) > num_cus; ++i) ++cap;
      int64_t slots = 0;
      fill_units(tiles, n_hb, cap, 1, [&](int b, int, int lo, int hi, int) { slots += hi - lo < tiles[b]; });
      if (slots <= most_slots(wide.head_block)) {
        best.size = cap;
        kernel = wide;
        kernel.seg = 1;
      }
    }
    hp.head_block = kernel.head_block;
    lay_out(best, tiles, blocks_of(hp.head_block), num_cus, kernel, hp.segs, hp.unit_seg);
  }
  hp.n_hb = blocks_of(hp.head_block);

  // partial slots for every (sequence, head block) cut into more than one segment
  hp.combine.clear();
  hp.n_slots = 0;
  hp.max_splits = 1;
  size_t i = 0;
  // segments of one item are consecutive in hp.segs by construction
  while (i < hp.segs.size()) {
    size_t j = i + 1;
    while (j < hp.segs.size() && hp.segs[j].b == hp.segs[i].b && hp.segs[j].hb == hp.segs[i].hb) ++j;
    int n = (int)(j - i);
    if (n > 1) {
      hp.combine.push_back({hp.segs[i].b, hp.segs[i].hb, hp.n_slots, n});
      for (size_t k = i; k < j; ++k) hp.segs[k].slot = hp.n_slots++;
      hp.max_splits = std::max(hp.max_splits, n);
    }
    i = j;
  }
  for (Segment& s : hp.segs) s.L = seq_lens[s.b];
  // workspace: lse of every partial row (fp32), then the partial rows in the output type
  const size_t rows = (size_t)hp.n_slots * hp.head_block;
  hp.part_rows_offset = (rows * sizeof(float) + 255) & ~(size_t)255;
  hp.workspace_bytes = rows ? ((hp.part_rows_offset + rows * kV * elt + 255) & ~(size_t)255) : 0;
  return OMNIATTN_OK;
}

}  // namespace omniattn
