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
//   head_block, groups  head rows per work unit, and work groups that share them;
//   cus         compute units that a unit takes at a time: its groups run side by side or one after the other;
//   tile_us  a KV tile in the long loop when all compute units work;
//   seg      a segment (page-table entries, query block, first tile, last PV, result rows), in tiles;
//   combine  the second launch that merges partial rows, with the gap in front of it (6 us), in tiles;
//   slots_per_tile  partial rows of how many slots are written and read back in a tile's time by
//            the whole chip (131 KB each per 128 rows, both ways, at 5 TB/s).
struct KernelCost {
  int head_block, groups, cus;
  double tile_us;
  int seg;
  double combine;
  double slots_per_tile;
};
// decode_kernel, 128 rows: 9 us a segment.
constexpr KernelCost kWideBf16 = {4 * kHeadsPerWave, 1, 1, 1.8, 5, 3.3, 36.0};
// decode_mid_kernel, 64 rows to a work group: blocks of 64, or two groups to a block of 128.  bf16: side by side, so that
// the second finds the tiles in its XCD's L2 and a sequence needs half the pieces; fp8: one behind the other, as many units
// as there are compute units.  fp8: a segment costs as much as ten tiles of the loop (Q split into two terms, 64 rows
// normalised and written), so sequences are cut only where that saves more: 93 mixed ones of 67 tiles at most go whole to
// 186 units, 94 us, where 255 units filled to 54 tiles with 416 partial rows' slots took 114; 287 of 10 tiles 130 -> 94.
// bf16 pair: the costs hold for rows in HBM (input sets in turn, 1.2 GB together) as for repeated calls, within 2 %; rows that
// another kernel has just written are another matter (see decode_mid_kernel.hip), but a decode's rows are older than that.
constexpr KernelCost kPairBf16 = {2 * kHeadBlockMid, 2, 2, 1.03, 8, 5.0, 20.0};
constexpr KernelCost kMidBf16 = {kHeadBlockMid, 1, 1, 1.5, 5, 3.5, 58.0};
constexpr KernelCost kPairFp8 = {2 * kHeadBlockMid, 2, 1, 3.6, 4, 1.8, 65.0};
constexpr KernelCost kMidFp8 = {kHeadBlockMid, 1, 1, 1.5, 10, 2.5, 40.0};
// decode_narrow_kernel, 32 rows: every tile passes through once per block.
constexpr KernelCost kNarrowBf16 = {kHeadsPerWave, 1, 1, 1.4, 4, 4.3, 112.0};
constexpr KernelCost kNarrowFp8 = {kHeadsPerWave, 1, 1, 1.5, 8, 4.0, 100.0};
// Do not leave slivers shorter than this many tiles unless the item itself is shorter.
constexpr int kMinSegTiles = 2;

// The sequences' tile counts: each sequence is n_hb items of that many.
struct Items {
  std::vector<int32_t> tiles;                        // per sequence
  std::vector<std::pair<int32_t, int32_t>> by_size;  // (tiles, sequences of that many), largest first
  int64_t sum = 0;                                   // of `tiles`
  int most = 0, least = 0;

  void count() {
    by_size.clear();
    by_size.reserve(16);
    // (windows make most sequences alike, and a batch of any lengths spans a few hundred counts)
    const int64_t span = (int64_t)most - least + 1;
    if (span <= 16 * (int64_t)tiles.size() + 256) {
      std::vector<int32_t> times(span, 0);
      for (int t : tiles) ++times[t - least];
      for (int64_t k = span - 1; k >= 0; --k)
        if (times[k]) by_size.emplace_back((int32_t)(least + k), times[k]);
    } else {
      std::vector<int32_t> sorted(tiles);
      std::sort(sorted.begin(), sorted.end(), std::greater<int32_t>());
      for (int t : sorted) {
        if (by_size.empty() || by_size.back().first != t) by_size.emplace_back(t, 0);
        ++by_size.back().second;
      }
    }
  }
  // Pieces of at most p tiles per head block, and those of sequences that are cut (an empty sequence is a piece too).
  int64_t cut_pieces(int p) const {
    int64_t k = 0;
    for (size_t i = 0; i < by_size.size() && by_size[i].first > p; ++i)
      k += (int64_t)((by_size[i].first + p - 1) / p) * by_size[i].second;
    return k;
  }
  int64_t pieces(int p) const {
    int64_t k = 0, whole = (int64_t)tiles.size();
    for (size_t i = 0; i < by_size.size() && by_size[i].first > p; ++i) {
      k += (int64_t)((by_size[i].first + p - 1) / p) * by_size[i].second;
      whole -= by_size[i].second;
    }
    return k + whole;
  }
};

// Deals the items (sequence b, head block hb) in order to units of capacity `cap` (tiles plus `seg` per
// segment), cutting an item where a unit is full.  emit(b, hb, tile_lo, tile_hi, unit) for every segment;
// stops where more than `most_units` units are needed.
struct Filled {
  int units = 0;      // units used (one more than `most_units`: they do not do)
  int longest = 0;    // tiles and segments of the longest
  int64_t slots = 0;  // segments of items that are cut
  double need = 0;    // the capacity that the work seen so far and the rest would fill evenly
};
template <typename Emit>
Filled fill_units(const Items& items, int n_hb, int cap, int seg, int most_units, Emit emit) {
  Filled f;
  int load = 0, unit = 0;
  auto close_unit = [&]() {
    if (load > 0) {
      f.longest = std::max(f.longest, load);
      ++unit;
      load = 0;
    }
  };
  const int batch = (int)items.tiles.size();
  int64_t rest = items.sum * n_hb;
  for (int b = 0; b < batch; ++b) {
    const int ntiles = items.tiles[b];
    for (int hb = 0; hb < n_hb; ++hb) {
      if (unit >= most_units) {
        f.units = unit + 1;
        f.need = (double)cap * unit / most_units + (double)(rest + ((int64_t)(batch - b) * n_hb - hb) * seg) / most_units;
        return f;
      }
      rest -= ntiles;
      if (ntiles <= cap - load - seg && ntiles <= kMaxSegTiles) {  // (as below, at once)
        emit(b, hb, 0, ntiles, unit);
        load += ntiles + seg;
        if (load >= cap) close_unit();
        continue;
      }
      if (ntiles == 0) {  // empty retained set: one segment that only writes zeros / -inf
        close_unit();
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
        f.slots += take < ntiles;
        emit(b, hb, done, done + take, unit);
        done += take;
        load += take + seg;
        if (load >= cap) close_unit();
      }
    }
  }
  f.need = ((double)cap * unit + load) / most_units;
  close_unit();
  f.units = unit;
  return f;
}
inline Filled measure_fill(const Items& items, int n_hb, int cap, int seg, int most_units) {
  return fill_units(items, n_hb, cap, seg, most_units, [](int, int, int, int, int) {});
}

// Loads of units that are dealt whole items, largest first, each to the unit with the least work so far: at
// most the average and one item.  Costs are small integers, so the units stand in lists by their load.
inline size_t most_load(const Items& items, int n_hb, int num_cus, int seg) {
  const int64_t n = (int64_t)items.tiles.size() * n_hb;
  return (size_t)((items.sum * n_hb + n * seg) / num_cus + items.most + seg + 1);
}
constexpr size_t kMostLoad = 1 << 22;  // a bound on the lists (a million items of 1024 tiles for 256 units)
// The longest of them (or any load of at least `limit` if it is none below).
int deal_whole(const Items& items, int n_hb, int num_cus, int seg, double limit) {
  std::vector<int32_t> units(most_load(items, n_hb, num_cus, seg) + 1, 0);  // how many at this load
  units[0] = num_cus;
  int longest = 0;
  size_t least = 0;
  for (const auto& s : items.by_size) {
    const int cost = s.first + seg;
    for (int64_t left = (int64_t)s.second * n_hb; left > 0;) {
      while (units[least] == 0) ++least;
      const int32_t k = (int32_t)std::min<int64_t>(left, units[least]);
      units[least] -= k;
      units[least + cost] += k;
      left -= k;
      longest = std::max(longest, (int)least + cost);
      if (longest >= limit) return longest;
    }
  }
  return longest;
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
// for every decode step.  Bounds from the tile counts rule out most of the rest before any search.  us on one
// 2.7 GHz core, 256 units, before this choice / now: 64 sequences alike 4.4 / 2.5; fp8, three kernels: 93 of
// 1024 to 65536 tokens, window 4096 7.6 / 6.2; 256 of 512 to 32768, all kept 12 / 14; 1000 of them 34 / 44.
struct Shape {
  enum { kFill, kWhole, kEven } kind = kFill;
  int size = 0;                  // kFill: capacity of a unit; kEven: tiles of a piece
  int64_t slots = 0;             // partial rows it leaves
  double us = INFINITY;
};

// No partition with this kernel takes fewer tiles' time: some unit has at least the average.
inline double least_tiles(const Items& items, int n_hb, int num_cus, const KernelCost& cost) {
  const double tiles = (double)items.sum * n_hb / num_cus, n = (double)items.tiles.size() * n_hb;
  return std::max(tiles + cost.seg, tiles + n * cost.seg / num_cus);
}

// `most_slots`: partial slots that fit the built-in scratch buffer; even pieces are not cut so short that
// omniattn_decode_static would refuse the plan.  Returns an estimate of `limit_us` or more when nothing below it
// exists.
Shape choose_shape(const Items& items, int n_hb, int num_cus, const KernelCost& cost, int most_slots, double limit_us) {
  Shape r;
  const int64_t n = (int64_t)items.tiles.size() * n_hb;
  const int64_t sum = items.sum * n_hb;
  const int n_max = items.most, seg = cost.seg;
  auto merge_cost = [&](int64_t slots) { return slots ? cost.combine + slots / cost.slots_per_tile : 0.0; };
  double best = limit_us / cost.tile_us;  // in tiles, as all below
  bool found = false;
  auto take = [&](double t) {
    if (t >= best) return false;
    best = t;
    return found = true;
  };
  if (least_tiles(items, n_hb, num_cus, cost) >= best) return r;

  // whole (a segment's tile table holds kMaxSegTiles)
  if (n_max <= kMaxSegTiles) {
    if (n <= num_cus) {
      if (take(n_max + seg)) r.kind = Shape::kWhole;
    } else if (most_load(items, n_hb, num_cus, seg) < kMostLoad) {
      // (of the j * num_cus + 1 largest items some unit has j + 1)
      int bound = n_max + seg;
      int64_t seen = 0, j = 1;
      for (const auto& s : items.by_size) {
        seen += (int64_t)s.second * n_hb;
        if (seen > j * num_cus) {
          j = (seen - 1) / num_cus;
          bound = (int)std::min<int64_t>(std::max<int64_t>(bound, (j + 1) * (s.first + seg)), INT32_MAX / 2);
          ++j;
        }
      }
      if (bound < best && take(deal_whole(items, n_hb, num_cus, seg, best))) r.kind = Shape::kWhole;
    }
  }
  // even: the smallest piece that needs no more pieces than there are units
  const int average = (int)std::min<int64_t>((sum + num_cus - 1) / num_cus, INT32_MAX / 2);
  if (n <= num_cus && n_max > 1 && average + seg < best) {
    int bad = average - 1, good = n_max;  // (shorter pieces than the average are too many; one piece per item fits)
    if (n < num_cus) good = std::min<int64_t>(good, sum / (num_cus - n) + 1);  // (fewer than sum / p + n pieces)
    while (good - bad > 1) {
      const int mid = bad + (good - bad) / 2;
      (items.pieces(mid) * n_hb > num_cus ? bad : good) = mid;
    }
    // (with few items the shortest pieces give more partial rows than they save tiles: sum / p
    // slots cost sum / p / slots_per_tile, which balances p at the square root below)
    const int balanced = (int)std::sqrt((double)sum / cost.slots_per_tile);
    for (int p : {good, std::max(good, balanced), 2 * good}) {
      p = std::min({p, n_max, kMaxSegTiles});
      if (p + seg >= best || items.pieces(p) * n_hb > num_cus) continue;
      const int64_t slots = items.cut_pieces(p) * n_hb;
      if (slots <= most_slots && take(p + seg + merge_cost(slots))) {
        r.kind = Shape::kEven;
        r.size = p;
        r.slots = slots;
      }
    }
  }
  // fill: the smallest capacity that needs no more units than there are, if one can win at all
  const int64_t least = std::max<int64_t>((sum + n * seg + num_cus - 1) / num_cus, seg + 1);
  int lo = (int)std::min<int64_t>(least, INT32_MAX / 2);
  // (a capacity c gives segments of at most c - seg tiles: at least that many of them)
  auto too_small = [&](int c) { return sum + seg * items.pieces(c - seg) * n_hb > (int64_t)num_cus * c; };
  if (lo < INT32_MAX / 4 && too_small(lo)) {
    int bad = lo, step = 1;
    while (too_small(bad + step)) {
      bad += step;
      step *= 2;
    }
    lo = bad + step;
    while (lo - bad > 1) {
      const int mid = bad + (lo - bad) / 2;
      (too_small(mid) ? bad : lo) = mid;
    }
  }
  // (a capacity that gives no more than whole items may come without a merge; then `whole` is as good)
  const double cap_max = best < INFINITY ? best - cost.combine : INFINITY;
  // Whether some capacity of [a, z) can win: a capacity gives at least the slots of a larger one.
  auto at_least = [&](int a, int z) { return a + merge_cost(items.cut_pieces(z - 1 - seg) * n_hb); };
  auto can_win = [&](auto& self, int a, int z) -> bool {
    if (a >= z || at_least(a, z) >= best) return false;
    if (z - a == 1 || at_least(a, a + 1) < best) return true;
    const int mid = a + (z - a) / 2;
    return self(self, a + 1, mid + 1) || self(self, mid + 1, z);
  };
  if (cap_max < INFINITY && !can_win(can_win, lo, (int)std::min(std::ceil(cap_max), INT32_MAX / 2.0))) {
    if (found) r.us = best * cost.tile_us;
    return r;
  }
  // Nearly every unit ends inside an item, which is a segment more than the items have: the smallest capacity that
  // does lies there, and each try says how much the units would hold evenly.  One or two tries.
  int bad = lo - 1, cap = 0, step = 1;
  Filled f;
  for (int c = std::max(lo, (int)std::min<int64_t>(least + seg - 1, INT32_MAX / 2)); c < cap_max && step < (1 << 28);) {
    const Filled g = measure_fill(items, n_hb, c, seg, num_cus);
    const int even = (int)std::min(std::ceil(g.need), INT32_MAX / 2.0);
    if (g.units <= num_cus) {
      cap = c;
      f = g;
      if (cap - bad <= 1 || even >= cap) break;
      c = std::max(even, bad + 1);
    } else {
      bad = c;
      if (cap - bad == 1) break;
      c = std::max(even, bad + step);
      if (cap) c = std::min(c, cap - 1);
      step *= 2;
    }
  }
  if (!cap && best == INFINITY) {  // (more units than compute units, then)
    cap = bad;
    f = measure_fill(items, n_hb, cap, seg, INT_MAX);
  }
  if (cap) {
    if (take(f.longest + merge_cost(f.slots))) {
      r.kind = Shape::kFill;
      r.size = cap;
      r.slots = f.slots;
    }
  }
  if (found) r.us = best * cost.tile_us;
  return r;
}

// Appends segments to a plan, units in ascending order, the pieces of an item one behind the other; an item
// that is cut gets its partial slots and its entry for the merge on the way.
struct Writer {
  HostPlan& hp;
  const std::vector<int32_t>& tiles;
  int last_unit = -1;

  Writer(HostPlan& plan, const std::vector<int32_t>& t, size_t segments, size_t units, size_t cut) : hp(plan), tiles(t) {
    hp.segs.clear();
    hp.segs.reserve(segments);
    hp.unit_seg.clear();
    hp.unit_seg.reserve(units + 1);
    hp.combine.clear();
    hp.combine.reserve(cut);
    hp.n_slots = 0;
    hp.max_splits = 1;
  }
  void operator()(int b, int hb, int lo, int hi, int unit) {
    if (unit != last_unit) hp.unit_seg.push_back((int32_t)hp.segs.size());
    last_unit = unit;
    int slot = -1;
    if (hi - lo < tiles[b]) {
      slot = hp.n_slots++;
      if (lo == 0) hp.combine.push_back({b, hb, slot, 0});
      hp.max_splits = std::max(hp.max_splits, ++hp.combine.back().nslots);
    }
    hp.segs.push_back({b, hb, lo, hi, slot, unit, hp.seq_lens[b], tiles[b]});
  }
  void finish() { hp.unit_seg.push_back((int32_t)hp.segs.size()); }
};

void lay_out(const Shape& shape, const Items& items, int n_hb, int num_cus, const KernelCost& cost, HostPlan& hp) {
  const std::vector<int32_t>& tiles = items.tiles;
  Writer add(hp, tiles, tiles.size() * n_hb + (size_t)shape.slots, num_cus, (size_t)shape.slots / 2);
  const int batch = (int)tiles.size(), n = batch * n_hb;
  if (shape.kind == Shape::kFill) {
    fill_units(items, n_hb, shape.size, cost.seg, INT_MAX, [&](int b, int hb, int lo, int hi, int u) { add(b, hb, lo, hi, u); });
  } else if (shape.kind == Shape::kEven) {
    int unit = 0;
    for (int b = 0; b < batch; ++b) {
      const int t = tiles[b], k = std::max(1, (t + shape.size - 1) / shape.size);
      for (int hb = 0; hb < n_hb; ++hb)
        for (int s = 0; s < k; ++s) add(b, hb, (int)((int64_t)t * s / k), (int)((int64_t)t * (s + 1) / k), unit++);
    }
  } else if (n <= num_cus) {
    for (int i = 0; i < n; ++i) add(i / n_hb, i % n_hb, 0, tiles[i / n_hb], i);
  } else {
    // sequences by size, as deal_whole takes them
    std::vector<int32_t> at_size(items.most + 2, 0), order(batch);
    for (int t : tiles) ++at_size[items.most - t + 1];
    for (int k = 0; k <= items.most; ++k) at_size[k + 1] += at_size[k];
    for (int b = 0; b < batch; ++b) order[at_size[items.most - tiles[b]]++] = b;
    // units in lists by their load, first in, first out
    struct List { int32_t head, tail; };
    std::vector<List> at_load(most_load(items, n_hb, num_cus, cost.seg) + 1, List{-1, -1});
    std::vector<int32_t> behind(num_cus, -1), first(num_cus + 1, 0), unit_of(n), item_at(n);
    auto append = [&](int unit, size_t load) {
      List& l = at_load[load];
      behind[unit] = -1;
      (l.head < 0 ? l.head : behind[l.tail]) = unit;
      l.tail = unit;
    };
    for (int u = 0; u < num_cus; ++u) append(u, 0);
    size_t least = 0;
    for (int b : order)
      for (int hb = 0; hb < n_hb; ++hb) {
        while (at_load[least].head < 0) ++least;
        const int unit = at_load[least].head;
        at_load[least].head = behind[unit];
        append(unit, least + tiles[b] + cost.seg);
        unit_of[b * n_hb + hb] = unit;
        ++first[unit + 1];
      }
    // units in order, each with its items
    for (int u = 0; u < num_cus; ++u) first[u + 1] += first[u];
    std::vector<int32_t> next(first.begin(), first.end() - 1);
    for (int i = 0; i < n; ++i) item_at[next[unit_of[i]]++] = i;
    for (int u = 0; u < num_cus; ++u)
      for (int k = first[u]; k < first[u + 1]; ++k) {
        const int b = item_at[k] / n_hb;
        add(b, item_at[k] - b * n_hb, 0, tiles[b], u);
      }
  }
  add.finish();
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
  const bool fp8 = prob.kv_dtype == OMNIATTN_FP8_E4M3;
  hp.tile = fp8 ? kTileFp8 : kTile;
  hp.heads_total = prob.num_heads * q_len;
  // Several causal queries: query t keeps [0, S) and the W positions ending at its own token.
  // Over all queries that is [0, S) and (for W > 0) the W + q_len - 1 positions ending at L:
  // tiles are laid out for that union, the kernel masks per query.
  hp.window_union = prob.window > 0 ? (int)std::min<int64_t>((int64_t)prob.window + q_len - 1, INT32_MAX) : 0;
  const size_t elt = prob.out_dtype == OMNIATTN_FP32 ? 4 : 2;
  Items items;
  std::vector<int32_t>& tiles = items.tiles;
  tiles.resize(prob.batch);
  items.least = INT_MAX;
  hp.retained_tokens = 0;
  for (int b = 0; b < prob.batch; ++b) {
    int L = seq_lens[b];
    int64_t sink_end = std::min<int64_t>(prob.sink, L);
    int64_t win_lo = std::max<int64_t>((int64_t)L - hp.window_union, 0);
    hp.retained_tokens += (win_lo <= sink_end) ? L : sink_end + (L - win_lo);
    // (divisions by constants)
    tiles[b] = (fp8 ? tile_layout(L, prob.sink, hp.window_union, kTileFp8) : tile_layout(L, prob.sink, hp.window_union, kTile)).count();
    items.sum += tiles[b];
    items.most = std::max(items.most, tiles[b]);
    items.least = std::min(items.least, tiles[b]);
  }
  // (segments are listed sequence-major: the head blocks of one sequence read the same tiles; as
  // neighbours they land on one XCD (see the unit mapping in the kernel) and share its L2)
  auto blocks_of = [&](int head_block) { return (hp.heads_total + head_block - 1) / head_block; };

  // The kernels that this problem can run on.  One block of 32 rows: only the narrow kernel, which does
  // the same work in fewer instructions whatever the lengths (128 sequences of 2176 kept tokens, 16
  // heads: 88 -> 62 us, fp8 94 -> 43 us).
  const KernelCost& wide = fp8 ? kPairFp8 : kWideBf16;
  std::vector<const KernelCost*> kernels;
  if (hp.heads_total > kHeadsPerWave) {
    kernels.push_back(&wide);
    // bf16, two groups of 64 rows side by side: up to 256 rows, of which the last block's second half has more than 16.
    // us with decode_kernel / with the pair, on rows that no cache holds.  Inside: 128 rows, 64 sequences of 2176 kept tokens
    // 58.7 / 52.3, 32 of 4096 56.6 / 50.6, 128 of 2176 93 / 84; 256 rows, 64 of 2176 87 / 79.  Outside the pair is not offered,
    // though most of these would gain too: 72 rows, 64 of 600 34 / 26, 64 of 2176 51 / 50; 192 rows, 64 of 600 41 / 27, 64 of 2176
    // 90 / 69, 40 of 2176 64 / 63; 208 rows, 128 of 2176 149 / 167; 384 rows, 40 of 2176 84 / 77, 64 of 2176 143 / 141, 64 of 600
    // 45 / 56; 512 rows, 64 of 2176 140 / 158, 64 of 600 52 / 58 (six or eight groups pull every tile through one L2).
    const int last_rows = (hp.heads_total - 1) % kPairBf16.head_block + 1;
    if (fp8) kernels.push_back(&kMidFp8);
    else if (hp.heads_total <= kHeadBlockMid) kernels.push_back(&kMidBf16);
    else if (num_cus >= kPairBf16.cus && hp.heads_total <= 2 * kPairBf16.head_block && last_rows > kHeadBlockMid + 16)
      kernels.push_back(&kPairBf16);
  }
  kernels.push_back(fp8 ? &kNarrowFp8 : &kNarrowBf16);
  if (prob.num_splits_hint > 0) {
    // forced splits: the smallest block that takes all rows, or the largest (bf16: 32 rows, or decode_kernel's 128)
    const KernelCost* kernel = kernels[0];
    for (const KernelCost* k : kernels)
      if (hp.heads_total <= k->head_block && k != &kMidBf16 && k != &kPairBf16) kernel = k;
    const int block = hp.head_block = kernel->head_block;
    hp.groups = kernel->groups;
    const int n_hb = blocks_of(block);
    Writer add(hp, tiles, tiles.size() * n_hb, tiles.size() * n_hb, 0);
    int unit = 0;
    for (int b = 0; b < prob.batch; ++b)
      for (int hb = 0; hb < n_hb; ++hb) {
        int pieces = std::max(1, std::min(prob.num_splits_hint, tiles[b]));
        pieces = std::max(pieces, (tiles[b] + kMaxSegTiles - 1) / kMaxSegTiles);
        for (int s = 0; s < pieces; ++s)
          add(b, hb, (int)((int64_t)tiles[b] * s / pieces), (int)((int64_t)tiles[b] * (s + 1) / pieces), unit++);
      }
    add.finish();
  } else {
    // The kernel with the smallest estimate is taken.  Narrow: few sequences, whose pieces would be short
    // (one sequence of 2176 kept tokens, 128 heads: 69 pieces of one tile and 69 partial rows to merge, or
    // 4 x 35 pieces of two tiles: 24.1 -> 15.4 us).  64 rows to a group: fp8 (32 sequences of 8320 tokens, 128 heads:
    // 83 -> 67 us), bf16 where decode_kernel would cut sequences into four and more
    // pieces, or has half a block of rows (64 of 2176, 128 heads 58 -> 53.5; 81 of 650 50 -> 33; 128 of 2176, 64 heads
    // 88 -> 66).  decode_kernel: long bf16 sequences that fill the units, half the loads (256 of 4256 tokens: 300 against
    // 318 us).
    const auto most_slots = [&](int head_block) {  // (+ 1: room for alignment)
      return (int)(OMNIATTN_STATIC_SCRATCH_BYTES / ((size_t)head_block * (sizeof(float) + kV * elt) + 1));
    };
    items.count();
    // (the one that may be cheapest first: its estimate often rules out the others)
    auto least_us = [&](const KernelCost* k) { return least_tiles(items, blocks_of(k->head_block), num_cus / k->cus, *k) * k->tile_us; };
    const KernelCost* order[3];
    const int n_kernels = (int)kernels.size();
    std::copy(kernels.begin(), kernels.end(), order);
    std::stable_sort(order, order + n_kernels, [&](const KernelCost* a, const KernelCost* b) { return least_us(a) < least_us(b); });
    Shape best;
    KernelCost kernel{};
    for (int i = 0; i < n_kernels; ++i) {
      const KernelCost& k = *order[i];
      Shape s = choose_shape(items, blocks_of(k.head_block), num_cus / k.cus, k, most_slots(k.head_block), best.us);
      if (s.us >= best.us) continue;
      // (not at the price of a plan that omniattn_decode_static would refuse)
      if (&k != kernels[0] && s.slots > most_slots(k.head_block)) continue;
      best = s;
      kernel = k;
    }
    // Units filled by tiles alone: a segment that costs as much as several tiles moves the cuts, and now and then
    // (two of 3000 random problems) that makes a few partial rows more than the built-in scratch buffer holds.
    // Then the cuts stay where one tile a segment puts them, if those fit.
    if (best.slots > most_slots(kernel.head_block)) {
      const int n_hb = blocks_of(wide.head_block), n = prob.batch * n_hb;
      int cap = std::max((int)std::min<int64_t>((items.sum * n_hb + n + num_cus - 1) / num_cus, INT32_MAX / 2), 2);
      Filled f = measure_fill(items, n_hb, cap, 1, num_cus);
      for (int i = 0; i < 64 && f.units > num_cus; ++i) f = measure_fill(items, n_hb, ++cap, 1, num_cus);
      if (f.units <= num_cus && f.slots <= most_slots(wide.head_block)) {
        best.size = cap;
        kernel = wide;
        kernel.seg = 1;
      }
    }
    // Else, fp8 with fp32 results (partial rows twice as large): blocks of 64 rows, if there are no more of them than units,
    // with cuts as for the largest segment cost that leaves few enough partial rows, and if by the estimate at that cost, which
    // understates it (a segment costs ten tiles whatever the cuts assume), they take no longer: a plan that fits is worth that.
    // (Of 780,000 random problems 3,310 come here; at ten tiles 11 are estimated to take up to 10 % longer, and three of those that
    // were timed took 104.8 -> 102.9, 94 -> 77 and 107 -> 98 us.)
    // us with 59 to 76 MB of partial rows -> with 42: 49 sequences of 6800 tokens at most 115 -> 99, 9 of 2845 with 640 rows
    // 66 -> 55, 66 of 8400 at most 105 -> 92.  (More blocks than units, 642 sequences of 9 tiles with 256 rows: 352 -> 383.)
    if (fp8 && elt == 4 && kernels.size() == 3 && kernel.seg == kernels[0]->seg && best.slots > most_slots(kernel.head_block) &&
        (int64_t)prob.batch * blocks_of(kMidFp8.head_block) <= num_cus) {
      for (KernelCost k = kMidFp8; k.seg > 0; --k.seg) {
        const Shape s = choose_shape(items, blocks_of(k.head_block), num_cus, k, most_slots(k.head_block), best.us);
        if (s.us >= best.us || s.slots > most_slots(k.head_block)) continue;
        best = s;
        kernel = k;
        break;
      }
    }
    hp.head_block = kernel.head_block;
    hp.groups = kernel.groups;
    lay_out(best, items, blocks_of(hp.head_block), num_cus / kernel.cus, kernel, hp);
  }
  hp.n_hb = blocks_of(hp.head_block);

  // workspace: lse of every partial row (fp32), then the partial rows in the output type
  const size_t rows = (size_t)hp.n_slots * hp.head_block;
  hp.part_rows_offset = (rows * sizeof(float) + 255) & ~(size_t)255;
  hp.workspace_bytes = rows ? ((hp.part_rows_offset + rows * kV * elt + 255) & ~(size_t)255) : 0;
  return OMNIATTN_OK;
}

}  // namespace omniattn
