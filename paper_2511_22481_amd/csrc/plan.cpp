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

struct Item {
  int b, hb, ntiles;
};

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
// The kernels for full head blocks: 9 us and 13 us a segment.
constexpr KernelCost kWideBf16 = {4 * kHeadsPerWave, 1.8, 5, 3.3, 36.0};
constexpr KernelCost kWideFp8 = {4 * kHeadsPerWave, 3.4, 4, 1.8, 65.0};
// The kernel for blocks of 32 rows: every tile passes through once per block, but its tile and its start
// cost less.
constexpr KernelCost kNarrowBf16 = {kHeadsPerWave, 1.4, 4, 4.3, 112.0};
constexpr KernelCost kNarrowFp8 = {kHeadsPerWave, 1.5, 4, 4.0, 120.0};
// Do not leave slivers shorter than this many tiles unless the item itself is shorter.
constexpr int kMinSegTiles = 2;

// Deals the items in order to units of capacity `cap` (tiles plus `seg` per segment), cutting an
// item where a unit is full.  emit(item, tile_lo, tile_hi, unit) for every segment; returns the
// number of units used.
template <typename Emit>
int fill_units(const std::vector<Item>& items, int cap, int seg, Emit emit) {
  int load = 0, unit = 0;
  auto close_unit = [&]() {
    if (load > 0) {
      ++unit;
      load = 0;
    }
  };
  for (const Item& it : items) {
    if (it.ntiles == 0) {  // empty retained set: one segment that only writes zeros / -inf
      if (load + seg > cap) close_unit();
      emit(it, 0, 0, unit);
      load += seg;
      continue;
    }
    int done = 0;
    while (done < it.ntiles) {
      const int rem = it.ntiles - done;
      int room = cap - load - seg;
      const int need = std::min(rem, kMinSegTiles);
      if (room < need) {
        if (load == 0) room = need;  // capacity smaller than one minimal segment
        else { close_unit(); continue; }
      }
      int take = std::min(std::min(rem, room), kMaxSegTiles);
      // avoid leaving a sliver behind
      if (rem - take > 0 && rem - take < kMinSegTiles) take = std::max(1, rem - kMinSegTiles);
      emit(it, done, done + take, unit);
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
// `most_slots`: partial slots that fit the built-in scratch buffer.  Even pieces are not cut so
// short that omniattn_decode_static would refuse the plan.  Returns the estimate in us.
double partition(const std::vector<Item>& items, int num_cus, const KernelCost& cost, int most_slots,
                 std::vector<Segment>& segs, std::vector<int32_t>& unit_seg) {
  const int n = (int)items.size();
  int64_t total = 0;
  int n_max = 0;
  for (const Item& it : items) {
    total += it.ntiles + cost.seg;
    n_max = std::max(n_max, it.ntiles);
  }
  auto merge_cost = [&](int slots) { return slots ? cost.combine + slots / cost.slots_per_tile : 0.0; };

  // fill: the smallest capacity that needs no more units than there are
  int lo = std::max((int)std::min<int64_t>((total + num_cus - 1) / num_cus, INT32_MAX / 2), cost.seg + 1), fill_cap = lo;
  auto units_at = [&](int cap) { return fill_units(items, cap, cost.seg, [](const Item&, int, int, int) {}); };
  if (units_at(lo) > num_cus) {
    int step = 1;
    while (units_at(lo + step) > num_cus && step < (1 << 28)) step *= 2;
    int bad = lo + step / 2, good = lo + step;
    while (good - bad > 1) {
      const int mid = bad + (good - bad) / 2;
      (units_at(mid) > num_cus ? bad : good) = mid;
    }
    fill_cap = good;
  }
  double best;
  {
    int slots = 0, longest = 0, load = 0, last_unit = -1;
    fill_units(items, fill_cap, cost.seg, [&](const Item& it, int a, int b, int unit) {
      if (b - a < it.ntiles) ++slots;
      load = (unit == last_unit ? load : 0) + b - a + cost.seg;
      last_unit = unit;
      longest = std::max(longest, load);
    });
    best = longest + merge_cost(slots);
  }
  enum { kFill, kWhole, kEven } shape = kFill;

  // whole (a segment's tile table holds kMaxSegTiles)
  std::vector<int32_t> unit_of;
  if (n_max <= kMaxSegTiles && n_max + cost.seg < best) {
    std::vector<int32_t> order(n);
    for (int i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return items[a].ntiles > items[b].ntiles; });
    unit_of.resize(n);
    std::vector<std::pair<int32_t, int32_t>> heap;  // (load, unit), least loaded on top
    const auto later = std::greater<std::pair<int32_t, int32_t>>();
    int longest = 0;
    for (int i = 0; i < n && longest < best; ++i) {
      const int cost_i = items[order[i]].ntiles + cost.seg;
      int unit = i, load = cost_i;
      if (i < num_cus) {
        heap.emplace_back(load, unit);
        if (i == num_cus - 1 || i == n - 1) std::make_heap(heap.begin(), heap.end(), later);
      } else {
        std::pop_heap(heap.begin(), heap.end(), later);
        unit = heap.back().second;
        load = heap.back().first += cost_i;
        std::push_heap(heap.begin(), heap.end(), later);
      }
      unit_of[order[i]] = unit;
      longest = std::max(longest, load);
    }
    if (longest < best) {
      best = longest;
      shape = kWhole;
    }
  }
  // even: the smallest piece that needs no more pieces than there are units
  int piece = 0;
  if (n <= num_cus && n_max > 1) {
    auto pieces_at = [&](int p) {
      int64_t k = 0;
      for (const Item& it : items) k += std::max(1, (it.ntiles + p - 1) / p);
      return k;
    };
    int bad = 0, good = n_max;  // (one piece per item fits)
    while (good - bad > 1) {
      const int mid = bad + (good - bad) / 2;
      (pieces_at(mid) > num_cus ? bad : good) = mid;
    }
    // (with few items the shortest pieces give more partial rows than they save tiles: sum / p
    // slots cost sum / p / slots_per_tile, which balances p at the square root below)
    const int balanced = (int)std::sqrt((double)(total - (int64_t)n * cost.seg) / cost.slots_per_tile);
    for (int p : {good, std::max(good, balanced), 2 * good}) {
      p = std::min({p, n_max, kMaxSegTiles});
      if (pieces_at(p) > num_cus) continue;
      int slots = 0;
      for (const Item& it : items)
        if (it.ntiles > p) slots += (it.ntiles + p - 1) / p;
      if (slots > most_slots) continue;
      const double t = p + cost.seg + merge_cost(slots);
      if (t < best) {
        best = t;
        shape = kEven;
        piece = p;
      }
    }
  }

  segs.clear();
  unit_seg.assign(1, 0);
  auto add = [&](const Item& it, int a, int b, int unit) {
    while ((int)unit_seg.size() <= unit) unit_seg.push_back((int32_t)segs.size());
    segs.push_back({it.b, it.hb, a, b, -1, unit, 0, it.ntiles});
  };
  if (shape == kFill) {
    fill_units(items, fill_cap, cost.seg, add);
  } else if (shape == kEven) {
    int unit = 0;
    for (const Item& it : items) {
      const int k = std::max(1, (it.ntiles + piece - 1) / piece);
      for (int s = 0; s < k; ++s)
        add(it, (int)((int64_t)it.ntiles * s / k), (int)((int64_t)it.ntiles * (s + 1) / k), unit++);
    }
  } else {
    // units in order, each with its items
    const int n_units = std::min(n, num_cus);
    std::vector<int32_t> first(n_units + 1, 0), at(n);
    for (int i = 0; i < n; ++i) ++first[unit_of[i] + 1];
    for (int u = 0; u < n_units; ++u) first[u + 1] += first[u];
    std::vector<int32_t> next(first.begin(), first.end() - 1);
    for (int i = 0; i < n; ++i) at[next[unit_of[i]]++] = i;
    for (int u = 0; u < n_units; ++u)
      for (int k = first[u]; k < first[u + 1]; ++k) add(items[at[k]], 0, items[at[k]].ntiles, u);
  }
  unit_seg.push_back((int32_t)segs.size());
  return best * cost.tile_us;
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
  // sequence-major: the head blocks of one sequence read the same tiles; as neighbours they
  // land on one XCD (see the unit mapping in the kernel) and share its L2
  std::vector<Item> items;
  auto deal_heads = [&](int head_block) {
    const int n_hb = (hp.heads_total + head_block - 1) / head_block;
    items.clear();
    items.reserve((size_t)prob.batch * n_hb);
    for (int b = 0; b < prob.batch; ++b)
      for (int hb = 0; hb < n_hb; ++hb) items.push_back({b, hb, tiles[b]});
    hp.head_block = head_block;
    hp.n_hb = n_hb;
  };

  const bool fp8 = prob.kv_dtype == OMNIATTN_FP8_E4M3;
  const KernelCost& wide = fp8 ? kWideFp8 : kWideBf16;
  const KernelCost& narrow = fp8 ? kNarrowFp8 : kNarrowBf16;
  // One block of 32 rows: the narrow kernel does the same work in fewer instructions, whatever the
  // lengths (128 sequences of 2176 kept tokens, 16 heads: 88 -> 63 us, fp8 94 -> 43 us).
  const bool one_block = hp.heads_total <= kHeadsPerWave;
  if (prob.num_splits_hint > 0) {
    deal_heads(one_block ? narrow.head_block : wide.head_block);
    hp.segs.clear();
    hp.unit_seg.assign(1, 0);
    for (const Item& it : items) {
      int pieces = std::max(1, std::min(prob.num_splits_hint, it.ntiles));
      pieces = std::max(pieces, (it.ntiles + kMaxSegTiles - 1) / kMaxSegTiles);
      for (int s = 0; s < pieces; ++s) {
        int lo = (int)((int64_t)it.ntiles * s / pieces);
        int hi = (int)((int64_t)it.ntiles * (s + 1) / pieces);
        hp.segs.push_back({it.b, it.hb, lo, hi, -1, (int32_t)hp.unit_seg.size() - 1, 0, it.ntiles});
        hp.unit_seg.push_back((int32_t)hp.segs.size());
      }
    }
  } else {
    auto try_kernel = [&](const KernelCost& k, std::vector<Segment>& segs, std::vector<int32_t>& unit_seg) {
      deal_heads(k.head_block);
      const size_t slot_bytes = (size_t)k.head_block * (sizeof(float) + kV * elt) + 1;  // (+ 1: room for alignment)
      return partition(items, num_cus, k, (int)(OMNIATTN_STATIC_SCRATCH_BYTES / slot_bytes), segs, unit_seg);
    };
    // With more rows the kernel with the smaller estimate is taken: the narrow one where the sequences
    // are too few to fill the chip with long pieces (one sequence of 2176 kept tokens, 128 heads: 69
    // pieces of one tile and 69 partial rows to merge, or 4 x 17 of four tiles: 24.1 -> 15.6 us), the
    // other where tiles are many.
    double best = one_block ? INFINITY : try_kernel(wide, hp.segs, hp.unit_seg);
    const int n_narrow = (hp.heads_total + kHeadsPerWave - 1) / kHeadsPerWave;
    if ((double)(sum_tiles * n_narrow) / num_cus * narrow.tile_us < best) {
      std::vector<Segment> segs;
      std::vector<int32_t> unit_seg;
      const int blocks = hp.head_block;
      if (try_kernel(narrow, segs, unit_seg) < best) {
        hp.segs.swap(segs);
        hp.unit_seg.swap(unit_seg);
      } else {
        deal_heads(blocks);
      }
    }
  }

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
