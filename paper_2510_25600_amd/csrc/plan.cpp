// Host planner: turns (F, P, T, pattern) into per-query-tile key-tile lists with per-block masks, cuts long
// lists into slices, and deals (slice, head group) units onto persistent workgroups.
// The mask follows the two ST-SpAttn paragraphs of Sec. 3.2 (spatial: first frame + own frame;
// temporal: first frame + same patch one frame back), always causal, text queries dense.
#include "plan.h"

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <functional>
#include <limits>
#include <queue>
#include <utility>
#include <vector>

namespace purekv {

namespace {

// Allowed keys of query row i: j <= i with (j <= a  or  j >= lo  or  j == prev  or  j == self).
struct RowSet {
  int32_t a, lo, prev, self;
};

inline RowSet row_set(const Geometry& g, int32_t i) {
  if (g.pattern == PUREKV_PATTERN_DENSE || i >= g.Nv) return {i, 0, -1, -1};
  const int32_t f = i / g.P;
  RowSet r;
  r.a = std::min(i, g.P - 1);
  r.lo = (g.pattern & PUREKV_PATTERN_SPATIAL) ? f * g.P : i + 1;
  r.prev = ((g.pattern & PUREKV_PATTERN_TEMPORAL) && f >= 1) ? i - g.P : -1;
  r.self = (g.pattern & PUREKV_PATTERN_TEMPORAL) ? i : -1;
  return r;
}

inline bool in_range(int32_t x, int32_t k0, int32_t k1) { return x >= k0 && x <= k1; }

// Some key of [k0, k1] is allowed.
inline bool row_hits(const RowSet& s, int32_t i, int32_t k0, int32_t k1) {
  return (k0 <= s.a) || (std::max(k0, s.lo) <= std::min(k1, i)) || in_range(s.prev, k0, k1) ||
         in_range(s.self, k0, k1);
}

// Every key of [k0, k1] is allowed; an empty range counts as allowed.  Single keys of the temporal path
// are ignored here, so the answer can be a conservative "no".
inline bool row_full(const RowSet& s, int32_t i, int32_t k0, int32_t k1) {
  if (k0 > k1) return true;
  if (s.lo <= s.a + 1) return k1 <= i;
  return (k1 <= s.a) || (k0 >= s.lo && k1 <= i);
}

// The only key of [k0, k1] that can be allowed is the previous-frame key.
inline bool row_prev_only(const RowSet& s, int32_t i, int32_t k0, int32_t k1) {
  return k0 > s.a && !(std::max(k0, s.lo) <= std::min(k1, i)) && !in_range(s.self, k0, k1);
}

inline double row_pairs(const RowSet& s, int32_t i) {
  double cnt = (s.lo <= s.a + 1) ? double(i) + 1.0 : double(s.a) + 1.0 + std::max(0, i - s.lo + 1);
  if (s.prev > s.a && s.prev < s.lo) cnt += 1.0;
  if (s.self > s.a && s.self < s.lo) cnt += 1.0;
  return cnt;
}

// Largest divisor of g that is at most `cap`.
inline int32_t largest_divisor_up_to(int32_t g, int32_t cap) {
  for (int32_t x = std::min(g, cap); x >= 1; --x)
    if (g % x == 0) return x;
  return 1;
}

// Lists, schedule and steps of a plan whose workgroup shape (Gs, R, n_groups) is given; returns the model's prediction of when
// its last workgroup ends, in steps of a plain tile.
double build_shape(purekv_plan& p, int n_cu) {
  Geometry& g = p.g;
  const int32_t BK = PUREKV_BK;
  auto group_selected = [&](int32_t grp) { return p.head_sel.empty() || p.head_sel[grp * g.Gs] != 0; };
  const int32_t n_groups_sel = p.n_heads_sel / g.Gs;
  const int32_t rows_per_qtile = g.R * kBlockRows;
  p.n_qtiles = (g.N + rows_per_qtile - 1) / rows_per_qtile;
  const int32_t n_ktiles = (g.N + BK - 1) / BK;
  p.qtile_begin.assign(1, 0);
  p.tiles.clear();
  p.n_blocks = 0;
  for (auto& c : p.n_kind) c = 0;
  p.mask_pairs = 0;

  std::vector<RowSet> sets(rows_per_qtile);
  for (int32_t qt = 0; qt < p.n_qtiles; ++qt) {
    const int32_t r0 = qt * rows_per_qtile, r1 = std::min(r0 + rows_per_qtile, g.N);  // rows [r0, r1)
    for (int32_t i = r0; i < r1; ++i) {
      sets[i - r0] = row_set(g, i);
      p.mask_pairs += row_pairs(sets[i - r0], i);
    }
    const int32_t last_tile = std::min((r1 - 1) / BK, n_ktiles - 1);  // causal: no key beyond the last row
    // Two shortcuts keep the planner linear in the number of listed tiles for long sequences; both only skip
    // work whose outcome is known.  (1) Rows that see every earlier key (dense pattern, text rows): a key tile that
    // ends at or before the first row of the query tile is needed in full by every row block.  (2) Video rows of a
    // sparse pattern can only see the first frame, their own frame up to themselves and their previous-frame keys:
    // tiles outside those three ranges are not examined.
    const bool all_dense_rows = g.pattern == PUREKV_PATTERN_DENSE || r0 >= g.Nv;
    const bool all_video_rows = g.pattern != PUREKV_PATTERN_DENSE && r1 <= g.Nv;
    uint32_t need_all = 0;
    int32_t blocks_all = 0;
    for (int32_t rb = 0; rb < g.R; ++rb)
      if (r0 + rb * kBlockRows < r1) need_all |= 3u << (2 * rb), blocks_all += 2;
    int32_t own_tile = 0, prev_lo = 1, prev_hi = 0;   // first tile of the own-frame range; previous-frame tiles
    if (all_video_rows) {
      const int32_t own0 = (g.pattern & PUREKV_PATTERN_SPATIAL) ? (r0 / g.P) * g.P : r0;
      own_tile = own0 / BK;
      if ((g.pattern & PUREKV_PATTERN_TEMPORAL) && r1 - 1 - g.P >= 0) {
        prev_lo = std::max(0, r0 - g.P) / BK;
        prev_hi = (r1 - 1 - g.P) / BK;
      }
    }
    const int32_t first_frame_tile = (g.P - 1) / BK;
    for (int32_t c = 0; c <= last_tile; ++c) {
      if (all_dense_rows && (c + 1) * BK - 1 <= r0) {
        p.tiles.push_back({c, need_all | kStepPlain, 0u});   // kind "full" is 0 in every field
        p.n_blocks += blocks_all;
        p.n_kind[kKindFull] += blocks_all;
        continue;
      }
      if (all_video_rows && c > first_frame_tile && c < own_tile && !(c >= prev_lo && c <= prev_hi)) {
        c = std::min(own_tile, prev_lo > c && prev_lo <= prev_hi ? prev_lo : own_tile) - 1;   // jump to the next range
        continue;
      }
      uint32_t need = 0, kinds = 0;
      for (int32_t rb = 0; rb < g.R; ++rb) {
        const int32_t w0 = r0 + rb * kBlockRows, w1 = std::min(w0 + kBlockRows, r1);
        if (w0 >= w1) continue;  // a row block without real rows is never needed
        for (int32_t kb = 0; kb < 2; ++kb) {
          const int32_t k0 = c * BK + kb * kBlockKeys, k1 = k0 + kBlockKeys - 1;
          bool any = false, full = true, causal = true, prev = true;
          for (int32_t i = w0; i < w1; ++i) {
            const RowSet& s = sets[i - r0];
            any |= row_hits(s, i, k0, k1);
            full &= row_full(s, i, k0, k1);
            causal &= row_full(s, i, k0, std::min(k1, i));
            prev &= row_prev_only(s, i, k0, k1);
          }
          if (!any) continue;
          const uint32_t kind = full ? kKindFull : causal ? kKindCausal : prev ? kKindPrev : kKindGeneral;
          need |= 1u << (2 * rb + kb);
          kinds |= kind << (4 * rb + 2 * kb);
          ++p.n_blocks;
          ++p.n_kind[kind];
        }
      }
      if (need) p.tiles.push_back({c, need | (need == need_all && kinds == 0u ? kStepPlain : 0u), kinds});
    }
    p.qtile_begin.push_back(static_cast<int32_t>(p.tiles.size()));
  }

  // ---- cost model, in steps of one plain tile ----
  // Fitted to the cycles of the workgroups of 60 shapes of both patterns and head widths, with 1 to 8 stacked heads, against
  // what they ran.  A half skipped saves MFMAs but no time; a step with the full predicate takes 0.2 to 0.5 more.  A unit (rows
  // written, state reset, query rows fetched) takes 1.2, with several heads stacked 1.4 under the dense pattern and more
  // where masked steps lie around the switch.  A slice takes 3.5 to 6 more (tiles that nobody else reads meanwhile, fp32 rows
  // through to memory, acknowledged, the look whether its list is complete), and the workgroup that runs a list's closing
  // slice, last in its queue, combines the list: 5 more for three slices of 256 rows x 128.  Workgroups that run slices get
  // that much less besides: with 2.5 for a slice and 1.4 for every stacked unit, the sparse plan of 8 frames of 24 x 24 + 128
  // tokens, 32/8 heads, ended with closing workgroups of 153 thousand cycles (mean 131).  With these figures its prefill takes
  // 0.98 of that, 13 frames of 17 x 19 + 45, 28/4 heads, 0.87; 300 drawn shapes 0.978 in the mean, at most 1.07.
  constexpr double kGeneralCost = 1.3, kSliceCost = 5.0;
  const bool dense = g.pattern == PUREKV_PATTERN_DENSE;
  const double kUnitCost = g.Gs == 1 ? 1.2 : dense ? 1.4 : g.d == 128 ? 1.7 : 2.1;
  auto combine_cost = [&](int32_t n_slices) { return 2.5 + 0.7 * n_slices; };
  std::vector<double> cost_before(p.tiles.size() + 1, 0.0);   // of the tiles before, in list order
  for (size_t i = 0; i < p.tiles.size(); ++i) {
    const TileRef& t = p.tiles[i];
    const bool general = (t.kinds & (t.kinds >> 1) & 0x55555555u) != 0u;
    cost_before[i + 1] = cost_before[i] + (general ? kGeneralCost : 1.0);
  }
  const double total_steps = double(p.tiles.size()) * n_groups_sel;

  // ---- window plans: the query tiles whose rows want the log-sum-exp get workgroups of their own ----
  // Only the last lse_rows rows are asked for their log-sum-exp (the recent window of Eq. 2).  Keeping the exact row
  // sum costs a step 7 % with heads of 128, 9 % with heads of 64 (two more vector instructions per pair of scores), so the
  // query tiles that hold such rows ("window tiles") are dealt to a set of workgroups of their own, sized by their share of
  // the work, and only those workgroups run the variant of the loop that keeps the sum.  A set of few workgroups needs units
  // small enough to be balanced over it: the window tiles' lists are cut into the number of slices that minimises an
  // estimate of the set's longest queue (equal units dealt evenly, the combination charged to the queue that closes a
  // list), and the set is made large enough not to be the last to finish.
  // KV-head groups of the XCD affinity of the dealing below: workgroup q runs on XCD q % 8, and the units of a KV
  // head stay on the XCDs x with x % Hkv == kvh (Hkv < 8) or x == kvh % 8
  const int32_t affinity_groups = (p.head_sel.empty() && n_cu % 8 == 0 && (g.Hkv % 8 == 0 || 8 % g.Hkv == 0)) ? std::min(g.Hkv, 8) : 1;
  auto window_tile = [&](int32_t qt) {
    return p.lse_rows > 0 && int64_t(qt + 1) * rows_per_qtile > int64_t(g.N) - p.lse_rows;
  };
  // Of a step that keeps the exact sum.  The cycles of every workgroup with the sum against those of the same plan without it:
  // median 1.070 and 1.085 over dense plans of 19 to 274 steps a workgroup (a launch as a whole differs by 2 to 7 %: units and
  // slices cost the same, and the clock is a little higher).
  const double kExactSumCost = g.d == 128 ? 1.07 : 1.09;
  struct WindowSet {
    int32_t n_queues, slices;
  };
  std::vector<WindowSet> window_sets;   // candidates; {0, 1}: no workgroups of their own
  {
    double steps_w = 0;
    int64_t lists_w = 0;
    int32_t shortest = INT32_MAX;
    for (int32_t qt = 0; qt < p.n_qtiles; ++qt)
      if (window_tile(qt)) {
        const int32_t len = p.qtile_begin[qt + 1] - p.qtile_begin[qt];
        steps_w += len;
        ++lists_w;
        shortest = std::min(shortest, len);
      }
    const double cost_w = kExactSumCost * steps_w * n_groups_sel, cost_rest = (double(p.tiles.size()) - steps_w) * n_groups_sel;
    // (not when the window tiles are a large share of the work -- text rows under a sparse pattern: units cut fine
    // enough to balance a large set pay more in unit switches and combinations than the other set saves)
    if (lists_w > 0 && 4 * cost_w <= cost_w + cost_rest && n_cu >= 2 &&
        (p.n_qtiles - lists_w) * int64_t(n_groups_sel) >= n_cu) {
      const int64_t units_w = lists_w * n_groups_sel, units_rest = (p.n_qtiles - lists_w) * int64_t(n_groups_sel);
      const double len = steps_w / double(lists_w);
      // longest queue of a set of nq workgroups, and the number of slices per list that gives it
      auto window_set = [&](int32_t nq, int32_t& slices) {
        double best = 0;
        for (int32_t ns = 1; ns <= std::min<int32_t>(kMaxSplits, std::max(1, shortest / 8)); ++ns) {
          const int64_t per_queue = (units_w * ns + nq - 1) / nq;
          const double longest = double(per_queue) * (len / ns + kUnitCost + (ns > 1 ? kSliceCost : 0.0)) +
                                 (ns > 1 ? combine_cost(ns) : 0.0);
          if (ns == 1 || longest < best) best = longest, slices = ns;
        }
        return kExactSumCost * best;
      };
      auto rest_set = [&](int32_t nq) { return (cost_rest + kUnitCost * double(units_rest)) / double(n_cu - nq); };
      // smallest set, from the window tiles' share of the work on, whose longest queue ends no later than the
      // other set's average one; failing that, the size with the smallest later end of the two
      // (a multiple of the number of KV-head groups of the XCD affinity below, so that every KV head keeps the same
      // number of workgroups in both sets)
      const int32_t nq0 = std::max<int32_t>(1, static_cast<int32_t>(cost_w / (cost_w + cost_rest) * n_cu));
      const int32_t nq_first = (nq0 + affinity_groups - 1) / affinity_groups * affinity_groups;
      const int32_t nq_last = std::min<int32_t>(n_cu - 1, 2 * nq0 + 8 + affinity_groups);
      WindowSet best{0, 1};
      double best_end = 0;
      for (int32_t nq = nq_first; nq <= nq_last; nq += affinity_groups) {
        int32_t slices = 1;
        const double end_w = window_set(nq, slices), end_r = rest_set(nq), end = std::max(end_w, end_r);
        if (best.n_queues == 0 || end < best_end) best_end = end, best = {nq, slices};
        if (end_w <= end_r) break;
      }
      // a neighbouring size may suit the other set's units better: the dealing below decides
      for (int32_t nq : {best.n_queues, best.n_queues - affinity_groups, best.n_queues + affinity_groups}) {
        if (nq < nq_first || nq > nq_last) continue;
        int32_t slices = 1;
        (void)window_set(nq, slices);
        window_sets.push_back({nq, slices});
      }
    }
  }
  if (window_sets.empty()) window_sets.push_back({0, 1});

  // ---- schedules: cut lists that are long against the average load, deal the units, keep the schedule that ends first ----
  // Workgroup q runs on XCD q % 8 (round-robin dispatch); when the head counts allow it, the units of one KV head stay on a
  // fixed set of XCDs, a home, so that each L2 holds the K/V of few KV heads.  Homes have equally many queues and the same
  // units, one for each of their head groups: one home is dealt, the others are copies of it.
  struct Deal {                            // of the units of one class onto the queues [q_lo, q_lo + n_homes * load.size())
    int32_t q_lo = 0, n_homes = 1;
    std::vector<double> load;              // of the queues of one home
    std::vector<std::vector<std::pair<int32_t, int32_t>>> units;   // per queue of a home: (item, n-th head group of the home)
  };
  struct Schedule {
    std::vector<WorkItem> items;
    std::vector<MergeItem> merges;
    std::vector<double> item_cost;
    Deal deal[2];                               // of the other tiles' units, of the window tiles'
    int32_t n_slots = 0, n_queues = 0, lse_queue0 = 0;
    double dealt_end = 0, end = 0;              // predicted, of the last queue, before and after the refinement
  };
  auto cut = [&](Schedule& s, double factor, const WindowSet& ws) {
    const int32_t chunk = std::max<int32_t>(8, static_cast<int32_t>(std::min(factor * total_steps / std::max(1, n_cu) + 0.5, 1e9)));
    for (int32_t qt = 0; qt < p.n_qtiles; ++qt) {
      const int32_t b = p.qtile_begin[qt], len = p.qtile_begin[qt + 1] - b;
      int32_t ns = 1;
      if (2 * int64_t(len) > 3 * int64_t(chunk)) ns = std::min<int32_t>((len + chunk - 1) / chunk, kMaxSplits);
      if (ws.n_queues > 0 && window_tile(qt)) ns = std::min(ws.slices, std::max(1, len / 8));
      if (ns == 1) {
        s.items.push_back({qt, b, len, 0, 1, -1});
        continue;
      }
      s.merges.push_back({qt, s.n_slots, ns, 0});
      int32_t pos = b;
      for (int32_t i = 0; i < ns; ++i) {
        const int32_t cnt = len / ns + (i < len % ns ? 1 : 0);
        s.items.push_back({qt, pos, cnt, i, ns, s.n_slots + i});
        pos += cnt;
      }
      s.n_slots += ns;
    }
    std::stable_sort(s.items.begin(), s.items.end(),
                     [](const WorkItem& x, const WorkItem& y) { return x.n_tiles > y.n_tiles; });
    for (const WorkItem& w : s.items) {
      double c = kUnitCost + cost_before[w.list_begin + w.n_tiles] - cost_before[w.list_begin];
      if (w.n_splits > 1) c += kSliceCost + (w.split == w.n_splits - 1 ? combine_cost(w.n_splits) : 0.0);
      s.item_cost.push_back(c);
    }
  };
  // Units are dealt longest first, each to the least-loaded queue that may run it.  Queues [0, lse_queue0) hold the units of
  // the other tiles, [lse_queue0, n_queues) those of the window tiles; a plan without a window keeps one class: every
  // workgroup keeps the exact sum when the log-sum-exp is asked for.
  auto item_class = [&](const Schedule& s, size_t it) { return s.lse_queue0 > 0 && window_tile(s.items[it].qtile) ? 1 : 0; };
  auto homes_of = [&](const Schedule& s, int32_t n) {
    // (not for a head subset: its KV heads may be few, and every queue has to receive a unit; and only with the same number
    // of queues for every KV head: the sets of a divided plan are sized for that)
    const int32_t homes = std::min(g.Hkv, 8);
    return p.head_sel.empty() && s.n_queues % 8 == 0 && (g.Hkv % 8 == 0 || 8 % g.Hkv == 0) && n % homes == 0 ? homes : 1;
  };
  // Head groups of home `home` of n_homes, ascending (without homes: every selected group).
  auto groups_of_home = [&](int32_t n_homes, int32_t home) {
    std::vector<int32_t> groups;
    for (int32_t grp = 0; grp < g.n_groups; ++grp)
      if (group_selected(grp) && grp * g.Gs / g.G % n_homes == home % n_homes) groups.push_back(grp);
    return groups;
  };
  auto deal_class = [&](const Schedule& s, int cls, int32_t q_lo, int32_t q_hi, bool loads_only) {
    Deal d;
    d.q_lo = q_lo;
    d.n_homes = homes_of(s, q_hi - q_lo);
    const int32_t n = (q_hi - q_lo) / d.n_homes, n_groups_home = n_groups_sel / d.n_homes;
    d.load.assign(n, 0.0);
    if (!loads_only) d.units.resize(n);
    typedef std::pair<double, int32_t> LoadQueue;   // least loaded first, then lowest index
    std::vector<LoadQueue> idle(n);
    for (int32_t q = 0; q < n; ++q) idle[q] = {0.0, q};
    std::priority_queue<LoadQueue, std::vector<LoadQueue>, std::greater<LoadQueue>> heap(std::greater<LoadQueue>(), std::move(idle));
    for (size_t it = 0; it < s.items.size(); ++it) {
      if (item_class(s, it) != cls) continue;
      for (int32_t i = 0; i < n_groups_home; ++i) {
        LoadQueue lq = heap.top();
        heap.pop();
        if (!loads_only) d.units[lq.second].emplace_back(static_cast<int32_t>(it), i);
        lq.first = d.load[lq.second] += s.item_cost[it];
        heap.push(lq);
      }
    }
    return d;
  };
  // Refinement: while it lowers the larger of the two loads, move a unit from the fullest queue to another one, or exchange a
  // unit of each.
  auto refine = [](const Schedule& s, Deal& d) {
    const int32_t n = static_cast<int32_t>(d.load.size());
    auto& load = d.load;
    for (int32_t round = 0; round < 8 * n; ++round) {
      const int32_t qa = static_cast<int32_t>(std::max_element(load.begin(), load.end()) - load.begin());
      auto& ua = d.units[qa];
      double best_gain = 1e-9;
      int32_t best_q = -1;
      size_t best_u = 0, best_v = SIZE_MAX;
      for (size_t u = 0; u < ua.size(); ++u) {
        const double cu = s.item_cost[ua[u].first];
        bool seen = false;   // a unit of the same cost
        for (size_t x = 0; x < u && !seen; ++x) seen = s.item_cost[ua[x].first] == cu;
        if (seen) continue;
        for (int32_t qb = 0; qb < n; ++qb) {
          if (0.5 * (load[qa] - load[qb]) <= best_gain) continue;   // (no larger gain there)
          // move u: new pair maximum = max(load[qa] - cu, load[qb] + cu)
          double gain = load[qa] - std::max(load[qa] - cu, load[qb] + cu);
          if (gain > best_gain) best_gain = gain, best_q = qb, best_u = u, best_v = SIZE_MAX;
          for (size_t v = 0; v < d.units[qb].size(); ++v) {
            const double cv = s.item_cost[d.units[qb][v].first];
            if (cv >= cu) continue;
            gain = load[qa] - std::max(load[qa] - cu + cv, load[qb] + cu - cv);
            if (gain > best_gain) best_gain = gain, best_q = qb, best_u = u, best_v = v;
          }
        }
      }
      if (best_q < 0) break;
      auto& ub = d.units[best_q];
      const double cu = s.item_cost[ua[best_u].first];
      double moved = cu;
      if (best_v == SIZE_MAX) {
        ub.push_back(ua[best_u]);
        ua.erase(ua.begin() + best_u);
      } else {
        moved -= s.item_cost[ub[best_v].first];
        std::swap(ua[best_u], ub[best_v]);
      }
      load[qa] -= moved;
      load[best_q] += moved;
    }
  };
  // `limit`: a schedule whose queues end no sooner on average, or whose longest unit does not, is given up undealt.
  auto make = [&](double factor, const WindowSet& ws, bool loads_only, double limit) {
    Schedule s;
    cut(s, factor, ws);
    const int64_t n_units = int64_t(s.items.size()) * n_groups_sel;
    s.n_queues = static_cast<int32_t>(std::min<int64_t>(std::max(1, n_cu), std::max<int64_t>(1, n_units)));
    int64_t units_w = 0;
    if (ws.n_queues > 0)
      for (const WorkItem& w : s.items) units_w += window_tile(w.qtile) ? n_groups_sel : 0;
    s.lse_queue0 = ws.n_queues > 0 ? s.n_queues - static_cast<int32_t>(std::min<int64_t>(ws.n_queues, units_w)) : 0;
    const int32_t q_split = s.lse_queue0 > 0 ? s.lse_queue0 : s.n_queues;
    double sum[2] = {0, 0}, longest[2] = {0, 0};   // per class
    for (size_t it = 0; it < s.items.size(); ++it) {
      const int cls = item_class(s, it);
      sum[cls] += s.item_cost[it] * n_groups_sel;
      longest[cls] = std::max(longest[cls], s.item_cost[it]);
    }
    s.end = std::max(sum[0] / q_split, longest[0]);
    if (q_split < s.n_queues) s.end = std::max(s.end, kExactSumCost * std::max(sum[1] / (s.n_queues - q_split), longest[1]));
    if (s.end >= limit) return s;
    auto last_end = [&]() {
      double end = *std::max_element(s.deal[0].load.begin(), s.deal[0].load.end());
      if (!s.deal[1].load.empty())
        end = std::max(end, kExactSumCost * *std::max_element(s.deal[1].load.begin(), s.deal[1].load.end()));
      return end;
    };
    if (q_split < s.n_queues) s.deal[1] = deal_class(s, 1, q_split, s.n_queues, loads_only);
    s.deal[0] = deal_class(s, 0, 0, q_split, loads_only);
    s.dealt_end = s.end = last_end();
    if (loads_only) return s;
    for (Deal& d : s.deal) refine(s, d);
    s.end = last_end();
    return s;
  };
  // Slice lengths, as factors of the average load of a workgroup.  None suits all: whole lists leave a shape with few units
  // per workgroup with a long tail, short slices cost unit switches and combinations.  0.8 unless another one ends 3 %
  // sooner by the model, whose workgroups' ends scatter by as much.  Prefill alone, always 0.8 -> this, with the costs of its day:
  // dense, 14 frames of 19 x 8 patches + 51 tokens, 28/4 heads of 128: 65.2 -> 53.7 us; 11 of 22 x 11 + 10, 8/8 of 64: 33.7 ->
  // 25.0; sparse, 55 of 24 x 8 + 264, 8/8 of 128: 75.3 -> 61.1; 6 of 22 x 19 + 22, 28/4 of 64: 32.5 -> 26.5; 66 drawn shapes 0.97
  // in the mean.
  // Plans with more than three units per workgroup balance with any of them and take 0.8 without a search, as do those whose
  // first schedule ends within 3 % of the average load of uncut lists.  The search deals loads only, and no schedule that the
  // one in hand beats on the average already; the one it finds is dealt in full and refined like the first.  Planning 178
  // shapes (170 drawn), one length always -> all homes dealt, with the search -> one home, with the search: 184 -> 142 -> 95 ms
  // in all; dense window plan, 8 frames of 24 x 24 + 128, 32/8 heads, 0.37 -> 0.62 -> 0.20; sparse, 64 frames of 16 x 16 + 256,
  // 28/4 heads, 5.6 -> 2.0 -> 1.3; dense, 128 frames, 18 -> 14 -> 13 (its lists and steps, not the schedule).
  constexpr double kSliceFactor = 0.8, kOtherFactors[] = {0.4, 0.55, 0.65, 1.0, 1.25, 1.6, 1e9}, kSooner = 1.03;
  const double kNoLimit = std::numeric_limits<double>::infinity();
  Schedule chosen = make(kSliceFactor, window_sets[0], false, kNoLimit);
  const double no_sooner = (cost_before.back() + kUnitCost * p.n_qtiles) * n_groups_sel / std::max(1, n_cu);
  if (int64_t(p.n_qtiles) * n_groups_sel <= 3 * int64_t(n_cu) && chosen.end > kSooner * no_sooner) {
    double other_end = chosen.dealt_end / kSooner, other_factor = 0;
    WindowSet other_set = window_sets[0];
    auto consider = [&](double factor, const WindowSet& ws) {
      const double end = make(factor, ws, true, other_end).end;
      if (end < other_end) other_end = end, other_factor = factor, other_set = ws;
    };
    for (size_t i = 1; i < window_sets.size(); ++i) consider(kSliceFactor, window_sets[i]);
    const WindowSet ws = other_set;
    for (double factor : kOtherFactors) consider(factor, ws);
    if (other_factor > 0) {
      Schedule other = make(other_factor, other_set, false, kNoLimit);
      if (other.end * kSooner < chosen.end) chosen = std::move(other);
    }
  }
  p.items = std::move(chosen.items);
  p.merges = std::move(chosen.merges);
  p.n_slots = chosen.n_slots;
  p.n_queues = chosen.n_queues;
  p.lse_queue0 = chosen.lse_queue0;
  std::vector<std::vector<int32_t>> queues(p.n_queues);   // flat (item, group) pairs
  for (const Deal& d : chosen.deal)
    for (int32_t home = 0; home < d.n_homes && !d.load.empty(); ++home) {
      // queues of home x: q % n_homes == x
      const std::vector<int32_t> groups = groups_of_home(d.n_homes, d.q_lo + home);
      for (size_t i = 0; i < d.units.size(); ++i)
        for (const auto& u : d.units[i]) {
          auto& queue = queues[d.q_lo + home + d.n_homes * static_cast<int32_t>(i)];
          queue.push_back(u.first);
          queue.push_back(groups[u.second]);
        }
    }
  // Order within a queue: slices of split lists first, except the closing slice of a list, which goes last (when it
  // ends, the other slices of its list, run first elsewhere, have normally long arrived: the workgroup that the
  // cost model charged for combining them is then the one that does); whole lists in between, longest first (item
  // indices ascend with decreasing length).
  auto order_class = [&](int32_t it) {
    const WorkItem& w = p.items[it];
    return w.n_splits == 1 ? 1 : (w.split == w.n_splits - 1 ? 2 : 0);
  };
  for (auto& qv : queues) {
    std::vector<std::pair<int32_t, int32_t>> pairs;
    for (size_t u = 0; u + 1 < qv.size(); u += 2) pairs.emplace_back(qv[u], qv[u + 1]);
    std::stable_sort(pairs.begin(), pairs.end(), [&](const std::pair<int32_t, int32_t>& x, const std::pair<int32_t, int32_t>& y) {
      const int cx = order_class(x.first), cy = order_class(y.first);
      return cx != cy ? cx < cy : x < y;
    });
    for (size_t u = 0; u < pairs.size(); ++u) {
      qv[2 * u] = pairs[u].first;
      qv[2 * u + 1] = pairs[u].second;
    }
  }

  std::vector<uint8_t> owned(size_t(g.Hkv) * size_t(n_ktiles), 0);   // (KV head, key tile) pairs that have an owner step
  p.units.clear();
  p.stream.clear();
  p.queue_begin.assign(1, 0);
  p.queue_units.clear();
  p.queue_units_begin.assign(1, 0);
  for (int32_t q = 0; q < p.n_queues; ++q) {
    for (size_t u = 0; u + 1 < queues[q].size(); u += 2) {
      const WorkItem& w = p.items[queues[q][u]];
      const int32_t grp = queues[q][u + 1], head0 = grp * g.Gs, kvh = head0 / g.G;
      p.queue_units.push_back(queues[q][u]);
      p.queue_units.push_back(head0);
      Unit un{};
      un.row0 = w.qtile * rows_per_qtile;
      un.head0 = head0;
      un.n_splits = w.n_splits;
      un.ws_row0 = w.slot >= 0 ? (w.slot * g.n_groups + grp) * (kWaves * kBlockRows) : -1;
      un.ws_row_first = w.slot >= 0 ? ((w.slot - w.split) * g.n_groups + grp) * (kWaves * kBlockRows) : -1;
      un.counter = w.slot >= 0 ? (w.slot - w.split) * g.n_groups + grp : -1;
      p.units.push_back(un);
      for (int32_t t = 0; t < w.n_tiles; ++t) {
        const TileRef& r = p.tiles[w.list_begin + t];
        StreamEntry e;
        e.kv_off = uint32_t((int64_t(kvh) * g.kv_sh + int64_t(r.tile) * BK * g.kv_st) * 2);
        const int32_t k0 = r.tile * BK, rows = std::min(BK, g.N - k0);
        uint8_t& own = owned[size_t(kvh) * size_t(n_ktiles) + size_t(r.tile)];
        e.need = r.need | ((t == w.n_tiles - 1) ? kStepLast : 0u) | ((t == 0) ? kStepFirst : 0u) |
                 (uint32_t(rows - 1) << 18) | (own ? 0u : kStepOwner);
        own = 1;
        e.kinds = r.kinds;
        e.k0 = k0;
        p.stream.push_back(e);
      }
      if (u + 2 < queues[q].size())   // another unit follows
        p.stream[p.stream.size() - (w.n_tiles >= 2 ? 2 : 1)].need |= kStepFetchQ;
    }
    const size_t n_units_q = queues[q].size() / 2;
    for (size_t u = n_units_q, next = 0; u-- > 0;) {   // how far the next slice of the queue, or its end, is
      Unit& un = p.units[p.units.size() - n_units_q + u];
      un.to_next_slice = static_cast<int32_t>(++next);
      if (un.n_splits > 1) next = 0;
    }
    p.queue_begin.push_back(static_cast<int32_t>(p.stream.size()));
    p.queue_units_begin.push_back(static_cast<int32_t>(p.queue_units.size() / 2));
  }
  p.units.push_back(Unit{});  // spare record: the kernel fetches the record after the current unit unconditionally
  return chosen.end;
}

}  // namespace

void build_plan(purekv_plan& p, int n_cu) {
  Geometry& g = p.g;
  p.n_cu = n_cu;
  // Stacking the query heads of a KV group in one workgroup makes every wavefront of the workgroup need the
  // same key tiles (the mask depends on the row, not on the head), so nobody waits at the tile barriers for
  // work it does not share.  The dense pattern has little such imbalance (only the diagonal tiles): it stacks
  // only when that fills all wavefronts, else one head x 8 row blocks keeps every SIMD busy.
  const bool sparse = g.pattern != PUREKV_PATTERN_DENSE;
  const int32_t gs = largest_divisor_up_to(g.G, kWaves), r = kWaves / gs;
  const bool stack = (sparse && gs >= 2) || (gs * r == kWaves && gs >= 2);
  // A head subset keeps the stacked shape when it is made of whole stacks (e.g. whole KV groups); otherwise it is
  // planned head by head.
  bool whole_stacks = true;
  p.n_heads_sel = g.Hq;
  if (!p.head_sel.empty()) {
    p.n_heads_sel = 0;
    for (int32_t hq = 0; hq < g.Hq; ++hq) {
      p.n_heads_sel += p.head_sel[hq] != 0;
      whole_stacks &= (p.head_sel[hq] != 0) == (p.head_sel[hq - hq % gs] != 0);
    }
  }
  auto build = [&](int32_t gs1, int32_t r1) {
    g.Gs = gs1;
    g.R = r1;
    g.n_groups = g.Hq / gs1;
    return build_shape(p, n_cu);
  };
  const bool use_stack = stack && whole_stacks;
  int32_t Gs = use_stack ? gs : 1, R = use_stack ? r : kWaves;

  // Few units: fewer wavefronts share a compute unit.  A SIMD with one wavefront takes about 0.7 of the time for a step that one
  // with two takes, so half the row blocks, or half the heads, in a workgroup pay where compute units would be idle otherwise;
  // going on to two wavefronts and one (shorter starts, a few %) where half of them still would.  Where every compute unit has
  // plenty of steps either way (slices of the long lists fill them) the same work in twice the steps is slower: up to 15 steps
  // a compute unit the halves are taken, beyond that only halves of eight wavefronts that end sooner by the model.
  // Prefill alone, dense, us, eight wavefronts -> four, steps a compute unit with four: 8/2 heads of 128, 1327 tokens (3.4) 26.4 ->
  // 21.4; 16/2 of 128, 1990 (15) 35.8 -> 32.1; 8/8 of 64, 2896 (16) 26.2 -> 28.3; 8/8 of 128, 3279 (20) 39.8 -> 46.8; 4/2 of 64, 5203
  // (26) 34.8 -> 43.2; and 2/1 of 64, 5792 (16) 31.6 -> 27.7, by the model.  Four -> two: 2/1 of 128, 2793 (7) 26.5 -> 26.1, 4579
  // (20) 32.4 -> 46.6.  535 plans of 318 shapes: 0.884 of eight wavefronts' time (0.904 without the limit, 51 slower than with
  // eight by more than 3 %, up to 1.37; now four: 1.06 and 1.08, 1448 tokens, 16/2, and 1.10 and 1.23, 3946 sparse, 4/2).
  // (Sparse plans keep two heads stacked.  Left out and not measured with fewer wavefronts: head subsets, and the sparse plans of
  // one head per KV head that a subset of single heads shares its lists with at any number of workgroups.)
  if (p.head_sel.empty() && !(sparse && g.G == 1)) {
    double pairs = -1;   // allowed pairs of a head
    auto steps = [&](int32_t waves) {   // a compute unit's share of the steps, partly used ones left out
      if (pairs < 0) {
        pairs = 0;
        for (int32_t i = 0; i < g.N; ++i) pairs += row_pairs(row_set(g, i), i);
      }
      return pairs * g.Hq / (double(waves) * kBlockRows * PUREKV_BK * n_cu);
    };
    constexpr double kFewSteps = 15.0;
    const double kAloneCost = g.d == 128 ? 0.68 : 0.70;   // of a step, with one wavefront a SIMD
    while (Gs * R > 1) {
      const bool rows = R % 2 == 0;
      if (!rows && (Gs % 2 != 0 || (sparse && Gs == 2))) break;
      const int32_t gs1 = rows ? Gs : Gs / 2, r1 = rows ? R / 2 : R, waves = gs1 * r1;
      const int64_t units = int64_t((g.N + r1 * kBlockRows - 1) / (r1 * kBlockRows)) * (g.Hq / gs1);
      if ((waves < kWaves / 2 ? 2 : 1) * units > n_cu) break;
      if (steps(waves) > kFewSteps) {
        if (Gs * R <= kWaves / 2) break;
        const double end = build(Gs, R);
        if (kAloneCost * build(gs1, r1) >= end) break;
      }
      Gs = gs1;
      R = r1;
    }
  }
  (void)build(Gs, R);
}

}  // namespace purekv
