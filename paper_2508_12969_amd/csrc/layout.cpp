// Host-side layout builder: per-head CSR of kept key tiles, launch order and padding masks.
//
// Keep rule (Sec. 4.1 of the paper, with Eq. 1 / Eq. 2 read in tile units): the tile-frame
// distance |kt-qt| selects a group; inside the group a key tile is kept when it lies in either
// of two query-centred windows, clipped by the tile grid.  Both windows contain the query's own
// column, so on one tile row of one frame the kept columns form a single interval; the builder
// walks frames and tile rows in ascending order and emits those intervals, which yields the
// ascending tile ids directly.  No HIP call is made here.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <new>
#include <queue>

#include "layout.h"

namespace ca {

static thread_local char g_error[512] = "";

void set_error(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_error, sizeof(g_error), fmt, ap);
  va_end(ap);
}
void clear_error() { g_error[0] = '\0'; }
const char* last_error() { return g_error; }

namespace {

struct Interval {
  int32_t lo, hi;  // inclusive; empty when lo > hi
};

inline Interval clip(int32_t center, int32_t radius, int32_t len) {
  // radius can be as large as INT32_MAX; widen before adding
  int64_t lo = (int64_t)center - radius, hi = (int64_t)center + radius;
  return {(int32_t)std::max<int64_t>(lo, 0), (int32_t)std::min<int64_t>(hi, len - 1)};
}

// Tiles of one axis a window covers: clipped around the query, or (clamp) moved inward so that it
// keeps its 2*radius+1 tiles (the whole axis if that is shorter).
inline Interval window_range(int32_t center, int32_t radius, int32_t len, bool clamp) {
  if (!clamp) return clip(center, radius, len);
  if (2 * (int64_t)radius + 1 >= len) return {0, len - 1};
  const int32_t c = std::min(std::max(center, radius), len - 1 - radius);
  return {c - radius, c + radius};
}

inline bool present(const ca_window& w) { return w.rh >= 0 && w.rw >= 0; }

// Resolved windows of one head for every tile-frame distance 0..nT-1 (group lookup done once).
struct HeadPlan {
  std::vector<int8_t> has;      // [nT] distance covered by some group
  std::vector<ca_window> a, b;  // [nT]
  bool clamp = false;           // windows keep their size at the border (centre moved inward)
};

int plan_head(const ca_head& h, int32_t head_index, int32_t nT, HeadPlan& plan) {
  if (h.num_groups < 0 || h.num_groups > CA_MAX_GROUPS) {
    set_error("head %d: num_groups=%d outside 0..%d", head_index, h.num_groups, CA_MAX_GROUPS);
    return CA_ERR_INVALID_ARG;
  }
  if (h.num_groups > 0 && h.groups == nullptr) {
    set_error("head %d: groups is null", head_index);
    return CA_ERR_INVALID_ARG;
  }
  int32_t last = -1;
  for (int32_t g = 0; g < h.num_groups; ++g) {
    if (h.groups[g].max_dt <= last) {
      set_error("head %d: max_dt must be non-negative and strictly increasing (group %d has %d after %d)",
                head_index, g, h.groups[g].max_dt, last);
      return CA_ERR_INVALID_ARG;
    }
    last = h.groups[g].max_dt;
  }
  if (h.clamp_centre != 0 && h.clamp_centre != 1) {
    set_error("head %d: clamp_centre must be 0 or 1", head_index);
    return CA_ERR_INVALID_ARG;
  }
  plan.clamp = h.clamp_centre == 1;
  plan.has.assign(nT, 0);
  plan.a.assign(nT, ca_window{-1, -1});
  plan.b.assign(nT, ca_window{-1, -1});
  int32_t g = 0;
  for (int32_t dt = 0; dt < nT; ++dt) {
    while (g < h.num_groups && h.groups[g].max_dt < dt) ++g;
    if (g == h.num_groups) break;
    plan.has[dt] = 1;
    plan.a[dt] = h.groups[g].a;
    plan.b[dt] = h.groups[g].b;
  }
  return CA_OK;
}

// Visits the kept video tiles of query tile (qt,qh,qw) as runs [first_id, first_id+len) in ascending order.
template <class F>
inline void for_each_run(const ca_layout& L, const HeadPlan& plan, int32_t qt, int32_t qh, int32_t qw, F&& emit) {
  for (int32_t kt = 0; kt < L.nT; ++kt) {
    const int32_t dt = kt > qt ? kt - qt : qt - kt;
    if (!plan.has[dt]) continue;
    const ca_window &wa = plan.a[dt], &wb = plan.b[dt];
    const bool pa = present(wa), pb = present(wb);
    if (!pa && !pb) continue;
    Interval ha{0, -1}, hb{0, -1}, ca_{0, -1}, cb{0, -1};
    if (pa) { ha = window_range(qh, wa.rh, L.nH, plan.clamp); ca_ = window_range(qw, wa.rw, L.nW, plan.clamp); }
    if (pb) { hb = window_range(qh, wb.rh, L.nH, plan.clamp); cb = window_range(qw, wb.rw, L.nW, plan.clamp); }
    const int32_t h_lo = pa && pb ? std::min(ha.lo, hb.lo) : (pa ? ha.lo : hb.lo);
    const int32_t h_hi = pa && pb ? std::max(ha.hi, hb.hi) : (pa ? ha.hi : hb.hi);
    for (int32_t kh = h_lo; kh <= h_hi; ++kh) {
      const bool in_a = pa && kh >= ha.lo && kh <= ha.hi;
      const bool in_b = pb && kh >= hb.lo && kh <= hb.hi;
      int32_t lo, hi;
      if (in_a && in_b) { lo = std::min(ca_.lo, cb.lo); hi = std::max(ca_.hi, cb.hi); }
      else if (in_a) { lo = ca_.lo; hi = ca_.hi; }
      else if (in_b) { lo = cb.lo; hi = cb.hi; }
      else continue;  // rows between two disjoint height ranges cannot occur (both contain qh, clamped or not), kept for safety
      const int64_t first = ((int64_t)kt * L.nH + kh) * L.nW + lo;
      emit((int32_t)first, hi - lo + 1);
    }
  }
}

void build_slot_masks(ca_layout& L) {
  // A tile's padding pattern depends only on whether it is the last tile along each axis.  A mask holds the
  // first 128 slots; no kernel that reads masks takes larger tiles.
  const ca_problem& p = L.prob;
  const int32_t rem_t = p.T - (L.nT - 1) * p.tt, rem_h = p.H - (L.nH - 1) * p.th, rem_w = p.W - (L.nW - 1) * p.tw;
  L.class_mask.clear();
  SlotMask full{};
  constexpr int64_t kMaskSlots = 8 * (int64_t)sizeof(SlotMask);
  for (int64_t s = 0; s < std::min(L.B, kMaskSlots); ++s) full.w[s >> 5] |= 1u << (s & 31);
  L.class_mask.push_back(full);
  int class_of_edge[8];
  for (int e = 0; e < 8; ++e) {
    const int32_t lim_t = (e & 4) ? rem_t : p.tt, lim_h = (e & 2) ? rem_h : p.th, lim_w = (e & 1) ? rem_w : p.tw;
    if (lim_t == p.tt && lim_h == p.th && lim_w == p.tw) { class_of_edge[e] = 0; continue; }
    SlotMask m{};
    for (int32_t dt = 0; dt < lim_t; ++dt)
      for (int32_t dy = 0; dy < lim_h; ++dy)
        for (int32_t dx = 0; dx < lim_w; ++dx) {
          const int32_t s = (dt * p.th + dy) * p.tw + dx;
          if (s < kMaskSlots) m.w[s >> 5] |= 1u << (s & 31);
        }
    class_of_edge[e] = (int)L.class_mask.size();
    L.class_mask.push_back(m);
  }
  L.tile_class.assign(L.n, 0);
  for (int32_t kt = 0; kt < L.nT; ++kt)
    for (int32_t kh = 0; kh < L.nH; ++kh)
      for (int32_t kw = 0; kw < L.nW; ++kw) {
        const int e = (kt == L.nT - 1 ? 4 : 0) | (kh == L.nH - 1 ? 2 : 0) | (kw == L.nW - 1 ? 1 : 0);
        L.tile_class[((int64_t)kt * L.nH + kh) * L.nW + kw] = class_of_edge[e];
      }
  // Tile mass of 128-token tiles: with the tokens first, a padded tile costs its blocks of 32 keys that hold any, instead of all
  // four, but its rows are gathered one by one.  Over 100 layouts of the two head dims, without / with (every layout): empty share
  // of 0.12 to 0.19 at head dim 128 1.01 to 1.15 times, of 0.2 to 0.3 1.05 to 1.24, from there to 1.49; 0.10 0.97, 0.07 (119K tokens x
  // 12 heads) 48.6 / 49.7 ms; at head dim 64 of 0.06 and 0.08 1.07 and 1.13 times, then to 1.52.
  int64_t empty = 0;  // blocks of 32 keys without a token, of four per tile
  for (int32_t c : L.tile_class) {
    int tokens = 0;
    for (uint32_t w : L.class_mask[c].w) tokens += __builtin_popcount(w);
    empty += (128 - tokens) / 32;
  }
  L.mass_tokens_first = L.B == 128 && empty * (p.head_dim == 64 ? 16 : 8) >= 4 * L.n;
}

void build_order(ca_layout& L) {
  // Descending kept count, ties by ascending row id: a counting sort over counts 0..n.
  const int64_t rows = (int64_t)L.prob.num_heads * L.n;
  std::vector<int64_t> bucket_start(L.n + 2, 0);
  for (int64_t r = 0; r < rows; ++r) {
    const int64_t c = L.row_ptr[r + 1] - L.row_ptr[r];
    ++bucket_start[(L.n - c) + 1];  // bucket 0 holds count n, bucket n holds count 0
  }
  for (int64_t b = 0; b <= L.n; ++b) bucket_start[b + 1] += bucket_start[b];
  L.order.resize(rows);
  for (int64_t r = 0; r < rows; ++r) {
    const int64_t c = L.row_ptr[r + 1] - L.row_ptr[r];
    L.order[bucket_start[L.n - c]++] = (int32_t)r;
  }
}

}  // namespace

// A workgroup of the paired kernel: two rows of one head (b = -1: one), the assignment of its waves,
// and the length of its walk (the union of the two rows).
struct PairGroup {
  int32_t a, b;
  uint32_t desc;
  int64_t walked;
};

static int64_t union_size(const ca_layout& L, int64_t ra, int64_t rb) {
  if (rb < 0) return L.row_ptr[ra + 1] - L.row_ptr[ra];
  int64_t i = L.row_ptr[ra], ie = L.row_ptr[ra + 1], j = L.row_ptr[rb], je = L.row_ptr[rb + 1], m = 0;
  while (i < ie && j < je) {
    const int32_t ti = L.col_idx[i], tj = L.col_idx[j];
    i += ti <= tj;
    j += tj <= ti;
    ++m;
  }
  return m + (ie - i) + (je - j);
}

// Launch order and walk lists of the paired kernel from its workgroups: longest walks first, ties
// in the order built (head, then tile id); pair_rows[2i], pair_rows[2i+1] are row ids head*n + tile.
// The walk of a workgroup is the union of its two rows in ascending tile order, one word per tile:
// tile id | kPairInFirst if the first row keeps the tile | kPairInSecond if the second does.
static void emit_pair_tables(ca_layout& L, std::vector<PairGroup>& groups) {
  std::stable_sort(groups.begin(), groups.end(), [](const PairGroup& x, const PairGroup& y) { return x.walked > y.walked; });
  L.pair_rows.resize(2 * groups.size());
  L.pair_desc.resize(groups.size());
  for (size_t i = 0; i < groups.size(); ++i) {
    L.pair_rows[2 * i] = groups[i].a;
    L.pair_rows[2 * i + 1] = groups[i].b;
    L.pair_desc[i] = (int32_t)groups[i].desc;
  }
  L.pair_walk_ptr.assign(groups.size() + 1, 0);
  for (size_t i = 0; i < groups.size(); ++i) L.pair_walk_ptr[i + 1] = L.pair_walk_ptr[i] + groups[i].walked;
  L.pair_walk.resize((size_t)L.pair_walk_ptr[groups.size()]);
  for (size_t p = 0; p < groups.size(); ++p) {
    const int64_t ra = groups[p].a, rb = groups[p].b;
    int64_t i = L.row_ptr[ra], ie = L.row_ptr[ra + 1];
    int64_t j = rb < 0 ? 0 : L.row_ptr[rb], je = rb < 0 ? 0 : L.row_ptr[rb + 1];
    int64_t o = L.pair_walk_ptr[p];
    while (i < ie || j < je) {
      const int32_t ti = i < ie ? L.col_idx[i] : INT32_MAX, tj = j < je ? L.col_idx[j] : INT32_MAX;
      const int32_t t = ti < tj ? ti : tj;
      L.pair_walk[o++] = (int32_t)((uint32_t)t | (ti == t ? kPairInFirst : 0u) | (tj == t ? kPairInSecond : 0u));
      i += ti == t;
      j += tj == t;
    }
  }
}

// 64-token tiles: every query tile of a head is paired with a neighbour.
static void build_pair_table(ca_layout& L) {
  // Partner of a video tile: its neighbour along one grid axis (coordinates 2i and 2i+1; the last
  // tile of an odd extent stays single).  Which axis costs the fewest walked tiles depends on the
  // head's windows (a neighbour along an axis in which the windows are wide shares almost all of
  // its list), so every head takes the axis with the smallest sum of union sizes.  Text tiles pair
  // up in id order.
  const int64_t n = L.n;
  const int32_t ext[3] = {L.nT, L.nH, L.nW};
  const int64_t stride[3] = {(int64_t)L.nH * L.nW, L.nW, 1};
  auto for_pairs = [&](int axis, auto&& visit) {  // visit(tile_a, tile_b or -1) over the video tiles
    for (int32_t t = 0; t < L.nT; ++t)
      for (int32_t h = 0; h < L.nH; ++h)
        for (int32_t w = 0; w < L.nW; ++w) {
          const int32_t c[3] = {t, h, w};
          if (c[axis] & 1) continue;
          const int64_t id = ((int64_t)t * L.nH + h) * L.nW + w;
          visit(id, c[axis] + 1 < ext[axis] ? id + stride[axis] : (int64_t)-1);
        }
  };
  std::vector<PairGroup> groups;
  for (int32_t head = 0; head < L.prob.num_heads; ++head) {
    const int64_t base = (int64_t)head * n;
    // candidates: the axes with at least two tiles, tried in the order w, h, t; the first of the cheapest wins
    int best_axis = 2;
    int64_t best_cost = -1;
    for (int axis = 2; axis >= 0; --axis) {
      if (ext[axis] < 2) continue;
      int64_t cost = 0;
      for_pairs(axis, [&](int64_t a, int64_t b) { cost += union_size(L, base + a, b < 0 ? -1 : base + b); });
      if (best_cost < 0 || cost < best_cost) best_cost = cost, best_axis = axis;
    }
    constexpr uint32_t kSingle = pair_desc_wave(0, 0, 0) | pair_desc_wave(1, 0, 1);  // a tile without a partner
    for_pairs(best_axis, [&](int64_t a, int64_t b) {
      const int64_t rb = b < 0 ? -1 : base + b;
      groups.push_back({(int32_t)(base + a), (int32_t)rb, rb < 0 ? kSingle : kPairPlain, union_size(L, base + a, rb)});
    });
    for (int64_t a = L.n_vid; a < n; a += 2) {
      const int64_t rb = a + 1 < n ? base + a + 1 : -1;
      groups.push_back({(int32_t)(base + a), (int32_t)rb, rb < 0 ? kSingle : kPairPlain, union_size(L, base + a, rb)});
    }
  }
  emit_pair_tables(L, groups);
}

// 128-token tiles: a query tile on a padded face of the grid holds tokens for one to three waves
// only (its slots are handed to lanes token-holding slots first), and in a workgroup of its own the
// other waves idle while the workgroup still pays for the tile copies and the barriers of every
// step.  Such tiles are packed along w, inside one row of tiles of the grid: their waves fill
// workgroups of four in order, a tile's waves may continue in the next workgroup, and a workgroup
// serves at most two tiles (it walks the union of their rows).  A head is packed only if that is
// cheaper by the measured cost of a tile step with 1, 2, 3 or 4 working waves (65, 73, 88, 100):
// neighbours with narrow windows share too little of their lists.  launch_rows is then the launch
// order of both kinds of workgroup: the rows that keep a workgroup of their own and the packed ones.
static void build_packed_faces(ca_layout& L) {
  const int64_t n = L.n;
  static const int64_t kStepCost[5] = {0, 65, 73, 88, 100};
  std::vector<int32_t> waves(n, 4);
  bool any = false;
  for (int64_t t = 0; t < L.n_vid; ++t) {
    const SlotMask& m = L.class_mask[L.tile_class[t]];
    const int valid = __builtin_popcount(m.w[0]) + __builtin_popcount(m.w[1]) + __builtin_popcount(m.w[2]) + __builtin_popcount(m.w[3]);
    waves[t] = (valid + 31) / 32;
    any = any || waves[t] < 4;
  }
  L.packed_faces = false;
  L.launch_rows.clear();
  if (!any) return;
  std::vector<PairGroup> groups, head_groups;
  std::vector<char> packed((size_t)L.prob.num_heads * n, 0);
  for (int32_t head = 0; head < L.prob.num_heads; ++head) {
    const int64_t base = (int64_t)head * n;
    head_groups.clear();
    int64_t plain_cost = 0;
    for (int32_t kt = 0; kt < L.nT; ++kt)
      for (int32_t kh = 0; kh < L.nH; ++kh) {
        PairGroup cur{-1, -1, 0, 0};
        int used = 0;
        auto flush = [&]() {
          if (used) head_groups.push_back(cur);
          cur = PairGroup{-1, -1, 0, 0};
          used = 0;
        };
        for (int32_t kw = 0; kw < L.nW; ++kw) {
          const int64_t t = ((int64_t)kt * L.nH + kh) * L.nW + kw;
          if (waves[t] >= 4) {
            flush();
            continue;
          }
          plain_cost += (L.row_ptr[base + t + 1] - L.row_ptr[base + t]) * kStepCost[waves[t]];
          for (int first = 0; first < waves[t];) {
            if (used == 4 || (cur.b >= 0 && cur.b != base + t)) flush();
            int second = 0;
            if (cur.a < 0) cur.a = (int32_t)(base + t);
            else if (cur.a != base + t) cur.b = (int32_t)(base + t), second = 1;
            const int take = std::min(waves[t] - first, 4 - used);
            for (int i = 0; i < take; ++i) cur.desc |= pair_desc_wave(used + i, second, first + i);
            used += take;
            first += take;
          }
        }
        flush();
      }
    int64_t packed_cost = 0;
    for (PairGroup& g : head_groups) {
      g.walked = union_size(L, g.a, g.b);
      packed_cost += g.walked * kStepCost[__builtin_popcount((g.desc >> 4) & 0xFu)];
    }
    if (head_groups.empty() || packed_cost >= plain_cost) continue;
    for (const PairGroup& g : head_groups) {
      packed[g.a] = 1;
      if (g.b >= 0) packed[g.b] = 1;
      groups.push_back(g);
    }
  }
  if (groups.empty()) return;
  emit_pair_tables(L, groups);
  L.packed_faces = true;
  // one launch order for both kinds of workgroup, longest first: a row id, or the complement of a
  // packed workgroup's index (ties: the packed workgroup first)
  L.launch_rows.reserve(L.order.size());
  size_t g = 0;
  for (int32_t r : L.order) {
    if (packed[r]) continue;
    const int64_t len = L.row_ptr[r + 1] - L.row_ptr[r];
    while (g < groups.size() && groups[g].walked >= len) L.launch_rows.push_back(~(int32_t)g++);
    L.launch_rows.push_back(r);
  }
  while (g < groups.size()) L.launch_rows.push_back(~(int32_t)g++);
}

// The XCDs of one card do not run at the same speed (measured: up to 5 % apart in finishing time on
// equal shares), and workgroup ids are bound to XCDs, so a launch dealt out by id alone ends when the
// slowest XCD does.  The entries that hold the last kPoolWork of the launch's work (the shortest
// rows: the order is by descending length) are therefore not bound to ids: workgroups past the
// static part draw them by ticket, and an XCD that is ahead draws more.  The static part is a whole
// number of rounds of the XCD-aware order (8 chunks of 64).
LaunchSplit split_launch(const int64_t* work, int64_t entries) {
  constexpr double kPoolWork = 0.06;
  constexpr int64_t kRound = 8 * 64;
  constexpr int64_t kEntryCost = 3;  // fixed cost of an entry in tile steps (launch, first copies, epilogue)
  LaunchSplit sp;
  sp.static_entries = entries;
  if (entries < kPoolMinItems) return sp;
  double total = 0;
  for (int64_t i = 0; i < entries; ++i) total += (double)(work[i] + kEntryCost);
  double tail = 0;
  int64_t s = entries;
  while (s > 0 && tail + (double)(work[s - 1] + kEntryCost) <= kPoolWork * total) tail += (double)(work[--s] + kEntryCost);
  s = (s + kRound - 1) / kRound * kRound;
  if (s < entries && entries - s < ((int64_t)1 << 30)) {
    sp.static_entries = s;
    sp.pool_entries = (int32_t)(entries - s);
  }
  return sp;
}

namespace {
void build_launch_splits(ca_layout& L) {
  const std::vector<int32_t>& launched = L.packed_faces ? L.launch_rows : L.order;
  const int64_t rows = (int64_t)launched.size();
  std::vector<int64_t> work(rows);
  for (int64_t i = 0; i < rows; ++i) {
    const int32_t e = launched[i];
    work[i] = e < 0 ? L.pair_walk_ptr[~e + 1] - L.pair_walk_ptr[~e] : L.row_ptr[e + 1] - L.row_ptr[e];
  }
  L.split_rows = split_launch(work.data(), rows);
  std::fill(work.begin(), work.end(), L.n);
  L.split_rows_dense = split_launch(work.data(), rows);
  const int64_t pairs = (int64_t)L.pair_rows.size() / 2;
  L.split_pairs = L.split_pairs_dense = LaunchSplit{};
  if (pairs && !L.packed_faces) {
    work.resize(pairs);
    for (int64_t i = 0; i < pairs; ++i) work[i] = L.pair_walk_ptr[i + 1] - L.pair_walk_ptr[i];
    L.split_pairs = split_launch(work.data(), pairs);
    std::fill(work.begin(), work.end(), L.n);
    L.split_pairs_dense = split_launch(work.data(), pairs);
  }
}
}  // namespace

namespace {

// Every entry has one workgroup.
constexpr bool is_a_permutation(int64_t total) {
  bool taken[4200] = {};
  for (int64_t id = 0; id < total; ++id) {
    const int64_t entry = xcd_launch_order(id, total, xcd_chunk(total));
    if (entry < 0 || entry >= total || taken[entry]) return false;
    taken[entry] = true;
  }
  return true;
}
static_assert(is_a_permutation(511) && is_a_permutation(512) && is_a_permutation(577) && is_a_permutation(4095) && is_a_permutation(4097), "");

// Predicted time of a launch in us.  Its workgroups are dealt to the XCDs by id and to the free places of their
// XCD in order, which decides it for launches of a few rounds: one workgroup more than the card holds, or the
// long rows on the XCD that has the first of them, are worth up to half of the time.  A step is 128 keys, or one
// tile of the paired kernel's walk.
struct LaunchCost {
  int per_cu;    // workgroups a CU holds
  double start;  // launch, first copies, epilogue
  double step;   // per workgroup and step, as time of a whole CU that is full
  double walk;   // per step of a workgroup alone on its CU
  double group;  // per workgroup
  double gather; // share by which all granules taken from padded tiles lengthen everything
};

// `walks`: steps of the workgroups of one batch entry in launch order, below zero: no token, returns at once.  A launch that
// cannot take less than `limit` is not followed to its end.
double launch_time(const LaunchCost& c, const std::vector<float>& walks, int64_t batch, double gathered, double limit, int64_t chunk = kXcdChunk) {
  constexpr int64_t kXcds = 8, kXcdCus = 32;
  constexpr int64_t kExact = 6000;  // workgroups; beyond, rounds and XCDs even out
  const int64_t entries = (int64_t)walks.size(), total = entries * batch;
  double sum = 0, active = 0;
  bool uniform = true;
  for (float w : walks) {
    uniform = uniform && w == walks[0];
    if (w < 0) continue;
    sum += w;
    active += 1;
  }
  if (active == 0) return c.start;
  const double share = std::min((double)c.per_cu, std::max(1.0, active * (double)batch / (kXcds * kXcdCus)));  // of them on a CU
  const double slot = c.per_cu == 1 ? c.walk : c.walk + (std::max(c.step * c.per_cu, c.walk) - c.walk) * (share - 1) / (c.per_cu - 1);
  const double longer = 1 + c.gather * gathered;
  const double mean = (slot * sum + c.group * active) * (double)batch / (double)(kXcds * kXcdCus * c.per_cu);
  if (total > kExact) return c.start + longer * (mean + 0.3 * slot * sum / active);
  if (c.start + longer * mean >= limit) return limit;
  if (uniform) {
    const int64_t deepest = (total + kXcds - 1) / kXcds, rounds = (deepest + kXcdCus * c.per_cu - 1) / (kXcdCus * c.per_cu);
    return c.start + longer * (double)rounds * (slot * walks[0] + c.group);
  }
  double end = 0;
  std::vector<double> free_at;  // of the places taken so far; a heap, earliest first, once all are
  const size_t places = (size_t)(kXcdCus * c.per_cu);
  for (int64_t xcd : {0, 7}) {  // the ends of a round of chunks, and even and odd ids; all eight give the same choices
    free_at.clear();
    for (int64_t id = xcd; id < total; id += kXcds) {
      const float w = walks[(size_t)(xcd_launch_order(id, total, chunk) % entries)];
      double t = w < 0 ? 0.1 * slot : slot * w + c.group;
      if (free_at.size() < places) {
        free_at.push_back(t);
        if (free_at.size() == places) std::make_heap(free_at.begin(), free_at.end(), std::greater<double>());
      } else {
        t += free_at[0];
        size_t at = 0;
        for (size_t child = 1; child < places; child = 2 * at + 1) {
          if (child + 1 < places && free_at[child + 1] < free_at[child]) ++child;
          if (free_at[child] >= t) break;
          free_at[at] = free_at[child];
          at = child;
        }
        free_at[at] = t;
      }
      end = std::max(end, t);
    }
  }
  return c.start + longer * end;
}

constexpr double kMergeLaunch = 2.0;   // us: the second launch
constexpr double kMergeByte = 0.6e-6;  // us per byte of the shares, written and read

// Dense calls on closed-up copies: us of two launches (q, k and v at once; the result), us per byte of the four tensors, each read
// and written once, what has to be gained, and the shortest walk (shorter ones wait for launches and first copies).
constexpr double kCloseLaunches = 7.0, kCloseByte = 1 / 5.3e6, kCloseGain = 0.92;
constexpr int64_t kCloseTokens = 2048;

struct WayCost {
  Ways ways;
  int stage_keys, part_queries;
  LaunchCost cost;
};

// Rows are split if that is predicted to take this much of the time.  Measured, whole / split: 3 heads x 15K of head dim 128 250 /
// 218 us, 2 x 12 heads x 20K of head dim 64 1267 / 1142 us, 102 rows 153 / 38 us; of 630 split launches, 1.35 times faster as a whole
// (geometric mean), 14 are 2 to 9 % slower, all but two of kWays8x2 at head dim 64.
// With three waves per SIMD whole rows take 0.68 to 1.05 of what is predicted for them, so that more has to be gained: five of 28
// such launches were 4 to 9 % slower priced as with two waves and with the first limit, none of 23 is now (1.03 to 1.65 times faster).
constexpr double kSplitGain = 0.9, kSplitGainThree = 0.77;

// What a workgroup of an unsplit launch walks: an entry of its launch order and a part of the row's query slots.
struct Unit {
  int32_t entry, part;
  int64_t tiles;  // of its list; 0: no token, or no key
};

// Splits the units of a launch (of one batch entry) along the keys for the kernel `ways` (kWaysNone: the one-tile or paired kernel)
// of workgroups of `waves` 32-query waves, and takes the best such plan into `plan` (and its time into `best`) if it is predicted to
// take less than `best`.  step_of: steps of 128 keys of so many tiles.
template <class StepOf>
void plan_split(const ca_layout& L, const std::vector<Unit>& units, Ways ways, int waves, const LaunchCost& cost, double gathered, StepOf step_of, double& best,
                SplitPlan& plan) {
  const int64_t batch = L.prob.batch, bytes = batch * share_bytes(32 * waves, L.prob.head_dim);
  double steps = 0;
  int64_t longest = 0;
  for (const Unit& u : units) {
    steps += step_of(u.tiles) * (double)batch;
    longest = std::max(longest, u.tiles);
  }
  if ((int64_t)units.size() > kMaxSplitItems || longest < 2) return;
  // what leaving a share costs its workgroup: with one to a CU nothing runs meanwhile
  const double share_steps = ways == kWaysNone ? 0.0 : cost.per_cu == 1 ? 2.0 : 1.0;
  const double places = 256.0 * cost.per_cu, tiles_of_step = (double)longest / step_of(longest), per_place = steps / places;
  const double full_step = (1 + cost.gather * gathered) * std::max(cost.step * cost.per_cu, cost.walk), full_group = (1 + cost.gather * gathered) * cost.group / places;
  if (kMergeLaunch + cost.start + full_step * per_place >= best) return;

  // How a launch is cut: no item of more than `limit` tiles (a share of what a place has to do in all, two steps at least),
  // and the last rows, those with `tail` of the work, into items of `small` tiles, which even out what the others leave.
  struct Cut {
    int64_t limit, small;
    double tail;
  } taken{0, 0, 0};
  auto for_pieces = [&](const Cut& cut, auto&& visit) {  // visit(unit, pieces)
    double seen = 0;
    for (const Unit& u : units) {
      const int64_t most = seen < (1 - cut.tail) * steps ? cut.limit : cut.small;
      seen += step_of(u.tiles) * (double)batch;
      visit(u, std::max<int64_t>(1, (u.tiles + most - 1) / most));
    }
  };
  auto tiles_of = [&](double share) { return std::max((int64_t)std::ceil(std::max(share * per_place, 2.0) * tiles_of_step), (int64_t)1); };
  std::vector<int32_t> whole, shared;  // items of so many tiles
  std::vector<float> walks;
  std::vector<std::pair<int64_t, int64_t>> tried;
  for (double tail : {0.0, 0.12, 0.3}) {
    for (double share : {1.1, 0.6, 0.4, 0.25}) {
      const Cut cut{tiles_of(share), tail > 0 ? std::min(tiles_of(share), tiles_of(0.12)) : tiles_of(share), tail};
      int64_t items = 0, shares = 0, splits = 0;
      for_pieces(cut, [&](const Unit&, int64_t pieces) {
        items += pieces;
        if (pieces > 1) shares += pieces, ++splits;
      });
      if (splits == 0 || items > kMaxSplitItems || shares * bytes > kMaxShareBytes) continue;
      if (std::find(tried.begin(), tried.end(), std::make_pair(items, splits)) != tried.end()) continue;
      tried.push_back({items, splits});
      const double room = best - kMergeLaunch - (double)(shares * bytes) * kMergeByte;
      if (cost.start + full_step * (per_place + share_steps * (double)(shares * batch) / places) + full_group * (double)(items * batch) >= room) continue;
      whole.assign((size_t)longest + 1, 0);
      shared.assign((size_t)longest + 1, 0);
      for_pieces(cut, [&](const Unit& u, int64_t pieces) {  // the sizes differ by one at most
        (pieces > 1 ? shared : whole)[(size_t)(u.tiles / pieces)] += (int32_t)(pieces - u.tiles % pieces);
        if (u.tiles % pieces) (pieces > 1 ? shared : whole)[(size_t)(u.tiles / pieces + 1)] += (int32_t)(u.tiles % pieces);
      });
      walks.clear();
      for (int64_t t = longest; t >= 0; --t) {
        const double w = t ? step_of(t) : 0;
        walks.insert(walks.end(), (size_t)whole[(size_t)t], t ? (float)w : -1.f);
        walks.insert(walks.end(), (size_t)shared[(size_t)t], (float)(w + share_steps));
      }
      const double t = launch_time(cost, walks, batch, gathered, room, kXcdSplitChunk);
      if (t < room) {
        best -= room - t;
        taken = cut;
      }
    }
  }
  if (taken.limit == 0) return;
  plan = SplitPlan{};
  plan.ways = ways;
  plan.waves = waves;
  for_pieces(taken, [&](const Unit& u, int64_t pieces) {
    if (pieces > 1) plan.merges.push_back({u.entry, u.part, plan.shares, (int32_t)pieces});
    for (int64_t k = 0; k < pieces; ++k) {
      const int64_t first = u.tiles * k / pieces, end = u.tiles * (k + 1) / pieces;
      const int32_t share_id = pieces > 1 ? ++plan.shares : 0;
      plan.items.push_back({u.entry, (int32_t)first, (int32_t)(end - first), u.part | share_id << 2});
    }
  });
  // longest first; of equal ones, those that read the same keys together (xcd_launch_order keeps neighbours on one XCD)
  auto head_of = [&](int64_t e) { return (e < 0 ? L.pair_rows[2 * ~e] : e) / L.n; };
  std::stable_sort(plan.items.begin(), plan.items.end(), [&](const WorkItem& x, const WorkItem& y) {
    if (x.count != y.count) return x.count > y.count;
    const int64_t hx = head_of(x.entry), hy = head_of(y.entry);
    return hx != hy ? hx < hy : x.first < y.first;
  });
}

}  // namespace

// 16-token granules of an average kept tile (first) and the part of them that lies in padded tiles (second).  Rows
// are sampled where they keep more than `max_words` tiles: every `stride`-th, and a stride without a common factor
// with the tiles of a head or of an axis, so that all columns and faces of the grid have their turn.
std::pair<double, double> granules_per_tile(const ca_layout& L, bool dense, int64_t max_words) {
  const int64_t rows = (int64_t)L.prob.num_heads * L.n;
  std::vector<int> granules(L.class_mask.size());
  for (size_t c = 0; c < granules.size(); ++c) {
    int tokens = 0;
    for (uint32_t w : L.class_mask[c].w) tokens += __builtin_popcount(w);
    granules[c] = (tokens + 15) / 16;
  }
  int64_t tiles = 0, all = 0, padded = 0;
  auto add = [&](int64_t tile) {
    const int32_t c = L.tile_class[tile];
    ++tiles;
    all += granules[c];
    if (c != 0) padded += granules[c];
  };
  if (dense) {
    for (int64_t t = 0; t < L.n; ++t) add(t);
  } else if (granules.size() == 1) {
    return {(double)granules[0], 0.0};
  } else {
    auto gcd = [](int64_t a, int64_t b) {
      while (b) std::swap(a %= b, b);
      return a;
    };
    int64_t stride = 1 + (int64_t)L.col_idx.size() / max_words;
    while (stride > 1 && (gcd(stride, L.n) > 1 || gcd(stride, L.nW) > 1 || gcd(stride, L.nH) > 1)) ++stride;
    for (int64_t r = 0; r < rows; r += stride)
      for (int64_t i = L.row_ptr[r]; i < L.row_ptr[r + 1]; ++i) add(L.col_idx[i]);
  }
  return {tiles ? (double)all / (double)tiles : 0.0, all ? (double)padded / (double)all : 0.0};
}

// Which kernel serves the sparse (or the dense) walk: the one with the shortest predicted time, the
// one-tile and paired kernels unless another is at least 13 % better.
// The constants are a fit of log time over 480 launches of under 3 TFLOP (1-40 heads, grids of 1-64 x 8-60 x 8-104,
// masks from 5 % to dense, all entry points), per kernel, tile size and head dim; residual 5-11 %, 14-16 % for
// kWays8x2 on 128-token tiles.  On 160 other launches of that kind the choice is 1.19 times faster than the one-tile and
// paired kernels (geometric mean; 1.22 is the best choice in hindsight), on 100 of 3 to 40 TFLOP 1.04 (1.04), and
// none of these is slower; of the 480 one is, by 3 %.  A model of the sums and the longest walk alone (residual
// 10-18 %), from a predicted 10 % on, made twelve of the 480 slower by up to 25 %, eleven of them launches of one to
// three rounds of workgroups.
Ways choose_ways(const ca_layout& L, bool dense, int64_t max_words, SplitPlan* plan, double* predicted_us) {
  if (plan) *plan = SplitPlan{};
  if (predicted_us) *predicted_us = HUGE_VAL;  // not priced
  const ca_problem& p = L.prob;
  if (p.dtype != CA_BF16 || (L.B != 64 && L.B != 128) || (p.head_dim != 64 && p.head_dim != 128) || L.class_mask.size() > 8) return kWaysNone;
  // 32-bit lane offsets inside a tile of the natural order; a grid dimension of fewer than 2^32 threads
  if ((int64_t)p.tt * p.H * p.W * p.head_dim * 2 >= (int64_t)1 << 31) return kWaysNone;
  if ((int64_t)p.batch * p.num_heads * L.n * 2 * 512 >= (int64_t)1 << 32) return kWaysNone;
  static const LaunchCost kPlain[2][2] = {{{4, 2.99, 0.57, 1.89, 0.65, 0}, {2, 2.35, 0.93, 1.54, 3.25, 0}},
                                          {{2, 0.0, 0.76, 1.27, 5.74, 0}, {2, 0.0, 1.39, 2.17, 6.5, 0}}};
  static const WayCost k64x64[] = {{kWays8x2, 128, 64, {2, 2.15, 0.84, 1.37, 4.47, 0.09}}};
  static const WayCost k64x128[] = {{kWays4x4, 64, 128, {4, 0.0, 0.87, 2.27, 7.13, 0.03}}, {kWays8x2, 128, 64, {2, 0.0, 0.8, 1.28, 6.65, 0.1}}};
  static const WayCost k128x64[] = {{kWays8x2, 128, 64, {1, 1.76, 1.43, 1.79, 6.68, 0.14}}};
  static const WayCost k128x128[] = {{kWays4x4, 64, 128, {2, 0.0, 1.62, 2.81, 6.9, 0.15}},
                                     {kWays8x4, 128, 128, {1, 0.28, 1.35, 2.0, 8.95, 0.08}},
                                     {kWays8x2, 128, 64, {1, 0.0, 1.35, 1.79, 7.9, 0.18}}};
  const bool big_d = p.head_dim == 128, big_b = L.B == 128;
  const WayCost* options = big_d ? (big_b ? k128x128 : k128x64) : (big_b ? k64x128 : k64x64);
  const int count = big_b ? (big_d ? 3 : 2) : 1;

  // the workgroups of the one-tile and paired kernels
  const std::vector<int32_t>& launched = L.packed_faces ? L.launch_rows : L.order;
  const bool paired = !L.pair_rows.empty() && !L.packed_faces;
  const int64_t plain_groups = paired ? (int64_t)L.pair_rows.size() / 2 : (int64_t)launched.size();
  std::vector<float> walks;
  walks.reserve((size_t)std::max(plain_groups, (int64_t)L.order.size() * 2));
  for (int64_t i = 0; i < plain_groups; ++i) {
    const int64_t e = paired ? ~i : launched[i];
    const int64_t tiles = dense ? L.n : e < 0 ? L.pair_walk_ptr[~e + 1] - L.pair_walk_ptr[~e] : L.row_ptr[e + 1] - L.row_ptr[e];
    walks.push_back(paired ? (float)tiles : (float)(tiles * L.B) / 128);
  }
  constexpr double kPlainBias = 0.87;
  double best = kPlainBias * launch_time(kPlain[big_d][big_b], walks, p.batch, 0, HUGE_VAL);
  Ways ways = kWaysNone;

  // the workgroups of the others: every part of every row
  std::vector<int> tokens(L.class_mask.size());
  for (size_t c = 0; c < tokens.size(); ++c)
    for (uint32_t w : L.class_mask[c].w) tokens[c] += __builtin_popcount(w);
  const auto [per_tile, padded] = granules_per_tile(L, dense, max_words);
  for (int i = 0; i < count; ++i) {
    const WayCost& w = options[i];
    const int parts = (int)L.B / w.part_queries;
    const double stage = w.stage_keys / 16;  // in granules
    walks.clear();
    for (int64_t j = 0; j < (int64_t)L.order.size(); ++j) {
      const int64_t r = dense ? j : L.order[j];
      const int64_t tiles = dense ? L.n : L.row_ptr[r + 1] - L.row_ptr[r];
      const float steps = (float)(std::ceil((double)tiles * per_tile / stage) * stage / 8);
      const int held = (tokens[L.tile_class[r % L.n]] + w.part_queries - 1) / w.part_queries;  // parts with a token
      for (int part = 0; part < parts; ++part) walks.push_back(part < held ? steps : -1.f);
    }
    const double t = launch_time(w.cost, walks, p.batch, padded, best);
    if (t < best) best = t, ways = w.ways;
  }
  if (predicted_us) *predicted_us = ways == kWaysNone ? best / kPlainBias : best;
  if (plan && std::min(plain_groups, (int64_t)L.order.size()) <= kMaxSplitItems) {
    if (ways == kWaysNone) best /= kPlainBias;
    // Rows of 64-token tiles of head dim 64 run with three waves per SIMD where choose_simd_waves says so, and so do their items,
    // which no other kernel is tried for (kWays8x2, the one that was predicted to gain there, did not).
    static const LaunchCost kThreeWaves{6, 2.99, 0.54, 1.89, 0.65, 0};
    const bool three_waves = ways == kWaysNone && !big_d && !big_b && (dense ? L.simd_waves_dense : L.simd_waves) == 3;
    const LaunchCost& plain = three_waves ? kThreeWaves : kPlain[big_d][big_b];
    if (three_waves) {
      walks.clear();
      for (int64_t i = 0; i < plain_groups; ++i) walks.push_back((float)((dense ? L.n : L.row_ptr[launched[i] + 1] - L.row_ptr[launched[i]]) * L.B) / 128);
      best = launch_time(plain, walks, p.batch, 0, HUGE_VAL);
    }
    best *= three_waves ? kSplitGainThree : kSplitGain;
    std::vector<Unit> units;
    for (int64_t i = 0; i < plain_groups; ++i) {
      const int64_t e = paired ? ~i : dense && !L.packed_faces ? i : launched[i];
      units.push_back({(int32_t)e, 0, dense ? L.n : e < 0 ? L.pair_walk_ptr[~e + 1] - L.pair_walk_ptr[~e] : L.row_ptr[e + 1] - L.row_ptr[e]});
    }
    // only in the place of themselves: they multiply the padding slots of K and V too (by zero), the others never read them
    const auto walk = [&](int64_t tiles) { return paired ? (double)tiles : (double)(tiles * L.B) / 128; };
    if (ways == kWaysNone) plan_split(L, units, kWaysNone, paired ? 4 : (int)L.B / 32, plain, 0, walk, best, *plan);
    for (int i = 0; i < (three_waves ? 0 : count); ++i) {
      const WayCost& w = options[i];
      const int parts = (int)L.B / w.part_queries;
      const double stage = w.stage_keys / 16;
      units.clear();
      for (int64_t j = 0; j < (int64_t)L.order.size(); ++j) {
        const int64_t r = dense ? j : L.order[j];
        const int held = (tokens[L.tile_class[r % L.n]] + w.part_queries - 1) / w.part_queries;
        for (int part = 0; part < parts; ++part) units.push_back({(int32_t)r, part, part >= held ? 0 : dense ? L.n : L.row_ptr[r + 1] - L.row_ptr[r]});
      }
      plan_split(L, units, w.ways, w.part_queries / 32, w.cost, padded, [&](int64_t tiles) { return std::ceil((double)tiles * per_tile / stage) * stage / 8; }, best, *plan);
    }
    if (predicted_us && plan->shares > 0) *predicted_us = best;
  }
  return ways;
}

// Kernel of fp32 calls that bring a workspace: the one of attn_f32_planes.hip with the shortest predicted time, or attn_f32.hip,
// unless the former is predicted to be at least 13 % better.  Tiles of at most 32 tokens, which leave 32 queries of a wave
// without work, stay with attn_f32.hip (16 tokens: 1.25 times faster to 2.5 times slower).
// The constants are a fit over 276 launches of under 0.1 TFLOP (1-40 heads, head dims 32-128, tiles of 60-128 tokens, masks from 5 %
// to dense), per kernel and head dim, a step being 128 keys; residual 5-16 %.  On these the choice is 1.36 times faster than
// attn_f32.hip (geometric mean; 1.41 is the best choice in hindsight), and four of them, calls of one head, are slower, by up to 8 %.
// Without the 13 % ten are slower, by up to 20 %.  They were taken with launches dealt in chunks of kXcdChunk, as launch_time has
// them; the kernels' own order (xcd_chunk) and the rounding of the parts came later, and made launches of 512 to 4095 workgroups up to 1.25 times as fast.
Ways choose_planes(const ca_layout& L, bool dense, int64_t max_words) {
  const ca_problem& p = L.prob;
  if (p.dtype != CA_F32 || L.B <= 32 || L.B > 128 || (p.head_dim != 32 && p.head_dim != 64 && p.head_dim != 128) || L.class_mask.size() > 8) return kWaysNone;
  if (plane_bytes((int64_t)p.batch * p.num_heads, L.n, L.B, p.head_dim) > kMaxPlaneBytes) return kWaysNone;
  struct PlaneCost {
    Ways planes;
    int part_queries;
    LaunchCost cost;
    double split;  // us per million elements of K, to split K and V
  };
  static const PlaneCost kOptions[3][3] = {
      {{kPlanes2x2, 64, {4, 7.4, 1.08, 2.97, 1.0, 0}, 9.3}, {kPlanes2x4, 64, {2, 7.8, 1.26, 2.14, 1.0, 0}, 10.5}, {kPlanes1x4, 32, {3, 7.2, 0.73, 1.61, 1.0, 0}, 12.3}},
      {{kPlanes2x2, 64, {3, 5.6, 1.85, 3.81, 4.34, 0}, 6.6}, {kPlanes2x4, 64, {1, 7.6, 0, 2.76, 3.23, 0}, 7.9}},
      {{kPlanes2x2, 64, {2, 12.0, 4.09, 6.18, 1.0, 0}, 6.3}, {kPlanes2x4, 64, {1, 6.7, 0, 4.76, 7.67, 0}, 6.4}, {kPlanes1x4, 32, {1, 7.9, 0, 4.18, 1.02, 0}, 14.7}}};
  // attn_f32.hip with 16, 32 and 64 queries to a workgroup (the split of 64 at head dim 128 is that of 32 with twice the work)
  static const LaunchCost kF32[3][3] = {{{2, 5.5, 0.69, 1.86, 0.5, 0}, {2, 4.4, 0.46, 2.66, 6.0, 0}, {2, 27.0, 2.12, 3.53, 5.2, 0}},
                                        {{2, 1.0, 0.79, 2.9, 4.2, 0}, {2, 27.0, 2.78, 3.83, 0.5, 0}, {2, 30.0, 4.02, 4.0, 16.0, 0}},
                                        {{2, 1.0, 5.11, 6.92, 7.2, 0}, {2, 1.0, 5.11, 6.92, 7.2, 0}, {2, 1.0, 10.2, 13.8, 14.0, 0}}};
  constexpr double kF32Bias = 0.87;
  const int d = p.head_dim == 32 ? 0 : p.head_dim == 64 ? 1 : 2;
  std::vector<int> tokens(L.class_mask.size());
  for (size_t c = 0; c < tokens.size(); ++c)
    for (uint32_t w : L.class_mask[c].w) tokens[c] += __builtin_popcount(w);
  const double per_tile = granules_per_tile(L, dense, max_words).first;
  std::vector<float> walks;
  auto cut = [&](int part_queries) {  // the workgroups of a launch
    const int parts = (int)(L.B + part_queries - 1) / part_queries;
    walks.clear();
    for (int64_t j = 0; j < (int64_t)L.order.size(); ++j) {
      const int64_t r = dense ? j : L.order[j];
      const float steps = (float)((double)(dense ? L.n : L.row_ptr[r + 1] - L.row_ptr[r]) * per_tile / 8);
      const int held = (tokens[L.tile_class[r % L.n]] + part_queries - 1) / part_queries;
      for (int part = 0; part < parts; ++part) walks.push_back(part < held ? steps : -1.f);
    }
  };
  const int qw = f32_query_groups((int64_t)p.batch * p.num_heads * L.n, L.B, p.head_dim);
  cut(16 * qw);
  double best = kF32Bias * launch_time(kF32[d][qw / 2], walks, p.batch, 0, HUGE_VAL);
  Ways planes = kWaysNone;
  const double elements = 1e-6 * (double)plane_bytes((int64_t)p.batch * p.num_heads, L.n, L.B, p.head_dim) / 12;
  for (const PlaneCost& o : kOptions[d]) {
    if (o.planes == kWaysNone) continue;  // 1x4 at head dim 64: never the best by more than a few per cent
    cut(o.part_queries);
    const double t = o.split * elements + launch_time(o.cost, walks, p.batch, 0, HUGE_VAL);
    if (t < best) best = t, planes = o.planes;
  }
  return planes;
}

namespace {

// Waves per SIMD of the one-tile kernel for 64-token tiles of head dim 64: 2, or 3.  The third makes a full card
// 1.07 times faster, but a workgroup then has a third of its SIMDs, so a launch that ends with its longest
// rows loses.  Greedy assignment of the rows to the slots of the card says which it is; the third wave is
// taken from a 1.05 times shorter makespan on.  Measured, makespans with 2 / 3 waves and times: 1536 rows of 128
// tiles 256 / 128 tiles, 299 / 240 us; 1536 rows of 86 on average 140 / 128, 221 / 209 us; 2048 rows of 128 256 / 256,
// 337 / 361 us; 1792 rows of 68 on average 128 / 128, 172 / 178 us; 10K rows 4.44 / 4.13 ms.
int choose_simd_waves(const ca_layout& L, bool dense) {
  if (L.prob.dtype != CA_BF16 || L.B != 64 || L.prob.head_dim != 64) return 2;
  const int64_t rows = (int64_t)L.order.size(), items = rows * L.prob.batch;
  if (items > 4096) return 3;
  auto makespan = [&](size_t slots) {
    if (dense) return (double)((items + (int64_t)slots - 1) / (int64_t)slots * L.n);  // all walks are equal
    std::priority_queue<int64_t, std::vector<int64_t>, std::greater<int64_t>> free_at;
    int64_t end = 0;
    for (int64_t i = 0; i < items; ++i) {  // in launch order: batch entry after batch entry
      const int64_t r = L.order[i % rows];
      int64_t t = L.row_ptr[r + 1] - L.row_ptr[r];
      if (free_at.size() >= slots) {
        t += free_at.top();
        free_at.pop();
      }
      free_at.push(t);
      end = std::max(end, t);
    }
    return (double)end;
  };
  constexpr size_t kSlots = 512;  // per wave of a SIMD: 256 CUs of four SIMDs, two waves to a workgroup
  return makespan(2 * kSlots) >= 1.05 * makespan(3 * kSlots) ? 3 : 2;
}

}  // namespace

namespace {

// Sets L.closed, if dense calls are predicted to be faster there.  `dense_us`: what they take as they are.
// A padded grid multiplies its padding in queries and keys (13 x 30 x 52 tokens in 1 x 8 x 8 tiles: 32 % more products), and the
// kernel for 128-token tiles beats those for 64 also where nothing is padded.  Measured with the copies: 16 heads x 20K in 64-token
// tiles 4.09 / 3.10 ms (copies 0.11); 18 heads x 44K of a grid filled to 0.79 23.5 / 15.5 ms; 8 heads x 8K without padding 259 /
// 247 us.  Over 50 launches of 11 us to 24 ms, each way measured on its own and the time of the copies added to one, what is chosen is 1.18
// times as fast (geometric mean; 1.20 is the best choice in hindsight), one launch 3 % slower.
void close_dense(ca_layout& L, double dense_us) {
  const ca_problem& p = L.prob;
  const bool padded = L.class_mask.size() > 1;
  if (p.dtype != CA_BF16 || (L.B != 64 && L.B != 128) || (p.head_dim != 64 && p.head_dim != 128) || (!padded && L.B == 128)) return;
  if (!std::isfinite(dense_us) || L.N_real < kCloseTokens || L.N_real >= ((int64_t)1 << 31) - 128) return;
  const bool in_place = !padded && L.N_pad % 128 == 0;
  const double bytes = (double)p.batch * p.num_heads * (double)L.N_real * p.head_dim * 2;
  const double copies = in_place ? 0 : kCloseLaunches + 8 * bytes * kCloseByte;
  const double fill = (double)L.N_real / (double)L.N_pad;
  if (kCloseGain * dense_us - copies < 0.5 * fill * fill * dense_us) return;  // not even if closing did more than it ever does
  auto c = std::make_unique<ca_layout>();
  c->is_closed = true;
  c->prob = p;
  c->prob.T = c->prob.H = c->prob.tt = c->prob.th = 1;
  c->prob.W = (int32_t)L.N_real;
  c->prob.tw = 128;
  c->prob.n_text = 0;
  c->B = 128;
  c->nT = c->nH = 1;
  c->n = c->n_vid = (L.N_real + 127) / 128;
  c->nW = (int32_t)c->n;
  c->N_real = L.N_real;
  c->N_pad = c->n * 128;
  c->scale = L.scale;
  if (!in_place && 4 * tensor_bytes(*c) > kMaxPlaneBytes) return;
  c->row_ptr.assign((size_t)p.num_heads * (size_t)c->n + 1, 0);
  finish_host_tables(*c);
  if (!(c->closed_us + copies <= kCloseGain * dense_us)) return;
  L.closed_in_place = in_place;
  L.closed = std::move(c);
}

}  // namespace

void finish_host_tables(ca_layout& L) {
  const int32_t Hd = L.prob.num_heads;
  // per-head relative offsets for the C-ABI view
  L.head_row_ptr.assign(Hd, std::vector<int64_t>());
  for (int32_t h = 0; h < Hd; ++h) {
    L.head_row_ptr[h].resize(L.n + 1);
    const int64_t base = L.row_ptr[(int64_t)h * L.n];
    for (int64_t q = 0; q <= L.n; ++q) L.head_row_ptr[h][q] = L.row_ptr[(int64_t)h * L.n + q] - base;
  }
  build_order(L);
  build_slot_masks(L);
  L.pair_rows.clear();
  L.pair_desc.clear();
  L.pair_walk_ptr.clear();
  L.pair_walk.clear();
  L.packed_faces = false;
  L.launch_rows.clear();
  if (L.prob.dtype == CA_BF16 && L.B == 64 && L.prob.head_dim == 128) build_pair_table(L);
  if (L.prob.dtype == CA_BF16 && L.B == 128 && L.prob.head_dim == 128) build_packed_faces(L);
  build_launch_splits(L);
  L.simd_waves = choose_simd_waves(L, false);
  L.simd_waves_dense = choose_simd_waves(L, true);
  L.ways = L.is_closed ? kWaysNone : choose_ways(L, false, kSampledWords, &L.split);
  double dense_us = HUGE_VAL;
  L.ways_dense = choose_ways(L, true, kSampledWords, &L.split_dense, &dense_us);
  L.closed_us = dense_us;
  L.closed.reset();
  if (!L.is_closed) close_dense(L, dense_us);
  L.planes = choose_planes(L, false, kSampledWords);
  L.planes_dense = choose_planes(L, true, kSampledWords);
}

int import_host_tables(ca_layout& L, const int64_t* const* row_ptr, const int32_t* const* col_idx) {
  const int32_t Hd = L.prob.num_heads;
  for (int32_t h = 0; h < Hd; ++h) {
    if (!row_ptr[h] || (!col_idx[h] && row_ptr[h][L.n] != 0)) {
      set_error("head %d: null CSR array", h);
      return CA_ERR_INVALID_ARG;
    }
    if (row_ptr[h][0] != 0) {
      set_error("head %d: row_ptr[0] must be 0", h);
      return CA_ERR_INVALID_ARG;
    }
    for (int64_t q = 0; q < L.n; ++q) {
      const int64_t b = row_ptr[h][q], e = row_ptr[h][q + 1];
      if (e < b || e - b > L.n) {
        set_error("head %d: row %lld has an invalid extent", h, (long long)q);
        return CA_ERR_INVALID_ARG;
      }
      for (int64_t i = b; i < e; ++i) {
        const int32_t c = col_idx[h][i];
        if (c < 0 || c >= L.n || (i > b && c <= col_idx[h][i - 1])) {
          set_error("head %d: row %lld must list tile ids in [0, n) in strictly ascending order", h, (long long)q);
          return CA_ERR_INVALID_ARG;
        }
      }
    }
  }
  try {
    const int64_t rows = (int64_t)Hd * L.n;
    L.row_ptr.assign(rows + 1, 0);
    int64_t total = 0;
    for (int32_t h = 0; h < Hd; ++h) {
      for (int64_t q = 0; q < L.n; ++q) L.row_ptr[(int64_t)h * L.n + q] = total + row_ptr[h][q];
      total += row_ptr[h][L.n];
    }
    L.row_ptr[rows] = total;
    L.col_idx.resize(total);
    for (int32_t h = 0; h < Hd; ++h) {
      const int64_t cnt = row_ptr[h][L.n];
      if (cnt) std::memcpy(L.col_idx.data() + L.row_ptr[(int64_t)h * L.n], col_idx[h], cnt * sizeof(int32_t));
    }
    finish_host_tables(L);
  } catch (const std::bad_alloc&) {
    set_error("out of host memory while importing the layout");
    return CA_ERR_ALLOC;
  }
  return CA_OK;
}

int union_host_tables(ca_layout& L, const ca_layout& a, const ca_layout& b) {
  try {
    const int64_t rows = (int64_t)L.prob.num_heads * L.n;
    L.row_ptr.assign(rows + 1, 0);
    L.col_idx.clear();
    L.col_idx.reserve(std::max(a.col_idx.size(), b.col_idx.size()));
    for (int64_t r = 0; r < rows; ++r) {
      const int32_t *pa = a.col_idx.data() + a.row_ptr[r], *ea = a.col_idx.data() + a.row_ptr[r + 1];
      const int32_t *pb = b.col_idx.data() + b.row_ptr[r], *eb = b.col_idx.data() + b.row_ptr[r + 1];
      while (pa < ea || pb < eb) {  // merge of two ascending lists without duplicates
        if (pb == eb || (pa < ea && *pa < *pb)) L.col_idx.push_back(*pa++);
        else if (pa == ea || *pb < *pa) L.col_idx.push_back(*pb++);
        else { L.col_idx.push_back(*pa++); ++pb; }
      }
      L.row_ptr[r + 1] = (int64_t)L.col_idx.size();
    }
    finish_host_tables(L);
  } catch (const std::bad_alloc&) {
    set_error("out of host memory while merging the layouts");
    return CA_ERR_ALLOC;
  }
  return CA_OK;
}

double head_similarity(const ca_layout& a, int32_t ha, const ca_layout& b, int32_t hb) {
  int64_t both = 0, either = 0;
  for (int64_t q = 0; q < a.n; ++q) {
    const int64_t ra = (int64_t)ha * a.n + q, rb = (int64_t)hb * b.n + q;
    const int32_t *pa = a.col_idx.data() + a.row_ptr[ra], *ea = a.col_idx.data() + a.row_ptr[ra + 1];
    const int32_t *pb = b.col_idx.data() + b.row_ptr[rb], *eb = b.col_idx.data() + b.row_ptr[rb + 1];
    while (pa < ea && pb < eb) {
      if (*pa < *pb) ++pa;
      else if (*pb < *pa) ++pb;
      else { ++both; ++pa; ++pb; }
    }
    either += (a.row_ptr[ra + 1] - a.row_ptr[ra]) + (b.row_ptr[rb + 1] - b.row_ptr[rb]);
  }
  either -= both;
  return either == 0 ? 1.0 : (double)both / (double)either;
}

int build_host_tables(ca_layout& L, const ca_head* heads) {
  const ca_problem& p = L.prob;
  const int32_t Hd = p.num_heads;
  std::vector<HeadPlan> plans(Hd);
  for (int32_t h = 0; h < Hd; ++h) {
    const int st = plan_head(heads[h], h, L.nT, plans[h]);
    if (st != CA_OK) return st;
  }
  try {
    const int64_t rows = (int64_t)Hd * L.n;
    L.row_ptr.assign(rows + 1, 0);
    // pass 1: row lengths
    for (int32_t h = 0; h < Hd; ++h)
      for (int64_t q = 0; q < L.n; ++q) {
        int64_t cnt;
        if (q >= L.n_vid) {
          cnt = L.n;  // text query tile keeps everything
        } else {
          const int32_t qw = (int32_t)(q % L.nW), qh = (int32_t)((q / L.nW) % L.nH), qt = (int32_t)(q / ((int64_t)L.nW * L.nH));
          cnt = L.n_txt;
          for_each_run(L, plans[h], qt, qh, qw, [&](int32_t, int32_t len) { cnt += len; });
        }
        L.row_ptr[(int64_t)h * L.n + q + 1] = cnt;
      }
    for (int64_t r = 0; r < rows; ++r) L.row_ptr[r + 1] += L.row_ptr[r];
    // pass 2: column ids
    L.col_idx.resize(L.row_ptr[rows]);
    for (int32_t h = 0; h < Hd; ++h)
      for (int64_t q = 0; q < L.n; ++q) {
        int32_t* dst = L.col_idx.data() + L.row_ptr[(int64_t)h * L.n + q];
        if (q >= L.n_vid) {
          for (int64_t k = 0; k < L.n; ++k) *dst++ = (int32_t)k;
          continue;
        }
        const int32_t qw = (int32_t)(q % L.nW), qh = (int32_t)((q / L.nW) % L.nH), qt = (int32_t)(q / ((int64_t)L.nW * L.nH));
        for_each_run(L, plans[h], qt, qh, qw, [&](int32_t first, int32_t len) {
          for (int32_t i = 0; i < len; ++i) *dst++ = first + i;
        });
        for (int64_t k = L.n_vid; k < L.n; ++k) *dst++ = (int32_t)k;
      }
    finish_host_tables(L);
  } catch (const std::bad_alloc&) {
    set_error("out of host memory while building the layout");
    return CA_ERR_ALLOC;
  }
  return CA_OK;
}

// The kernels read one packed word per kept tile: tile id | padding class << 24, and bit 31 set
// when the upper half of the tile's slots is padding only (such a tile costs half the products).
// `forward_only` leaves out what only the dense and the natural-order walks read.
int pack_device_tables(const ca_layout& layout, bool forward_only, PackedTables& t) {
  const ca_layout* L = &layout;
  if (L->n >= (int64_t)1 << 24 || L->class_mask.size() > 127) {
    set_error("layout too large for the device tables (%lld tiles, %zu padding classes)", (long long)L->n,
              L->class_mask.size());
    return CA_ERR_UNSUPPORTED;
  }
  try {
    std::vector<uint32_t> class_word(L->class_mask.size());
    const int words = L->B <= 128 ? (int)((L->B + 31) / 32) : 0;  // a mask holds no more
    for (size_t c = 0; c < class_word.size(); ++c) {
      bool upper_empty = words >= 2;
      for (int w = words / 2; w < words; ++w) upper_empty = upper_empty && L->class_mask[c].w[w] == 0;
      class_word[c] = ((uint32_t)c << 24) | (upper_empty ? 0x80000000u : 0u);
    }
    // Query slots of a tile in the order the bf16 kernels hand them to lanes: the slots that hold a
    // token first, so that the queries of a padded tile fill as few 32-query waves as possible.
    t.class_perm.assign(L->class_mask.size() * 128, 0);
    for (size_t c = 0; c < L->class_mask.size(); ++c) {
      int at = 0;
      for (int pass = 0; pass < 2; ++pass)
        for (int slot = 0; slot < (int)L->B && slot < 128; ++slot) {
          const bool valid = (L->class_mask[c].w[slot >> 5] >> (slot & 31)) & 1u;
          if (valid == (pass == 0)) t.class_perm[c * 128 + at++] = (uint8_t)slot;
        }
    }
    // two words of padding: the kernels fetch these tables two entries ahead of the one in use
    t.col_meta.assign(L->col_idx.size() + 2, 0);
    for (size_t i = 0; i < L->col_idx.size(); ++i)
      t.col_meta[i] = (int32_t)((uint32_t)L->col_idx[i] | class_word[L->tile_class[L->col_idx[i]]]);
    if (!forward_only) {
      t.dense_meta.assign(L->n + 2, 0);
      for (int64_t i = 0; i < L->n; ++i) t.dense_meta[i] = (int32_t)((uint32_t)i | class_word[L->tile_class[i]]);
      // natural-order row of slot 0 of every tile (kernels that gather tiles from natural order)
      const ca_problem& pr = L->prob;
      const int64_t n_video = (int64_t)pr.T * pr.H * pr.W;
      if (L->N_real < ((int64_t)1 << 31)) {
        t.tile_origin.resize(L->n);
        for (int64_t i = 0; i < L->n; ++i) {
          if (i >= L->n_vid) {
            t.tile_origin[i] = (int32_t)(n_video + (i - L->n_vid) * L->B);
          } else {
            const int64_t kw = i % L->nW, kh = (i / L->nW) % L->nH, kt = i / ((int64_t)L->nW * L->nH);
            t.tile_origin[i] = (int32_t)(((kt * pr.tt) * pr.H + kh * pr.th) * pr.W + kw * pr.tw);
          }
        }
      }
    }
    if (!L->pair_rows.empty()) {
      // walk words of the paired kernel carry the class in bits 24-29, below the two membership bits
      if (L->class_mask.size() > 63) {
        set_error("layout has too many padding classes for the paired kernel (%zu)", L->class_mask.size());
        return CA_ERR_UNSUPPORTED;
      }
      t.pair_walk.assign(L->pair_walk.size() + 2, 0);
      for (size_t i = 0; i < L->pair_walk.size(); ++i) {
        const uint32_t w = (uint32_t)L->pair_walk[i];
        t.pair_walk[i] = (int32_t)(w | ((uint32_t)L->tile_class[w & 0xffffffu] << 24));
      }
      if (!forward_only) {
        t.dense_pair_walk.assign(L->n + 2, 0);
        for (int64_t i = 0; i < L->n; ++i)
          t.dense_pair_walk[i] =
              (int32_t)((uint32_t)i | ((uint32_t)L->tile_class[i] << 24) | ca::kPairInFirst | ca::kPairInSecond);
      }
    }
  } catch (const std::bad_alloc&) {
    set_error("out of host memory while packing the device tables");
    return CA_ERR_ALLOC;
  }
  return CA_OK;
}


}  // namespace ca
