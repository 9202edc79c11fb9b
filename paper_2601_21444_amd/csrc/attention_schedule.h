// Merged heaviest-first order of the query tiles of several attention problems (host side builds it, the
// kernel decodes one entry per workgroup).  Plain C++: no HIP types, so host tests can compile it alone.
//
// Query tile qt (256 rows, or another `tile`) of a problem with n_vis fully visible keys visits about (n_vis + 256 (qt+1))
// / 64 key tiles; its level is n_vis / 256 + qt, so one level is one query tile's worth of keys for every problem.
// Levels are walked from the highest down; inside a level the problems come in index order.  The level axis
// is cut where a problem starts or ends, so inside a segment the set of active problems is fixed and an
// entry index decodes with one division.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define APBV_HOST_DEVICE __host__ __device__
#else
#define APBV_HOST_DEVICE
#endif

namespace apbv {

constexpr int kMaxGroupItems = 8;
constexpr int kGroupQueryTile = 256;     // query rows per workgroup of the attention kernel's main variant

struct GroupSchedule {
  struct Segment {
    int first;        // index of the segment's first (problem, query tile) entry
    int level_hi;     // its highest level; entries walk the levels downwards
    int n_active;     // problems with a query tile on each of the segment's levels
    uint32_t items;   // their indices, 4 bits each, in index order
  } seg[2 * kMaxGroupItems];
  int level0[kMaxGroupItems];   // level of query tile 0 of every problem
  int n_segs, n_entries;
};

// rows[m] >= 1 query rows and n_vis[m] >= 0 fully visible keys of problem m.  False if the sizes do not fit.
inline bool build_group_schedule(int n, const int64_t* n_vis, const int64_t* rows, GroupSchedule& s, int tile = kGroupQueryTile) {
  if (n < 1 || n > kMaxGroupItems) return false;
  int64_t lo[kMaxGroupItems], hi[kMaxGroupItems];      // level range [lo, hi) of every problem
  int64_t cuts[2 * kMaxGroupItems];
  int n_cuts = 0;
  for (int m = 0; m < n; ++m) {
    if (rows[m] < 1 || n_vis[m] < 0) return false;
    lo[m] = n_vis[m] / tile;
    hi[m] = lo[m] + (rows[m] + tile - 1) / tile;
    if (hi[m] > 0x3fffffff) return false;
    s.level0[m] = (int)lo[m];
    cuts[n_cuts++] = lo[m];
    cuts[n_cuts++] = hi[m];
  }
  for (int a = 1; a < n_cuts; ++a)                     // insertion sort, descending
    for (int c = a; c > 0 && cuts[c] > cuts[c - 1]; --c) {
      const int64_t t = cuts[c];
      cuts[c] = cuts[c - 1];
      cuts[c - 1] = t;
    }
  int n_segs = 0;
  int64_t first = 0;
  for (int a = 0; a + 1 < n_cuts; ++a) {
    const int64_t top = cuts[a], bottom = cuts[a + 1];  // levels [bottom, top)
    if (top == bottom) continue;
    uint32_t items = 0;
    int n_active = 0;
    for (int m = 0; m < n; ++m)
      if (lo[m] <= bottom && top <= hi[m]) items |= (uint32_t)m << (4 * n_active++);
    if (n_active == 0) continue;
    GroupSchedule::Segment& sg = s.seg[n_segs++];
    sg.first = (int)first;
    sg.level_hi = (int)(top - 1);
    sg.n_active = n_active;
    sg.items = items;
    first += (top - bottom) * n_active;
    if (first > 0x3fffffff) return false;
  }
  s.n_segs = n_segs;
  s.n_entries = (int)first;
  return true;
}

// Entry index (0 <= entry < n_entries) -> problem m and its query tile qt.
APBV_HOST_DEVICE inline void decode_group_entry(const GroupSchedule& s, int entry, int& m, int& qt) {
  int sg = 0;
  while (sg + 1 < s.n_segs && entry >= s.seg[sg + 1].first) ++sg;
  const int r = entry - s.seg[sg].first;
  const int level = s.seg[sg].level_hi - r / s.seg[sg].n_active;
  m = (int)((s.seg[sg].items >> (4 * (r % s.seg[sg].n_active))) & 15u);
  qt = level - s.level0[m];
}

// Workgroups of the attention kernel that a unit holds at once: of `waves` waves of `own` 16-row blocks each.  By LDS with
// head_dim 128, by registers with 64.
APBV_HOST_DEVICE constexpr int workgroups_per_unit(int head_dim, int waves, int own) {
  return waves == 8 ? 1 : head_dim == 128 ? 2 : own == 1 ? 4 : 3;
}

// Which of an XCD's n work items, numbered heaviest first, its s-th workgroup takes.  Workgroups are dispatched to the 32
// units in turn, so unit j gets numbers j, 32 + j, ... until it holds per_unit of them, and further ones go where one has
// ended.  Items taken in that order (kInTurn) give unit 0 the heaviest of every round and unit 31 the lightest.  So
//   - kFolded: odd rounds run backwards, so that two rounds add up to about the same on every unit.  Where the last round is not
//     full, its units are those with the lightest items of the round before, or, behind two rounds, units that have one item
//     more than the others.  With more items than the units hold only the first rounds are arranged;
//   - kThrees, with two a unit and up to one item more per unit than that (m > 0 of them): the lightest 3 m go to m units, three
//     each, the lightest of them dispatched last.  In turn the units' two workgroups could end together and take two of the last.
constexpr int kUnitsPerXcd = 32;
enum Arrangement { kInTurn, kFolded, kThrees };
APBV_HOST_DEVICE inline int arrange_workgroup(int s, int n, int per_unit, int how) {
  const int round = s / kUnitsPerXcd, unit = s % kUnitsPerXcd;
  if (n <= kUnitsPerXcd || how == kInTurn) return s;
  if (how == kThrees && per_unit == 2 && n > 2 * kUnitsPerXcd && n <= 3 * kUnitsPerXcd) {
    const int m = n - 2 * kUnitsPerXcd, pairs = kUnitsPerXcd - m;        // units with three items, with two
    if (round == 2) return n - m + unit;
    if (unit < pairs) return round == 0 ? unit : 2 * pairs - 1 - unit;
    return round == 0 ? pairs + unit : n - m - 1 - (unit - pairs);
  }
  if (round >= per_unit) return s;
  const int n_now = n < kUnitsPerXcd * per_unit ? n : kUnitsPerXcd * per_unit;
  const int last = (n_now - 1) / kUnitsPerXcd, more = (n_now - 1) % kUnitsPerXcd + 1;    // units with an item of the last round
  const int rank = unit >= more ? unit - more : unit + kUnitsPerXcd - more;
  if (round & 1) return round * kUnitsPerXcd + kUnitsPerXcd - 1 - rank;
  return round * kUnitsPerXcd + (round == last ? unit : rank);
}
// By the number of items, what a unit holds, its rows (tile), whether all are of one problem, and the weights, weight(r) of the
// r-th heaviest.  Which unit is free first is a matter of a few percent of a workgroup's time, and no estimate of it told the
// orders apart, so the lines lie where an order is seldom behind plain order and ahead of it on average.  Drawn from 1540
// launches of two and three a unit, each timed in all three.  Time in turn / as chosen, least and mean:
//   64 rows, head_dim 128    33 to 64 items 0.983, 1.021
//   128 rows, head_dim 128   33 to 64 0.988, 1.028 (always folded 0.927, 1.034)
//                            65 to 128, one problem 0.941, 1.013, and 500 near the lines 0.934, 1.050; several 0.972, 1.024
//                            65 to 96 always folded 0.926, 1.013; threes 0.878, 1.013; more than 128 folded 0.978, 0.996
//   128 rows, head_dim 64    33 to 96 0.985, 1.049 (always folded 0.941, 1.048)    97 to 128 0.974, 1.033 (folded 0.943, 1.030)
//                            more than 128 folded 0.973, 0.994
// Four a unit, the 64-row workgroups of head_dim 64, stay in turn: folded 0.957, 1.002.  us, in turn / folded / threes, the last taken:
// 8 heads of 128 with their own K/V, 8910 rows behind 5000 keys 356 / 341 / 325; 4 x 16 heads x 1160 rows behind 283 56 / 53 / 47; 28
// heads x 2382 behind 1500 116 / 109 / 111.
template <typename Weight>
inline Arrangement arrangement_of(int n, int per_unit, int tile, bool one, Weight&& weight) {
  if (n <= kUnitsPerXcd || n > 4 * kUnitsPerXcd || per_unit == 1 || per_unit == 4) return kInTurn;
  const int64_t heaviest = weight(0), lightest = weight(n - 1);
  if (n <= kUnitsPerXcd * per_unit) return tile == 64 || 2 * lightest < heaviest ? kFolded : kInTurn;
  if (per_unit == 2 && 2 * lightest < heaviest &&
      (one ? n > 68 && n < 96 && 4 * lightest >= heaviest : n > 70 && n < 92 && 3 * lightest >= heaviest))
    return kThrees;
  if (per_unit == 2 && n > 72 && n < 89) return kInTurn;
  return (one ? 4 : 3) * lightest < heaviest ? kFolded : kInTurn;
}

// The arrangements of a launch: of XCDs with an item in the last row of `group` workgroups each (n items), and, times four, of
// those without.
constexpr int64_t kFixedKeys = 400;      // keys that take as long as the start and the end of a workgroup (20000 cycles, 52 a key)
template <typename Weight>
inline int arrangements_of(int n, int group, int per_unit, int tile, bool one, Weight&& weight) {
  return arrangement_of(n, per_unit, tile, one, weight) + 4 * arrangement_of(n - group, per_unit, tile, one, weight);
}
// One problem, `tile` of its n_rows a workgroup; period: the items of a query tile for each of the group's query heads.
inline int tile_arrangements(int per_unit, int group, int64_t period, int tile, int64_t n_rows, int64_t n_vis, bool causal) {
  const int64_t rows = ((n_rows + tile - 1) / tile * period + 7) / 8;
  return arrangements_of((int)(rows * group), group, per_unit, tile, true, [&](int r) {
    const int64_t seen = causal ? n_rows - (int64_t)(r / group) * 8 / period * tile : 0;
    return kFixedKeys + n_vis + (seen > 0 ? seen : 0);
  });
}
// The problems of a schedule.
inline int schedule_arrangements(int per_unit, int group, int hkv, int tile, const GroupSchedule& s, const int64_t* n_vis) {
  const int64_t rows = ((int64_t)s.n_entries * hkv + 7) / 8;
  return arrangements_of((int)(rows * group), group, per_unit, tile, false, [&](int r) {
    const int64_t entry = (int64_t)(r / group) * 8 / hkv;
    int m, qt;
    decode_group_entry(s, entry < s.n_entries ? (int)entry : s.n_entries - 1, m, qt);
    return kFixedKeys + n_vis[m] + (int64_t)(qt + 1) * tile;
  });
}

}  // namespace apbv
