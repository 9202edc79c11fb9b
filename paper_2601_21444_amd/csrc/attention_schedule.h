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

// Which of an XCD's n work items, numbered heaviest first, its s-th workgroup takes.  Workgroups are dispatched to the 32
// units in turn, so unit j gets numbers j, 32 + j, ... until it holds per_unit of them, and further ones go where one has
// ended.  Items taken in that order (kInTurn) would give unit 0 the heaviest of every round and unit 31 the lightest.  So
//   - kFolded: odd rounds run backwards, and where the last round is not full its units are those with the lightest items of
//     the rounds before: what the units hold adds up to about the same.  With more items than the units hold the ends even out
//     by themselves, and only the first rounds are arranged;
//   - kThrees: of up to one item more per unit than two fit (m > 0 of them) the lightest 3 m go to m units, three each, the
//     lightest of them dispatched last.  In turn the units' two workgroups could end together and take two of the last ones.
// arrangement_of() says which.
constexpr int kUnitsPerXcd = 32;
enum Arrangement { kFolded, kThrees, kInTurn };
APBV_HOST_DEVICE inline int arrange_workgroup(int s, int n, int per_unit, int how = kThrees) {
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
// By the items' weights, weight(r) of the r-th heaviest of an XCD's n (two to a unit).  Folded where they lie far apart: the
// pairs beside the threes would weigh more than a folded pair and one of the lightest, which are dispatched where one has
// ended.  In turn for a few items beyond two a unit that weigh about as much as the others.  us, in turn / folded / threes:
//   16 heads of 128, 5279 rows behind 570 keys 135.3 / 134.2 / 148.2     4430 behind 1500 134.6 / 140.8 / 129.5
//   8 heads of 128 with their own K/V, 11179 rows behind 522 keys 252.7 / 250.7 / 286.2     8887 behind 1897 221.0 / 210.9 / 206.3
//   (m = 3) 8526 behind 1500 203.2 / 195.9 / 194.8, behind 5000 307.1 / 331.9 / 336.9     (6) 8910 behind 5000 361.9 / 347.3 / 332.5
//   28 heads of 128 (6) 2382 behind 1500 117.1 / 109.1 / 111.0, behind 5000 239.8 / 245.6 / 248.1, 2 x 1230 behind 1500 94.3 / 97.1 / 97.8
// Not always right: 28 heads x 1088 rows in three problems 37.4 / 40.5 / 38.9.
template <typename Weight>
inline Arrangement arrangement_of(int n, Weight&& weight) {
  const int m = n - 2 * kUnitsPerXcd, pairs = kUnitsPerXcd - m;
  if (m <= 0 || pairs <= 0) return kThrees;
  if (m <= 6 && (0.2 + 0.055 * m) * (double)weight(0) < (double)weight(n - 1)) return kInTurn;
  return weight(2 * pairs - 1) <= weight(2 * kUnitsPerXcd - 1) + weight(2 * kUnitsPerXcd) ? kThrees : kFolded;
}

}  // namespace apbv
