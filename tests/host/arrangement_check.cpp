// Host check of the order in which an XCD's workgroups take its items (arrange_workgroup): every item once, whatever the
// number of items and of workgroups a unit holds; with items whose weights fall evenly, what the units' items add up to; the
// rule that chooses (arrangement_of); and the workgroups, items and orders of the launches of tests/test_launch_arrangement.py.
#include <cstdio>
#include <vector>
#include "attention_schedule.h"
#include "host_validation.h"

using namespace apbv;

#define EXPECT(x) do { if (!(x)) { std::printf("n %d per_unit %d how %d line %d: %s\n", n, per_unit, how, __LINE__, #x); return 1; } } while (0)

// 100 times the largest sum of a unit's items over the mean.  (Of threes, the last ones go to the last units.)
static int spread(int n, int per_unit, int how) {
  std::vector<int64_t> load(kUnitsPerXcd, 0);
  int64_t hi = 0, total = 0;
  for (int s = 0; s < n; ++s) {
    const int unit = how != kThrees || s < 2 * kUnitsPerXcd ? s % kUnitsPerXcd : 3 * kUnitsPerXcd - n + s % kUnitsPerXcd;
    load[unit] += 2 * n - arrange_workgroup(s, n, per_unit, how);
  }
  for (const int64_t l : load) {
    hi = l > hi ? l : hi;
    total += l;
  }
  return (int)(100 * kUnitsPerXcd * hi / total);
}

int main() {
  for (int how : {kInTurn, kFolded, kThrees})
    for (int per_unit = 1; per_unit <= 4; ++per_unit)
      for (int n = 1; n <= 200; ++n) {
        std::vector<int> seen(n, 0);
        for (int s = 0; s < n; ++s) {
          const int item = arrange_workgroup(s, n, per_unit, how);
          EXPECT(item >= 0 && item < n && seen[item]++ == 0);
          EXPECT(how != kInTurn || item == s);
        }
      }
  for (int n = kUnitsPerXcd + 1; n <= 3 * kUnitsPerXcd; ++n) {
    int per_unit = 2, how = kFolded;
    if (n <= 2 * kUnitsPerXcd) {
      EXPECT(spread(n, 2, kFolded) <= 168 - n && spread(n, 2, kInTurn) >= 168 - n);       // 133 to 100, in plain order 193 to 117
    } else {
      how = kThrees;
      EXPECT(spread(n, 2, kThrees) <= 125);                                // in plain order up to 150
      per_unit = 3;
      how = kFolded;
      EXPECT(spread(n, 3, kFolded) <= 132 && spread(n, 3, kFolded) + 5 <= spread(n, 3, kInTurn));
    }
  }

  int n = 0, per_unit = 0, how = 0;
  // the rule: flat weights, lightest just below and just at a half, a third and a quarter of the heaviest, of one problem or several
  for (n = 1; n <= 200; ++n)
    for (per_unit = 1; per_unit <= 4; ++per_unit)
      for (how = 0; how < 2; ++how) {
        const bool one = how == 0, resident = n <= 32 * per_unit, arranged = n > 32 && n <= 128 && (per_unit == 2 || per_unit == 3);
        auto of = [&](int64_t lightest, int tile = 128) {
          return arrangement_of(n, per_unit, tile, one, [&](int r) { return r == 0 ? (int64_t)1200 : lightest; });
        };
        EXPECT(of(1200) == kInTurn && of(600) == kInTurn);
        EXPECT(of(1200, 64) == (arranged && resident ? kFolded : kInTurn));
        const bool gap = per_unit == 2 && n >= 73 && n <= 88;
        const Arrangement between = per_unit == 2 && n >= (one ? 69 : 71) && n <= (one ? 95 : 91) ? kThrees : kInTurn, below = gap ? kInTurn : kFolded;
        for (const int64_t lightest : {599, 400, 399, 300, 299}) {
          Arrangement expected = kInTurn;
          if (arranged) expected = resident ? kFolded : lightest >= (one ? 300 : 400) ? between : below;
          EXPECT(of(lightest) == expected);
        }
      }

  typedef AttentionKernel K;
  constexpr int T = kInTurn, F = kFolded, H = kThrees;
  struct { int batch, hq, hkv, d; int64_t L, n_vis; K kernel; int per_unit, n, left, all, fewer; } singles[] = {
      {3, 6, 3, 128, 1654, 136, K::kShared64, 2, 60, 2, F, F},  {2, 16, 2, 128, 655, 4, K::kShared64, 2, 48, 4, F, F},
      {4, 6, 3, 128, 2674, 572, K::k128, 2, 64, 4, F, F},       {2, 6, 3, 128, 2756, 42, K::k128, 2, 34, 4, F, T},
      {2, 16, 2, 128, 2111, 130, K::k128, 2, 72, 4, F, F},      {2, 16, 2, 128, 2324, 2, K::k128, 2, 80, 4, T, F},
      {3, 16, 2, 128, 1381, 32, K::k128, 2, 72, 2, H, F},
      {3, 28, 4, 128, 806, 121, K::k128, 2, 77, 4, H, H},       {3, 16, 2, 128, 1610, 559, K::k128, 2, 80, 6, H, T},
      {3, 28, 4, 128, 794, 1731, K::k128, 2, 77, 4, T, T},      {3, 28, 4, 128, 1084, 36, K::k128, 2, 98, 4, T, H},
      {3, 16, 2, 128, 2125, 33, K::k128, 2, 104, 6, F, T},      {3, 16, 2, 128, 2605, 5, K::k128, 2, 128, 6, F, F},
      {3, 16, 2, 128, 2728, 47, K::k128, 2, 136, 4, T, F},
      {2, 9, 3, 64, 3273, 1385, K::k128, 3, 60, 4, F, F},       {2, 9, 3, 64, 3657, 931, K::k128, 3, 66, 6, F, F},
      {4, 9, 3, 64, 3110, 110, K::k128, 3, 114, 4, F, F},       {3, 9, 3, 64, 3704, 1337, K::k128, 3, 99, 5, T, F},
      {3, 9, 3, 64, 1357, 48, K::kShared64, 4, 75, 6, T, T}};
  for (const auto& c : singles) {
    const int own = c.kernel == K::kShared64 ? 1 : 2, tile = 64 * own, group = c.hq / c.hkv;
    n = c.n;
    per_unit = workgroups_per_unit(c.d, 4, own);
    how = (int)c.L;
    EXPECT(attention_kernel(c.d, group, c.batch, c.hq, c.L, c.n_vis, true, 1) == c.kernel && per_unit == c.per_unit);
    const int64_t items = (c.L + tile - 1) / tile * c.batch * c.hkv;
    EXPECT((items + 7) / 8 * group == c.n && items % 8 == c.left);
    EXPECT(tile_arrangements(per_unit, group, c.batch * c.hkv, tile, c.L, c.n_vis, true) == c.all + 4 * c.fewer);
  }
  struct { int hq, hkv, d, count; int64_t rows[3], n_vis[3]; K kernel; int per_unit, n, left, all, fewer; } groups[] = {
      {6, 3, 128, 2, {1944, 1898}, {870, 15}, K::kShared64, 2, 46, 7, F, F},
      {16, 2, 128, 2, {696, 354}, {272, 30}, K::kShared64, 2, 40, 2, F, T},
      {6, 3, 128, 3, {2358, 2549, 2788}, {322, 1832, 1320}, K::k128, 2, 46, 7, F, F},
      {28, 4, 128, 2, {903, 1299}, {50, 1198}, K::k128, 2, 70, 4, F, F},
      {16, 2, 128, 2, {2319, 2047}, {726, 1963}, K::k128, 2, 72, 6, H, F},
      {28, 4, 128, 2, {755, 2133}, {847, 1218}, K::k128, 2, 84, 4, H, H},
      {28, 4, 128, 2, {1865, 1224}, {1227, 1526}, K::k128, 2, 91, 4, H, T},
      {28, 4, 128, 2, {2161, 1758}, {47, 17}, K::k128, 2, 112, 4, F, F},
      {28, 4, 128, 3, {1983, 472, 2116}, {23, 1812, 564}, K::k128, 2, 133, 4, T, F},
      {8, 2, 64, 3, {3515, 1838, 788}, {33, 1337, 78}, K::k128, 3, 52, 4, F, F},
      {9, 3, 64, 3, {1907, 2464, 2994}, {58, 1925, 1569}, K::k128, 3, 69, 1, F, F},
      {9, 3, 64, 3, {3774, 3413, 3642}, {1278, 307, 10}, K::k128, 3, 99, 2, F, F},
      {9, 3, 64, 2, {1800, 496}, {64, 396}, K::kShared64, 4, 42, 7, T, T}};
  for (const auto& c : groups) {
    const int own = c.kernel == K::kShared64 ? 1 : 2, tile = 64 * own, group = c.hq / c.hkv;
    n = c.n;
    per_unit = workgroups_per_unit(c.d, 4, own);
    how = (int)c.rows[0];
    EXPECT(attention_group_kernel(c.d, c.hq, c.hkv, c.count, c.n_vis, c.rows) == c.kernel && per_unit == c.per_unit);
    GroupSchedule s;
    EXPECT(build_group_schedule(c.count, c.n_vis, c.rows, s, tile));
    EXPECT((s.n_entries * c.hkv + 7) / 8 * group == c.n && s.n_entries * c.hkv % 8 == c.left);
    EXPECT(schedule_arrangements(per_unit, group, c.hkv, tile, s, c.n_vis) == c.all + 4 * c.fewer);
  }
  std::printf("arrangement ok\n");
  return 0;
}
