// Host check of the order in which an XCD's workgroups take its items (arrange_workgroup): every item once, whatever the
// number of items and of workgroups a unit holds; and with items whose weights fall evenly no unit gets much more than another.
#include <cstdio>
#include <vector>
#include "attention_schedule.h"

using namespace apbv;

#define EXPECT(x) do { if (!(x)) { std::printf("n %d per_unit %d line %d: %s\n", n, per_unit, __LINE__, #x); return 1; } } while (0)

int main() {
  // the other orders are permutations too, and the choice: weights that lie far apart, a flat few beyond two a unit, others
  for (int how : {kFolded, kInTurn})
    for (int per_unit = 1; per_unit <= 4; ++per_unit)
      for (int n = 1; n <= 200; ++n) {
        std::vector<int> seen(n, 0);
        for (int s = 0; s < n; ++s) {
          const int item = arrange_workgroup(s, n, per_unit, how);
          EXPECT(item >= 0 && item < n && seen[item]++ == 0);
          EXPECT(how != kInTurn || item == s);
        }
      }
  for (int n : {0, 32, 64, 65, 70, 71, 74, 95, 96, 97, 200}) {
    const int per_unit = 2;
    const bool few = n > 64 && n <= 70, more = n > 70 && n < 96;
    EXPECT(arrangement_of(n, [&](int) { return 500; }) == (few ? kInTurn : kThrees));
    EXPECT(arrangement_of(n, [&](int r) { return 9000 - 50 * r; }) == (n == 65 || n == 70 ? kInTurn : kThrees));
    if (more) EXPECT(arrangement_of(n, [&](int r) { return 1 + 100 * (n - 1 - r); }) == kFolded);
  }
  for (int per_unit = 1; per_unit <= 4; ++per_unit)
    for (int n = 1; n <= 200; ++n) {
      std::vector<int> seen(n, 0), load(kUnitsPerXcd, 0);
      for (int s = 0; s < n; ++s) {
        const int item = arrange_workgroup(s, n, per_unit);
        EXPECT(item >= 0 && item < n && seen[item]++ == 0);
        // past what the units hold at once, one each to the last units where three lie on some of them
        const int unit = s < 2 * kUnitsPerXcd || n > 3 * kUnitsPerXcd ? s % kUnitsPerXcd : 3 * kUnitsPerXcd - n + s % kUnitsPerXcd;
        load[unit] += 2 * n - item;
      }
      if (n <= kUnitsPerXcd || per_unit != 2 || n > 3 * kUnitsPerXcd) continue;
      int lo = load[0], hi = load[0], total = 0;
      for (int u = 0; u < kUnitsPerXcd; ++u) {
        lo = load[u] < lo ? load[u] : lo;
        hi = load[u] > hi ? load[u] : hi;
        total += load[u];
      }
      if (n % kUnitsPerXcd == 0 && n == 2 * kUnitsPerXcd) EXPECT(hi - lo <= 1);
      if (n > 2 * kUnitsPerXcd) EXPECT(kUnitsPerXcd * hi <= 1.25 * total);      // in plain order up to 1.5
    }
  std::printf("arrangement ok\n");
  return 0;
}
