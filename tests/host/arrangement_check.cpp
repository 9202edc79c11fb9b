// Host check of the order in which an XCD's workgroups take its items (arrange_workgroup): every item once, whatever the
// number of items and of workgroups a unit holds; and with items whose weights fall evenly no unit gets much more than another.
#include <cstdio>
#include <vector>
#include "attention_schedule.h"

using namespace apbv;

#define EXPECT(x) do { if (!(x)) { std::printf("n %d per_unit %d line %d: %s\n", n, per_unit, __LINE__, #x); return 1; } } while (0)

int main() {
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
