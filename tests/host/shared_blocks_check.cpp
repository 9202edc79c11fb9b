// Host check of the rule that gives a 32-row block to two waves (attention_shares_blocks): the launches of
// tests/test_gpu_shared_blocks.py alone and repeated, measured ones on both sides of the line, and the merged schedule of
// the 64-row workgroups it takes.
#include <cstdio>
#include <map>
#include <utility>
#include "attention_schedule.h"
#include "host_validation.h"

using namespace apbv;

#define EXPECT(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main() {
  struct { int hq, d; int64_t L, n_vis; bool causal; int repeats; } both[] = {
      {1, 64, 1, 0, true, 600},     {2, 128, 17, 5, true, 200},   {3, 64, 33, 47, true, 200},     {2, 128, 64, 31, true, 150},
      {1, 128, 65, 67, true, 150},  {2, 64, 100, 33, true, 140},  {1, 128, 128, 110, true, 140},  {4, 64, 161, 75, true, 70},
      {2, 128, 545, 1000, true, 40}, {2, 128, 40, 350, false, 150}, {4, 64, 200, 350, false, 60}};
  for (const auto& c : both) {
    EXPECT(attention_shares_blocks(c.d, 1, c.hq, c.L, c.n_vis, c.causal, 1));
    EXPECT(!attention_shares_blocks(c.d, c.repeats, c.hq, c.L, c.n_vis, c.causal, 1));
  }
  EXPECT(attention_shares_blocks(128, 1, 16, 1024, 224, true, 1) && !attention_shares_blocks(128, 1, 28, 1500, 400, true, 1));
  EXPECT(attention_shares_blocks(64, 1, 8, 4000, 720, true, 1) && !attention_shares_blocks(64, 1, 8, 8192, 0, true, 1));
  EXPECT(attention_shares_blocks(128, 1, 8, 3000, 850, true, 1) && !attention_shares_blocks(128, 4, 14, 288, 8345, true, 1));
  EXPECT(attention_shares_blocks(128, 1, 4, 40, 5000, false, 64) && !attention_shares_blocks(128, 1, 4, 40, 5000, false, 65));

  const int64_t n_vis[3] = {0, 150, 1207}, rows[3] = {70, 300, 333};
  GroupSchedule s;
  EXPECT(build_group_schedule(3, n_vis, rows, s, 64) && s.n_entries == 2 + 5 + 6);
  std::map<std::pair<int, int>, int> seen;
  for (int e = 0; e < s.n_entries; ++e) {
    int m, qt;
    decode_group_entry(s, e, m, qt);
    const int before = seen[std::make_pair(m, qt)]++;
    EXPECT(m >= 0 && m < 3 && qt >= 0 && qt * 64 < rows[m] && before == 0);
  }
  std::printf("shared blocks ok\n");
  return 0;
}
