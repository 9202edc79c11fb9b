// Host check of the rule that gives a 32-row block to two waves (attention_shares_blocks) and of the workgroups the launches
// take with it (attention_kernel, attention_group_kernel): those of tests/test_gpu_shared_blocks.py alone and repeated, of
// tests/test_gpu_attention_workgroups.py alone, repeated and grouped, of tests/test_gpu_group.py; measured ones on both sides
// of the line; and the merged schedule of the 64-row workgroups.
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

  typedef AttentionKernel K;
  // tests/test_gpu_reference_moves.py: waves of one 16-row block alone, of two in the batch
  EXPECT(attention_kernel(64, 2, 1, 2, 545, 1000, true, 1) == K::kShared64 && attention_kernel(64, 2, 44, 2, 545, 1000, true, 1) == K::k128);
  EXPECT(attention_kernel(128, 2, 1, 2, 545, 1000, true, 1) == K::kShared64 && attention_kernel(128, 2, 40, 2, 545, 1000, true, 1) == K::k256);
  struct { int hq, hkv, d; int64_t L, n_vis; int repeats; K alone, batch, group; } launches[] = {
      {2, 1, 64, 129, 0, 40, K::kShared64, K::kShared64, K::kShared64},   {2, 1, 64, 700, 128, 12, K::kShared64, K::kShared64, K::kShared64},
      {4, 1, 64, 300, 5000, 40, K::kShared64, K::k128, K::kShared64},     {8, 8, 64, 150, 1000, 30, K::kShared64, K::kShared64, K::kShared64},
      {4, 2, 128, 129, 7, 3, K::kShared64, K::kShared64, K::kShared64},   {4, 2, 128, 513, 4040, 20, K::kShared64, K::k256, K::kShared64},
      {28, 4, 128, 700, 1500, 3, K::k128, K::k256, K::k256},              {40, 8, 128, 289, 1700, 3, K::kShared64, K::k256, K::k256},
      {8, 4, 64, 77, 70, 40, K::kShared64, K::kNarrow64, K::kShared64},   {8, 2, 128, 100, 70, 20, K::kShared64, K::kNarrow64, K::kShared64},
      {16, 4, 64, 1700, 60, 2, K::kShared64, K::k128, K::k128},           {16, 2, 128, 1200, 100, 2, K::kShared64, K::k128, K::k128},
      {8, 8, 64, 1500, 200, 83, K::kShared64, K::k256, K::kShared64}};
  for (const auto& c : launches) {
    const int64_t n_vis[3] = {c.n_vis, c.n_vis, c.n_vis}, rows[3] = {c.L, c.L, c.L};
    EXPECT(attention_kernel(c.d, c.hq / c.hkv, 1, c.hq, c.L, c.n_vis, true, 1) == c.alone);
    EXPECT(attention_kernel(c.d, c.hq / c.hkv, c.repeats, c.hq, c.L, c.n_vis, true, 1) == c.batch);
    EXPECT(attention_group_kernel(c.d, c.hq, c.hkv, 3, n_vis, rows) == c.group);
  }
  struct { int hq, hkv, d, n; int64_t rows[5], n_vis[5]; K kernel; } groups[] = {
      {4, 2, 128, 3, {300, 700, 700}, {0, 300, 750}, K::kShared64},       {8, 2, 64, 4, {257, 1, 513, 256}, {1010, 0, 255, 512}, K::kShared64},
      {6, 3, 64, 2, {900, 1300}, {64, 264}, K::kShared64},                {16, 2, 128, 3, {900, 1300, 333}, {64, 264, 50}, K::k128},
      {16, 8, 128, 3, {1900, 1300, 333}, {64, 264, 50}, K::k128},         {32, 4, 64, 3, {700, 640, 333}, {64, 100, 15}, K::k128},
      {28, 4, 128, 3, {700, 901, 1000}, {1500, 1733, 333}, K::k128},      {16, 2, 128, 3, {2048, 16384, 16384}, {0, 2048, 17408}, K::k256},
      {27, 27, 64, 5, {5250, 5213, 5176, 5139, 5102}, {12000, 12101, 12202, 12303, 12404}, K::k256}};
  for (const auto& c : groups) EXPECT(attention_group_kernel(c.d, c.hq, c.hkv, c.n, c.n_vis, c.rows) == c.kernel);

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
