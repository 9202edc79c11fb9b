// Host checks of two rules of the compression, and of the comparison that collects the scores of a long block.  Selection of
// long blocks (plan_long_selection): which calls of tests/test_gpu_long_select.py take it, and for every call that does, that
// the histograms fit the pooled query's region and their counts, and the parts have outputs and divide them.  Pooled query without a launch
// of its own (pools_in_scores): both sides of the line, among them the calls of tests/test_gpu_pooled_scores.py.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>
#include "host_validation.h"

using namespace apbv;

#define EXPECT_OR(x, result) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return result; } } while (0)
#define EXPECT(x) EXPECT_OR(x, 1)

static LongSelection plan(int hkv, int batch, int d, int64_t L, int64_t l_p) {
  return plan_long_selection((int64_t)hkv * batch, d, L, l_p, plan_compress_workspace(batch, hkv, d, L, l_p));
}

// The shares of long_select_gather_kernel over random bins, from one score to nearly all in one: every output belongs to one
// part, a part that collects has whole bins (the last cut at l_p) that fit the LDS, and the others are those of large bins.
static bool shares_fit(int64_t L, int64_t l_p, int n_parts) {
  static std::mt19937_64 rng(5);
  const uint32_t most = most_of_a_bin(l_p, n_parts);
  for (int trial = 0; trial < 6; ++trial) {
    std::vector<uint32_t> begin{0};                       // first output of every bin, then L
    while (begin.back() < L) {
      const uint32_t sizes[] = {1, 40, 500, most, most + 1, 9000, (uint32_t)L};
      const uint32_t n = 1 + (uint32_t)(rng() % sizes[rng() % (trial + 2)]);
      begin.push_back((uint32_t)std::min<int64_t>(L, (int64_t)begin.back() + (rng() % 4 ? n : sizes[rng() % 7])));
    }
    uint32_t next = 0;
    for (int part = 0; part < n_parts; ++part) {
      const uint32_t from = (uint32_t)(l_p * part / n_parts), to = (uint32_t)(l_p * (part + 1) / n_parts);
      uint32_t share[2] = {0, 0}, last = 0;
      bool divided = false;
      for (size_t i = 0; i + 1 < begin.size(); ++i) {
        const uint32_t excl = begin[i], c = begin[i + 1] - excl;
        if (excl <= from && from < excl + c) share[0] = first_of_share(from, excl, c, most);
        if (excl <= to && to < excl + c) share[1] = first_of_share(to, excl, c, most);
        if (c > most && excl < to && from < excl + c) divided = true;
        if (excl >= from && excl < to) last = excl + c;
      }
      const uint32_t first = share[0], end = std::min<uint32_t>(share[1], (uint32_t)l_p);
      if (first >= end) continue;
      EXPECT_OR(first == next, false);
      next = end;
      if (divided) continue;
      const bool begins = std::binary_search(begin.begin(), begin.end(), first), ends = std::binary_search(begin.begin(), begin.end(), end) || end == l_p;
      EXPECT_OR(begins && ends && last >= end && last - first <= kLdsSortMax, false);
    }
    EXPECT_OR(next == l_p, false);
  }
  return true;
}

int main() {
  struct { int hkv, batch, d; int64_t L, l_p; int n_parts; } cases[] = {
      {1, 1, 64, 24576, 1, 1},     {1, 1, 64, 24575, 1, 0},     {2, 1, 64, 24577, 513, 16},  {2, 1, 128, 65536, 2000, 16}, {1, 2, 64, 40001, 8192, 16},
      {1, 1, 64, 40001, 8193, 0},  {1, 1, 64, 17000, 8065, 16}, {1, 1, 64, 131072, 700, 16}, {1, 1, 64, 131073, 700, 0},   {1, 1, 128, 140000, 64, 2},
      {2, 1, 64, 30000, 33, 1},    {4, 8, 64, 25000, 200, 6},   {3, 11, 64, 25000, 200, 0},  {2, 1, 128, 16384, 500, 0},   {1, 1, 64, 30000, 0, 0}};
  for (const auto& c : cases) EXPECT(plan(c.hkv, c.batch, c.d, c.L, c.l_p).n_parts == c.n_parts);
  for (int d : {64, 128})
    for (int heads = 1; heads <= 40; heads += heads / 4 + 1)
      for (int64_t L = 16000; L < 300000; L += L / 5 + 1)
        for (int64_t l_p = 1; l_p <= 8200 && l_p <= L; l_p += l_p / 3 + 1) {
          const CompressWorkspace w = plan_compress_workspace(1, heads, d, L, l_p);
          const LongSelection s = plan_long_selection(heads, d, L, l_p, w);
          if (s.n_parts == 0) continue;
          EXPECT(w.qbar_off + (size_t)heads * s.n_hist * sizeof(CoarseHistogram) <= w.scores_off && w.n_sort <= kLdsSortMax);
          EXPECT((L + s.n_hist - 1) / s.n_hist <= kResidentScores && s.n_parts <= l_p && s.n_parts * heads <= 256);
          EXPECT(L - l_p + 1 > kLdsSortMax);      // bin 0, if it has an output: the collecting loop does not take it
          if (!shares_fit(L, l_p, s.n_parts)) return 1;
        }
  // every part of every head once, those of a whole row of heads on one XCD
  for (int heads = 1; heads <= kMaxLongHeads; ++heads)
    for (int parts = 1; parts <= 16; ++parts) {
      std::vector<int> seen(heads * parts, 0);
      for (int w = 0; w < heads * parts; ++w) {
        const HeadPart at = head_and_part(w, parts, heads);
        EXPECT(at.head >= 0 && at.head < heads && at.part >= 0 && at.part < parts && seen[at.head * parts + at.part]++ == 0);
        EXPECT(at.head >= heads / 8 * 8 || at.head % 8 == w % 8);
      }
    }
  // the test that collects the scores of a range of bins, [lowest, past) in the order of their upper halves
  const double values[] = {-INFINITY, -1e300, -1234.5, -1.0, -1e-300, -0.0, 0.0, 1e-300, 1.0, 1234.5, 1e300, INFINITY};
  auto order_of = [](double x) {
    int64_t bits;
    std::memcpy(&bits, &x, sizeof bits);
    return upper_order((int)(bits >> 32));
  };
  for (double a : values) {
    EXPECT(upper_order(upper_order(order_of(a))) == order_of(a));
    for (double b : values) {
      EXPECT(!(a < b) || order_of(a) < order_of(b));
      for (int past : {order_of(b), kOrderInf + 1})
        for (double x : values)
          if (order_of(a) <= past)
            EXPECT((order_distance(order_of(a), order_of(x)) < order_distance(order_of(a), past)) == (order_of(a) <= order_of(x) && order_of(x) < past));
    }
  }
  EXPECT(pools_in_scores(64, 128, 2, 16384) && !pools_in_scores(160, 128, 2, 16384) && pools_in_scores(160, 128, 2, 8000));
  EXPECT(pools_in_scores(256, 64, 2, 16384) && !pools_in_scores(256, 64, 8, 16384) && !pools_in_scores(64, 128, 8, 12000));
  EXPECT(!pools_in_scores(512, 128, 2, 2000) && !pools_in_scores(512, 128, 1, 1) && pools_in_scores(1, 64, 1, 1));
  for (int64_t rows : {1, 15, 16, 17, 64, 65, 160}) EXPECT(pools_in_scores(rows, 128, 2, 700));
  for (int64_t rows : {31, 33, 128, 129, 320}) EXPECT(pools_in_scores(rows, 64, 2, 700));
  EXPECT(!pools_in_scores(161, 128, 2, 700) && !pools_in_scores(321, 64, 2, 700));
  // one launch for all steps (tests/test_gpu_short_blocks.py): its sizes on both sides of every line
  EXPECT(compresses_at_once(1, 64, 9, 1, 1) == 1 && compresses_at_once(1, 64, 8, 1, 1) == 0);
  EXPECT(compresses_at_once(129, 64, 12, 513, 100) == 3 && compresses_at_once(65, 128, 10, 257, 257) == 8 && compresses_at_once(264, 128, 12, 256, 96) == 3);
  EXPECT(compresses_at_once(512, 128, 96, 829, 100) == 0 && compresses_at_once(112, 64, 9, 600, 400) == 12);
  EXPECT(compresses_at_once(10, 64, 128, 1023, 33) == 1 && compresses_at_once(9, 128, 128, 700, 65) == 2 && compresses_at_once(4, 128, 256, 1024, 512) == 1);
  EXPECT(compresses_at_once(1024, 64, 272, 1024, 40) == 1 && compresses_at_once(1025, 64, 272, 1024, 40) == 0);
  EXPECT(compresses_at_once(2, 64, 256, 1025, 40) == 0 && compresses_at_once(2, 64, 256, 1024, 0) == 0);
  EXPECT(compresses_at_once(1, 64, 256, 1024, 1024) == 1 && compresses_at_once(2, 128, 256, 1024, 1024) == 1 && compresses_at_once(6, 64, 256, 1024, 1023) == 1);
  EXPECT(compresses_at_once(768, 128, 640, 768, 537) == 1 && compresses_at_once(768, 128, 640, 768, 538) == 0);      // the memory line, 3686.4 rows a head
  std::printf("compression rules ok\n");
  return 0;
}
