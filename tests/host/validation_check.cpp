// Host check of the C ABI's argument validation and planning (csrc/host_validation.h), compiled with the plain C++
// compiler under -fsanitize=address,undefined: every rejection case returns its status without touching the forged
// pointers, and the planners stay in range over a sweep of shapes.
#include <initializer_list>
#include <cstdio>
#include <cstdlib>
#include <limits>
#include "attention_schedule.h"
#include "host_validation.h"

using namespace apbv;

static int failures = 0;
#define EXPECT(cond)                                                              \
  do {                                                                            \
    if (!(cond)) {                                                                \
      std::printf("FAILED line %d: %s\n", __LINE__, #cond);                       \
      ++failures;                                                                 \
    }                                                                             \
  } while (0)

static apbv_tensor view(int64_t tokens, int heads, int d, uintptr_t ptr = 0x1000) {
  apbv_tensor t;
  t.ptr = tokens ? reinterpret_cast<const void*>(ptr) : nullptr;      // never dereferenced
  t.tokens = tokens;
  t.stride_token = (int64_t)heads * d;
  t.stride_head = d;
  t.stride_batch = tokens * heads * d;
  return t;
}
static const void* P(uintptr_t x) { return reinterpret_cast<const void*>(x); }

static apbv_status attn(int batch = 1, int hq = 4, int hkv = 2, int d = 128, int64_t L = 64, int64_t l_a = 16, int64_t n_p = 8,
                        float scale = 0.1f, const void* out = P(0x2000), const apbv_tensor* q = nullptr,
                        const apbv_tensor* k = nullptr, const apbv_tensor* v = nullptr) {
  apbv_tensor qq = q ? *q : view(L, hq, d), kk = k ? *k : view(L, hkv, d), vv = v ? *v : view(L, hkv, d);
  return validate_attention(batch, hq, hkv, d, qq, view(l_a, hkv, d), view(l_a, hkv, d), view(n_p, hkv, d), view(n_p, hkv, d),
                            kk, vv, scale, out, nullptr);
}

static apbv_status comp(int reducer = 0, float scale = 0.f, int batch = 1, int hq = 4, int hkv = 2, int d = 128, int64_t n_q = 4,
                        int64_t L = 64, int64_t l_p = 8, const void* idx = P(0x3000), const void* kc = P(0x4000),
                        const void* vc = P(0x5000), const apbv_tensor* v = nullptr) {
  apbv_tensor vv = v ? *v : view(L, hkv, d);
  return validate_compress(reducer, scale, batch, hq, hkv, d, view(n_q, hq, d), view(L, hkv, d), vv, l_p,
                           static_cast<const int32_t*>(idx), kc, vc, nullptr);
}

int main() {
  // ---- attention
  EXPECT(attn() == APBV_OK);
  EXPECT(attn(0) == APBV_ERR_SHAPE && attn(1, 5) == APBV_ERR_SHAPE && attn(1, 4, 2, 96) == APBV_ERR_UNSUPPORTED);
  EXPECT(attn(1, 4, 2, 128, 0) == APBV_ERR_SHAPE);
  EXPECT(attn(1, 4, 2, 128, 64, 16, 8, 0.f) == APBV_ERR_SHAPE && attn(1, 4, 2, 128, 64, 16, 8, -1.f) == APBV_ERR_SHAPE);
  EXPECT(attn(1, 4, 2, 128, 64, 16, 8, std::numeric_limits<float>::infinity()) == APBV_ERR_SHAPE);
  EXPECT(attn(1, 4, 2, 128, 64, 16, 8, std::numeric_limits<float>::quiet_NaN()) == APBV_ERR_SHAPE);
  EXPECT(attn(1, 4, 2, 128, 64, 16, 8, 0.1f, nullptr) == APBV_ERR_NULL && attn(1, 4, 2, 128, 64, 16, 8, 0.1f, P(0x2004)) == APBV_ERR_SHAPE);
  {
    apbv_tensor bad = view(64, 2, 128, 0x1008);                       // misaligned pointer
    EXPECT(attn(1, 4, 2, 128, 64, 16, 8, 0.1f, P(0x2000), nullptr, &bad) == APBV_ERR_SHAPE);
    apbv_tensor nul = view(64, 2, 128);
    nul.ptr = nullptr;
    EXPECT(attn(1, 4, 2, 128, 64, 16, 8, 0.1f, P(0x2000), nullptr, &nul) == APBV_ERR_NULL);
    apbv_tensor overlap = view(64, 2, 128);
    overlap.stride_token = 64;                                         // rows overlap
    EXPECT(attn(1, 4, 2, 128, 64, 16, 8, 0.1f, P(0x2000), nullptr, &overlap) == APBV_ERR_SHAPE);
    apbv_tensor odd = view(64, 2, 128);
    odd.stride_head = 132;                                             // not a multiple of 8
    EXPECT(attn(1, 4, 2, 128, 64, 16, 8, 0.1f, P(0x2000), nullptr, &odd) == APBV_ERR_SHAPE);
    apbv_tensor wide = view(64, 2, 128);
    wide.stride_token = (int64_t)1 << 24;
    EXPECT(attn(1, 4, 2, 128, 64, 16, 8, 0.1f, P(0x2000), nullptr, &wide) == APBV_ERR_UNSUPPORTED);
    apbv_tensor shortv = view(63, 2, 128);
    EXPECT(attn(1, 4, 2, 128, 64, 16, 8, 0.1f, P(0x2000), nullptr, nullptr, &shortv) == APBV_ERR_SHAPE);
    apbv_tensor none = view(0, 2, 128);
    EXPECT(attn(1, 4, 2, 128, 64, 0, 0, 0.1f, P(0x2000), nullptr, &none, &none) == APBV_ERR_SHAPE);      // no key at all
    EXPECT(attn(1, 4, 2, 128, 64, 16, 0, 0.1f, P(0x2000), nullptr, &none, &none) == APBV_OK);            // no causal segment
    apbv_tensor huge = view(((int64_t)1 << 24) + 1, 4, 128);
    EXPECT(attn(1, 4, 2, 128, 64, 16, 8, 0.1f, P(0x2000), &huge) == APBV_ERR_SHAPE);
    apbv_tensor batched = view(64, 4, 128);
    batched.stride_batch = 0;
    EXPECT(attn(2, 4, 2, 128, 64, 16, 8, 0.1f, P(0x2000), &batched) == APBV_ERR_SHAPE);
  }
  // ---- compression
  EXPECT(comp() == APBV_OK);
  EXPECT(comp(0, 0.f, 1, 4, 2, 128, 4, 64, 65) == APBV_ERR_SHAPE && comp(0, 0.f, 1, 4, 2, 128, 4, 64, -1) == APBV_ERR_SHAPE);
  EXPECT(comp(0, 0.f, 1, 5) == APBV_ERR_SHAPE && comp(0, 0.f, 1, 4, 2, 32) == APBV_ERR_UNSUPPORTED);
  EXPECT(comp(0, 0.f, 1, 4, 2, 128, 4, 64, 8, nullptr) == APBV_ERR_NULL);
  EXPECT(comp(0, 0.f, 1, 4, 2, 128, 4, 64, 0, nullptr, nullptr, nullptr) == APBV_OK);                   // l_p = 0 writes nothing
  EXPECT(comp(0, 0.f, 1, 4, 2, 128, 4, 64, 8, P(0x3000), P(0x4002)) == APBV_ERR_SHAPE);
  EXPECT(comp(0, 0.f, 1, 4, 2, 128, 0) == APBV_ERR_SHAPE);
  EXPECT(comp(3) == APBV_ERR_SHAPE && comp(-1) == APBV_ERR_SHAPE);
  EXPECT(comp(2, 0.f) == APBV_ERR_SHAPE && comp(2, 0.1f) == APBV_OK && comp(1, 0.f) == APBV_OK);
  {
    apbv_tensor shortv = view(63, 2, 128);
    EXPECT(comp(0, 0.f, 1, 4, 2, 128, 4, 64, 8, P(0x3000), P(0x4000), P(0x5000), &shortv) == APBV_ERR_SHAPE);
  }
  // ---- merge
  EXPECT(validate_merge(3, 10, 4, 128, P(0x1000), 10 * 4 * 128, static_cast<const float*>(P(0x2000)), 40, P(0x3000), nullptr) == APBV_OK);
  EXPECT(validate_merge(0, 10, 4, 128, P(0x1000), 5120, static_cast<const float*>(P(0x2000)), 40, P(0x3000), nullptr) == APBV_ERR_SHAPE);
  EXPECT(validate_merge(3, 10, 4, 128, P(0x1000), 5112, static_cast<const float*>(P(0x2000)), 40, P(0x3000), nullptr) == APBV_ERR_SHAPE);
  EXPECT(validate_merge(3, 10, 4, 128, P(0x1000), 5120, static_cast<const float*>(P(0x2000)), 39, P(0x3000), nullptr) == APBV_ERR_SHAPE);
  EXPECT(validate_merge(3, 10, 4, 96, P(0x1000), 5120, static_cast<const float*>(P(0x2000)), 40, P(0x3000), nullptr) == APBV_ERR_UNSUPPORTED);
  EXPECT(validate_merge(3, 10, 4, 128, nullptr, 5120, static_cast<const float*>(P(0x2000)), 40, P(0x3000), nullptr) == APBV_ERR_NULL);
  // rows per workgroup where blocks are not shared (tests/host/shared_blocks_check.cpp has the launches): problems alone, in a
  // batch and three in a group, and measured ones on both sides of the rule
  struct { int hq, hkv, d; int64_t L, n_vis; int repeats, alone, batch, group; } rows_of[] = {
      {2, 1, 64, 129, 0, 40, 64, 128, 128},       {2, 1, 64, 700, 128, 12, 64, 128, 128},    {4, 1, 64, 300, 5000, 40, 64, 128, 128},
      {8, 8, 64, 150, 1000, 30, 64, 256, 128},    {4, 2, 128, 129, 7, 3, 128, 128, 128},     {4, 2, 128, 513, 4040, 20, 128, 256, 128},
      {28, 4, 128, 700, 1500, 3, 128, 256, 256},  {40, 8, 128, 289, 1700, 3, 128, 256, 256}};
  for (const auto& c : rows_of) {
    EXPECT(attention_rows(c.d, c.hq / c.hkv, 1, c.hq, c.L, c.n_vis, true, 1) == c.alone);
    EXPECT(attention_rows(c.d, c.hq / c.hkv, c.repeats, c.hq, c.L, c.n_vis, true, 1) == c.batch);
    AttentionTiles tiles[3];
    for (int m = 0; m < 3; ++m)
      for (int i = 0; i < 3; ++i) add_attention_tiles(tiles[i], 64 << i, c.hq, c.L, c.n_vis, true);
    const double kv = 3.0 * (double)(c.n_vis + c.L) * c.hkv * c.d * 4, qo = 3.0 * (double)c.L * c.hq * c.d * 4;
    EXPECT(attention_rows(c.d, c.hq / c.hkv, c.hkv, tiles, kv, qo, false) == c.group);
  }
  EXPECT(attention_rows(128, 8, 1, 16, 2048, 8704, true, 1) == 128 && attention_rows(128, 8, 1, 16, 4096, 0, true, 1) == 128);
  EXPECT(attention_rows(128, 8, 1, 16, 4096, 32768, true, 1) == 256 && attention_rows(128, 8, 1, 16, 16384, 9216, true, 1) == 256);
  EXPECT(attention_rows(128, 4, 5, 32, 233, 1829, false, 1) == 256 && attention_rows(128, 1, 1, 32, 3899, 0, true, 1) == 256);
  EXPECT(attention_rows(128, 7, 2, 28, 3001, 564, true, 1) == 128 && attention_rows(128, 7, 4, 28, 2048, 500, true, 1) == 128);
  EXPECT(attention_rows(128, 1, 68, 16, 1752, 827, true, 1) == 256 && attention_rows(128, 8, 68, 16, 1752, 827, true, 1) == 128);
  EXPECT(attention_rows(128, 1, 1, 84, 3031, 0, true, 1) == 256 && attention_rows(128, 1, 1, 96, 2874, 0, true, 1) == 128);
  EXPECT(attention_rows(64, 1, 83, 16, 3743, 937, true, 1) == 256 && attention_rows(64, 4, 1, 8, 8192, 0, true, 1) == 128);
  // lanes per item: a launch stays below 2^32 threads (blocks of 256) at every number of parts and items, and only a few
  // items get more lanes than read 128 bytes of a part together
  for (int64_t items = 8; items <= (int64_t)1 << 31; items += items / 3 + 1)
    for (int n_parts = 1; n_parts <= 65536; n_parts += n_parts / 5 + 1) {
      const int lanes = merge_lanes(items, n_parts);
      EXPECT(lanes == 1 || lanes == 2 || lanes == 4 || lanes == 8 || lanes == 16 || lanes == 64);
      EXPECT((items * lanes + 255) / 256 * 256 < (int64_t)1 << 32 && (lanes <= 8 || items <= 4096));
      EXPECT(lanes > 1 || n_parts <= 8 || items > (int64_t)1 << 28);
    }
  EXPECT(merge_lanes(((int64_t)1 << 29) - 1, 65) == 1 && merge_lanes((int64_t)1 << 28, 17) == 8);
  EXPECT(merge_items(2, 3, 5, 128) == 2 * 3 * 5 * 16 && merge_items(1, (int64_t)1 << 24, 65535, 64) == ((int64_t)65535 << 27));
  // ---- planners over a sweep: the key split covers every tile exactly once with no empty range; workspaces are
  // aligned, ordered and monotone in the batch
  for (int64_t n_keys = 1; n_keys < 300000; n_keys = n_keys * 3 + 7)
    for (int64_t n_q = 1; n_q <= 4096; n_q *= 4)
      for (int req = 0; req <= 300; req = req * 2 + 1) {
        const KeySplit ks = plan_key_split(1, 16, n_q, n_keys, req);
        const int64_t n_tiles = (n_keys + kAttnKeyTile - 1) / kAttnKeyTile;
        EXPECT(ks.n_splits >= 1 && ks.n_splits <= kMaxKeySplits && ks.tiles_per_split >= 1);
        EXPECT((int64_t)ks.n_splits * ks.tiles_per_split >= n_tiles);
        EXPECT((int64_t)(ks.n_splits - 1) * ks.tiles_per_split < n_tiles);
        const size_t ws = query_attention_workspace_bytes(1, 16, 128, n_q, n_keys, req);
        EXPECT(ws % 256 == 0 && (ks.n_splits == 1) == (ws == 0));
      }
  // the query block's kernel and ranges: what was requested, or at most what the workspace is sized for and holds; every
  // tile covered; a kernel only where it can run
  for (int d : {64, 128})
    for (int hq : {1, 2, 16, 28, 65535})
      for (int g : {1, 2, 4, 7, 16, 65535})
        for (int batch : {1, 5, 130, 65535})
          for (int64_t n_q : {1, 2, 17, 128, 129, 700, 2048, 2049, 1 << 24})
            for (int64_t n_keys : {1, 64, 500, 9000, 131072, 3 << 24}) {
              if (hq % g) continue;
              const QueryBlock q{batch, hq, hq / g, d, n_q, n_keys};
              const int most = plan_key_split(batch, hq, n_q, n_keys, 0).n_splits;
              for (int req : {0, 1, 3, 40, 1000})
                for (int fits : {1, 2, 11, most}) {
                  if (fits > most || (req > 0 && fits > 1)) continue;
                  const QueryPlan plan = choose_query_plan(q, req, fits);
                  const KeySplit ks = plan.split, asked = key_split_of(req, key_tiles(n_keys));
                  EXPECT(query_kernel_takes(plan.kernel, q) && (plan.kernel == QueryKernel::kPerHead || n_q <= kQueryMaxTokens));
                  EXPECT(plan.kernel != QueryKernel::kWave || n_q * g <= kQueryWaveRows);
                  EXPECT(req == 0 ? ks.n_splits <= fits : ks.n_splits == asked.n_splits && ks.tiles_per_split == asked.tiles_per_split);
                  EXPECT(ks.n_splits >= 1 && (int64_t)ks.n_splits * ks.tiles_per_split >= key_tiles(n_keys));
                  EXPECT((int64_t)(ks.n_splits - 1) * ks.tiles_per_split < key_tiles(n_keys));
                }
            }
  // the launches of tests/test_gpu_packed_query.py
  struct { QueryKernel kernel; int ranges; QueryBlock q; int requested; } plans[] = {
      {QueryKernel::kWave, 2, {1, 9, 1, 64, 2, 1007}, 2},          {QueryKernel::kWave, 1, {1, 16, 1, 64, 2, 449}, 0},
      {QueryKernel::kWave, 3, {3, 16, 1, 64, 2, 5001}, 3},         {QueryKernel::kWave, 3, {4, 28, 4, 128, 4, 1344}, 3},
      {QueryKernel::kWave, 1, {48, 28, 4, 128, 4, 1344}, 0},       {QueryKernel::kWave, 8, {24, 1, 1, 64, 1, 1500}, 0},
      {QueryKernel::kWave, 21, {12, 32, 1, 128, 1, 9001}, 0},      {QueryKernel::kWave, 157, {1, 2, 1, 64, 1, 40001}, 0},
      {QueryKernel::kPacked128, 1, {48, 8, 1, 128, 2, 64}, 0},     {QueryKernel::kPacked128, 3, {16, 7, 1, 128, 1, 134}, 3},
      {QueryKernel::kPacked128, 2, {12, 11, 1, 128, 3, 320}, 2},   {QueryKernel::kPacked128, 4, {6, 16, 1, 128, 8, 908}, 4},
      {QueryKernel::kPacked128, 6, {3, 4, 4, 128, 5, 712}, 0},     {QueryKernel::kPacked128, 3, {8, 6, 2, 128, 129, 469}, 3},
      {QueryKernel::kPacked128, 3, {8, 8, 1, 64, 300, 640}, 3},    {QueryKernel::kPacked128, 1, {24, 16, 1, 64, 129, 329}, 0},
      {QueryKernel::kPacked256, 3, {6, 16, 1, 128, 129, 2000}, 3}, {QueryKernel::kPacked256, 1, {40, 7, 1, 128, 150, 700}, 0},
      {QueryKernel::kPacked256, 3, {8, 8, 1, 64, 257, 12000}, 3},
      {QueryKernel::kPerHead, 6, {2, 2, 1, 64, 2049, 2249}, 7},    {QueryKernel::kPerHead, 2, {1, 8, 2, 128, 2100, 1000}, 2},
      {QueryKernel::kPerHead, 4, {1, 12, 2, 128, 2100, 3640}, 4},
      // ... with peaked logits
      {QueryKernel::kWave, 3, {1, 16, 1, 64, 1, 5000}, 3},         {QueryKernel::kWave, 2, {1, 9, 1, 64, 2, 1005}, 2},
      {QueryKernel::kPacked128, 4, {6, 16, 1, 128, 8, 900}, 4},    {QueryKernel::kPacked128, 3, {8, 8, 1, 64, 300, 340}, 3}};
  for (const auto& c : plans) {
    const int most = plan_key_split(c.q.batch, c.q.n_q_heads, c.q.n_q, c.q.n_keys, 0).n_splits;
    const QueryPlan plan = choose_query_plan(c.q, c.requested, c.requested > 0 ? c.requested : most);
    EXPECT(plan.kernel == c.kernel && plan.split.n_splits == c.ranges);
  }
  EXPECT(attention_rows(128, 4, 1, 8, 2100, 1000, false, 2) == 256 && attention_rows(128, 6, 1, 12, 2100, 1540, true, 4) == 256);
  {  // measured shapes: one range goes through the packed kernels too, and a workgroup per head stays where it is faster
    const QueryPlan steps = choose_query_plan({120, 16, 2, 128, 1, 1402}, 0, 4), ragged = choose_query_plan({126, 2, 1, 64, 78, 26528}, 0, 4);
    EXPECT(steps.kernel != QueryKernel::kPerHead && ragged.kernel == QueryKernel::kPacked128 && ragged.split.n_splits > 1);
    EXPECT(choose_query_plan({1, 16, 1, 128, 603, 20814}, 6, 6).kernel == QueryKernel::kPerHead);
    const QueryPlan decode = choose_query_plan({1, 16, 2, 128, 1, 133121}, 0, 256), block = choose_query_plan({1, 16, 2, 128, 64, 16512}, 0, 64);
    EXPECT(decode.kernel == QueryKernel::kWave && decode.split.n_splits >= 64);
    EXPECT(block.kernel == QueryKernel::kPacked128 && block.split.n_splits >= 16);
  }
  for (int64_t L = 1; L <= ((int64_t)1 << 24); L = L * 5 + 3)
    for (int64_t l_p = 0; l_p <= L; l_p = l_p * 7 + 1) {
      const CompressWorkspace w1 = plan_compress_workspace(1, 2, 128, L, l_p), w3 = plan_compress_workspace(3, 2, 128, L, l_p);
      EXPECT(w1.total % 256 == 0 && w1.scores_off % 256 == 0 && w1.qbar_off < w1.scores_off && w1.scores_off < w1.total);
      EXPECT(w1.scores_off + (size_t)2 * L * 8 <= w1.sort_keys_off && w1.sort_keys_off <= w1.sort_idx_off && w1.sort_idx_off <= w1.total);
      EXPECT(w1.n_sort >= l_p && (w1.n_sort & (w1.n_sort - 1)) == 0 && w3.total >= w1.total);
      EXPECT(compress_workspace_bytes_checked(1, 2, 128, L, l_p) == w1.total);
    }
  // attention-mass pass: resident only where the probe rows fit, with blocks for every key; measured shapes on both sides
  for (int d : {64, 128})
    for (int r_pad = 32; r_pad <= 2048; r_pad += 32)
      for (int64_t L = 1; L <= ((int64_t)1 << 24); L = L * 3 + 1)
        for (int64_t heads : {1, 7, 192, 65535 * 16}) {
          const MassPlan m = plan_mass(d, r_pad, L, heads);
          EXPECT(m.waves == 0 || ((m.waves == 4 || m.waves == 8) && m.n_blocks >= 1 && m.n_blocks <= 8));
          EXPECT(m.waves == 0 || (r_pad * d * 2 >= kMassMinProbeBytes && r_pad * d * 2 <= kMassMaxProbeBytes));
        }
  EXPECT(plan_mass(64, 576, 20 * 64, 100).waves == 0 && plan_mass(128, 256, 1575, 192).waves == 0 && plan_mass(128, 512, 1266, 126).waves == 0);
  // ... and those of tests/test_gpu_mass_shapes.py
  EXPECT(plan_mass(128, 512, 63, 1).waves == 4 && plan_mass(128, 512, 65, 1).waves == 4 && plan_mass(128, 192, 70001, 1).waves == 8);
  EXPECT(plan_mass(64, 384, 70001, 1).waves != 0 && plan_mass(64, 1024, 129, 1).waves == 4 && plan_mass(128, 512, 9000, 34).n_blocks == 3);
  EXPECT(plan_mass(128, 512, 16384, 32).waves == 8 && plan_mass(128, 448, 16384, 4).waves != 0);
  // selection shared by several workgroups: few heads, resident scores, room for the candidates
  auto shared = [](int heads, int64_t L, int64_t l_p) { return share_selection(heads, L, l_p, plan_compress_workspace(1, heads, 64, L, l_p)); };
  EXPECT(shared(2, 16384, 1024) && shared(8, 16384, 6000) && shared(1, 16384, 8064) && shared(1, 8192, 8192) && shared(2, 700, 64));
  EXPECT(!shared(9, 16384, 1024) && !shared(2, 16385, 1024) && !shared(2, 16384, 0) && !shared(1, 16384, 8193));
  EXPECT(!shared(1, 16384, 8192) && !shared(2, 9000, 8100) && !shared(2, 2000, 2000) && !shared(1, 1, 1));
  // pooled-query partition: about 64 probe rows per range, at most kPoolSplitMax, no more ranges than fill the chip
  // twice over; and the partial sums of every partition fit the region the workspace plan reserves for them
  EXPECT(pool_splits(512, 2) == 8 && pool_splits(512, 192) == 2 && pool_splits(512, 1000) == 1 && pool_splits(10, 1) == 1);
  EXPECT(pool_splits(100000, 1) == kPoolSplitMax && pool_splits(1, 1) == 1 && pool_splits(130, 4) == 3);
  for (int batch : {1, 2, 7, 96, 300})
    for (int hkv : {1, 2, 4, 8})
      for (int64_t rows : {1, 63, 64, 65, 512, 4096}) {
        const int n = pool_splits(rows, (int64_t)batch * hkv);
        EXPECT(n >= 1 && n <= kPoolSplitMax);
        const CompressWorkspace w = plan_compress_workspace(batch, hkv, 128, 1024, 16);
        EXPECT(w.qbar_off + (size_t)batch * hkv * n * 128 * sizeof(double) <= w.scores_off);
      }
  EXPECT(compress_workspace_bytes_checked(1, 2, 128, 0, 0) == 0 && compress_workspace_bytes_checked(1, 2, 128, 8, 9) == 0);
  EXPECT(compress_workspace_bytes_checked(0, 2, 128, 8, 1) == 0 && compress_workspace_bytes_checked(1, 2, 100, 8, 1) == 0);
  if (failures) return 1;
  std::printf("host validation OK\n");
  return 0;
}
