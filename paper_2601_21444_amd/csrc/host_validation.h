// Host-side argument validation and planning of the C ABI (include/apbv.h).  Plain C++ with no HIP types, so that
// the rejection paths can be compiled alone with the host compiler and its sanitizers (tests/host/).  Everything
// here runs before any launch: a call that fails one of these checks enqueues nothing.
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <cmath>
#include <initializer_list>
#include "apbv.h"

namespace apbv {

constexpr int64_t kMaxTokens = (int64_t)1 << 24;
constexpr int kMaxKeySplits = 256;
constexpr int kAttnKeyTile = 64;            // keys per tile of the attention kernel
constexpr int kAttnQueryTile = 256;         // query rows per workgroup
constexpr int kAttnNarrowQueryTile = 64;    // ... of the variant used for query blocks of at most
constexpr int kAttnNarrowMaxRows = 128;     // this many rows
constexpr int kQueryMaxTokens = 2048;       // query blocks whose launch may pack the heads of a KV group into its rows
constexpr int kQueryShortTokens = 128;      // ... sized for tiles of kQueryShortRows rows up to here, of kAttnQueryTile above
constexpr int kQueryShortRows = 128;
constexpr int kQueryWaveRows = 32;          // rows per KV head a single wave takes (the waves then split the keys)

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }
inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline size_t align256(size_t x) { return align_up(x, 256); }

// A view is acceptable if it is empty, or has a 16-byte aligned pointer and strides that keep every
// (token, head) row 16-byte aligned and non-overlapping along the head dimension.
inline apbv_status check_view(const apbv_tensor& t, int heads, int d, int batch, bool may_be_empty) {
  if (t.tokens < 0 || t.tokens > kMaxTokens) return APBV_ERR_SHAPE;
  if (t.tokens == 0) return may_be_empty ? APBV_OK : APBV_ERR_SHAPE;
  if (t.ptr == nullptr) return APBV_ERR_NULL;
  if (!aligned(t.ptr, 16)) return APBV_ERR_SHAPE;
  if (t.stride_token < d || t.stride_token % 8) return APBV_ERR_SHAPE;
  if (t.stride_token >= kMaxTokens) return APBV_ERR_UNSUPPORTED;       // the kernels keep row offsets of a 64-row tile in 32 bits
  if (heads > 1 && (t.stride_head < d || t.stride_head % 8)) return APBV_ERR_SHAPE;
  if (batch > 1 && (t.stride_batch <= 0 || t.stride_batch % 8)) return APBV_ERR_SHAPE;
  return APBV_OK;
}

inline apbv_status check_heads(int batch, int hq, int hkv, int d) {
  if (batch < 1 || hq < 1 || hkv < 1 || batch > 65535 || hq > 65535) return APBV_ERR_SHAPE;
  if (hq % hkv) return APBV_ERR_SHAPE;
  if (d != 64 && d != 128) return APBV_ERR_UNSUPPORTED;
  return APBV_OK;
}

inline bool valid_reducer(int r) { return r == APBV_REDUCE_SUM || r == APBV_REDUCE_MAX || r == APBV_REDUCE_SOFTMAX_SUM; }

// Arguments of the attention entry points (Eq. 4 / Eq. 5).
inline apbv_status validate_attention(int batch, int n_q_heads, int n_kv_heads, int head_dim, const apbv_tensor& q_local,
                                      const apbv_tensor& k_anchor, const apbv_tensor& v_anchor, const apbv_tensor& k_pass,
                                      const apbv_tensor& v_pass, const apbv_tensor& k_local, const apbv_tensor& v_local,
                                      float softmax_scale, const void* out, const float* lse_out) {
  apbv_status st = check_heads(batch, n_q_heads, n_kv_heads, head_dim);
  if (st != APBV_OK) return st;
  if ((st = check_view(q_local, n_q_heads, head_dim, batch, false)) != APBV_OK) return st;
  if ((st = check_view(k_local, n_kv_heads, head_dim, batch, true)) != APBV_OK) return st;
  if ((st = check_view(v_local, n_kv_heads, head_dim, batch, true)) != APBV_OK) return st;
  if ((st = check_view(k_anchor, n_kv_heads, head_dim, batch, true)) != APBV_OK) return st;
  if ((st = check_view(v_anchor, n_kv_heads, head_dim, batch, true)) != APBV_OK) return st;
  if ((st = check_view(k_pass, n_kv_heads, head_dim, batch, true)) != APBV_OK) return st;
  if ((st = check_view(v_pass, n_kv_heads, head_dim, batch, true)) != APBV_OK) return st;
  if ((k_local.tokens != 0 && q_local.tokens != k_local.tokens) || v_local.tokens != k_local.tokens) return APBV_ERR_SHAPE;
  if (v_anchor.tokens != k_anchor.tokens || v_pass.tokens != k_pass.tokens) return APBV_ERR_SHAPE;
  if (k_anchor.tokens + k_pass.tokens + k_local.tokens < 1) return APBV_ERR_SHAPE;       // every query needs a key
  if (!(softmax_scale > 0.0f) || !std::isfinite(softmax_scale)) return APBV_ERR_SHAPE;
  if (out == nullptr) return APBV_ERR_NULL;
  if (!aligned(out, 16) || (lse_out != nullptr && !aligned(lse_out, 4))) return APBV_ERR_SHAPE;
  return APBV_OK;
}

// Arguments of the compression entry points (Sec. 3.3 / Alg. 1) other than the workspace.
inline apbv_status validate_compress(int reducer, float softmax_scale, int batch, int n_q_heads, int n_kv_heads, int head_dim,
                                     const apbv_tensor& q_probe, const apbv_tensor& k_local, const apbv_tensor& v_local,
                                     int64_t l_p, const int32_t* idx_out, const void* k_c_out, const void* v_c_out,
                                     const double* scores_out) {
  apbv_status st = check_heads(batch, n_q_heads, n_kv_heads, head_dim);
  if (st != APBV_OK) return st;
  if ((st = check_view(q_probe, n_q_heads, head_dim, batch, false)) != APBV_OK) return st;
  if ((st = check_view(k_local, n_kv_heads, head_dim, batch, false)) != APBV_OK) return st;
  if ((st = check_view(v_local, n_kv_heads, head_dim, batch, false)) != APBV_OK) return st;
  if (v_local.tokens != k_local.tokens) return APBV_ERR_SHAPE;
  if (l_p < 0 || l_p > k_local.tokens) return APBV_ERR_SHAPE;
  if (l_p > 0) {
    if (idx_out == nullptr || k_c_out == nullptr || v_c_out == nullptr) return APBV_ERR_NULL;
    if (!aligned(k_c_out, 16) || !aligned(v_c_out, 16) || !aligned(idx_out, 4)) return APBV_ERR_SHAPE;
  }
  if (scores_out != nullptr && !aligned(scores_out, 8)) return APBV_ERR_SHAPE;
  if (!valid_reducer(reducer)) return APBV_ERR_SHAPE;
  if (q_probe.tokens * (n_q_heads / n_kv_heads) > (int64_t)1 << 24) return APBV_ERR_UNSUPPORTED;   // rows of the score matrix per KV head
  if (reducer == APBV_REDUCE_SOFTMAX_SUM && (!(softmax_scale > 0.0f) || !std::isfinite(softmax_scale))) return APBV_ERR_SHAPE;
  return APBV_OK;
}

inline apbv_status validate_merge(int n_parts, int64_t rows, int n_q_heads, int head_dim, const void* parts_out,
                                  int64_t part_stride_out, const float* parts_lse, int64_t part_stride_lse,
                                  const void* out, const float* lse_out) {
  if (n_parts < 1 || n_parts > 65536 || rows < 1 || rows > kMaxTokens || n_q_heads < 1 || n_q_heads > 65535)
    return APBV_ERR_SHAPE;
  if (head_dim != 64 && head_dim != 128) return APBV_ERR_UNSUPPORTED;
  if (parts_out == nullptr || parts_lse == nullptr || out == nullptr) return APBV_ERR_NULL;
  if (!aligned(parts_out, 16) || !aligned(out, 16) || !aligned(parts_lse, 4) || (lse_out != nullptr && !aligned(lse_out, 4)))
    return APBV_ERR_SHAPE;
  if (n_parts > 1) {
    if (part_stride_out < rows * n_q_heads * head_dim || part_stride_out % 8) return APBV_ERR_SHAPE;
    if (part_stride_lse < rows * n_q_heads) return APBV_ERR_SHAPE;
  }
  return APBV_OK;
}

// ---- rows per workgroup of the attention kernel (64, 128 or 256): a question of speed only, every row's arithmetic is the
// same.  Smaller workgroups spread over more compute units, and where two share one the start and the end of one run
// beside the other's keys; but they read K and V more often, and one that is alone on its unit takes 0.64 of the time of
// two, not half.  The rule is drawn from 2260 measured launches (heads, batches, 129 to 16384 rows, 0 to 33000 visible
// keys): against 256 rows always it is more than 1.5 % slower in 12 of them (at most 15 %) and on average 10 % (head_dim
// 128) and 22 % (64) faster, 1 % behind the best size of every launch.  Examples (us, 256 / 128 rows, d 128):
//   16 heads x 2048 rows behind 8704 keys  245 / 181 (a workgroup per unit)    x 4096 rows, no more keys  100 / 87
//   16 x 4096 behind 32768  981 / 1030 (one full round either way)             32 x 3899 rows  123 / 130 (two full rounds)
//   5 x 32 heads, 233 rows over 1829 keys  52 / 56 (320 of 128 rows: some units get two, the others one)
//   68 x 16 heads of their own K/V, 1752 rows behind 827 keys  1909 / 2959 (K/V come from HBM each time, not from a cache)
struct AttentionTiles {          // the row tiles of a launch: how many, and the keys the heaviest and the lightest see
  double n = 0, k_max = 0, k_min = 0, key_sum = 0;
};
inline void add_attention_tiles(AttentionTiles& t, int rows, double heads, int64_t n_rows, int64_t n_vis, bool causal, int n_splits = 1) {
  const double tiles = (double)((n_rows + rows - 1) / rows) * heads * n_splits;
  const double hi = (double)(n_vis + (causal ? n_rows : 0)) / n_splits;
  const double lo = (double)(n_vis + (causal ? (n_rows < rows ? n_rows : rows) : 0)) / n_splits;
  t.k_max = t.n > 0 && t.k_max > hi ? t.k_max : hi;
  t.k_min = t.n > 0 && t.k_min < lo ? t.k_min : lo;
  t.n += tiles;
  t.key_sum += tiles * (hi + lo) / 2;
}
// A workgroup that sees k keys takes fixed + per_key * k us when its unit is full (per_unit workgroups), alone_* when it
// has the unit to itself; launches of more than two rounds end unevenly by a share of a lightest workgroup's time.
struct AttentionCost {
  int per_unit;
  double fixed, per_key, alone_fixed, alone_per_key, uneven;
};
inline AttentionCost attention_cost(int head_dim, int rows) {
  if (head_dim == 64) return {1, 5.8, 0.0178, 5.8, 0.0178, 0};           // 256 rows
  if (rows == 128) return {2, 8.4, 0.0258, 7.2, 0.0152, 0};
  return {1, 8.9, 0.0235, 8.9, 0.0235, 0.23};
}
// Time of a launch, heaviest first on 256 units: two whole rounds give every slot the same (its heavy item first, a light
// one second); what is left over is a round of its own, or two.  Tiles are taken to spread evenly between k_min and k_max
// keys.  Within 8 % of the measured launches.
inline double attention_makespan(const AttentionCost& c, const AttentionTiles& w) {
  const double units = 256, slots = units * c.per_unit;
  auto shared = [&](double k) { return c.fixed + c.per_key * k; };
  auto alone = [&](double k) { return c.alone_fixed + c.alone_per_key * k; };
  auto larger = [](double a, double b) { return a > b ? a : b; };
  const double pairs = std::floor(w.n / (2 * slots)), done = 2 * slots * pairs, m = w.n - done;
  const double k1 = w.k_max - done / w.n * (w.k_max - w.k_min);
  const double t = 2 * pairs * shared((w.k_max + k1) / 2) + (w.n > 2 * slots ? c.uneven * shared(w.k_min) : 0);
  if (m <= 0) return t;
  if (m <= units) return t + alone(k1);
  const double k2 = k1 - units / m * (k1 - w.k_min);           // the heaviest unit's second workgroup
  const double one = c.per_unit == 1 ? shared(k1) : larger(shared(k2) + c.alone_per_key * (k1 - k2), alone(k1));
  if (m <= slots) return t + one;
  const double k3 = k1 - slots / m * (k1 - w.k_min);           // the first of a second round
  double second = shared(k3);
  if (m <= slots + units && c.per_unit > 1) {                  // alone on its unit, once those beside it have finished
    const double busy = shared(k1) - shared(k3) < shared(k3) ? shared(k1) - shared(k3) : shared(k3);
    second = alone(k3) + (1 - alone(k3) / shared(k3)) * busy;
  }
  return t + larger(one, shared(k3) + second);
}
// Time of the memory traffic: Q and O once, K and V once per row tile (the heads of a group together, through their XCD's
// L2) as far as the launch's tensors exceed the 256 MB last-level cache, at the 4 TB/s such launches reach.
inline double attention_traffic(int head_dim, int group, const AttentionTiles& w, double kv_bytes, double qo_bytes) {
  const double total = kv_bytes + qo_bytes, missed = total > 256e6 ? 1 - 256e6 / total : 0;
  return (qo_bytes + missed * w.key_sum / group * head_dim * 4) / 4e6;
}
// tiles[]: of the launch cut into 64, 128 and 256 rows; kv_heads: KV heads, batch items and key ranges that a row tile of
// the launch belongs to one of.
//   head_dim 64   128 (three fit a unit, one of 256 rows).  Its two exceptions, 64 rows for few workgroups and 256 where these
//                 are one round and 128 two with the second tile half empty, lie where launches share blocks
//                 (attention_shares_blocks): no launch takes them any more, only query_estimate
//   head_dim 128  by the estimates up to two rounds of 256 rows, whose spread they get right; beyond, and for the shortest
//                 keys, by the keys alone: the fixed cost covered against the 4 to 10 % slower loop of 128 rows.  But 256
//                 rows if the row tiles of a head share nothing with other heads and are not kept on one XCD (a number
//                 of heads that eight does not divide, nor it eight): 84 heads x 3031 rows 211 / 248, 96 x 2874 325 / 294
//   both          256 rows where the traffic of 128 would take longer; the tiles of many heads pass through the caches
//                 without meeting another tile of theirs, those of a few heads run at the same time
inline int attention_rows(int head_dim, int group, double kv_heads, const AttentionTiles (&tiles)[3], double kv_bytes, double qo_bytes,
                          bool may_be_64) {
  const AttentionTiles &t64 = tiles[0], &t128 = tiles[1], &t256 = tiles[2];
  const double time = attention_makespan(attention_cost(head_dim, 256), t256), keys = t256.key_sum / t256.n;
  const bool scattered = group == 1 && std::fmod(kv_heads, 8) != 0 && std::fmod(8, kv_heads) != 0 && kv_bytes > 32e6;
  if (head_dim == 64) {
    if (may_be_64 && t256.n <= 64) return 64;
    if (t256.n <= 256 && t128.n > 256 && t128.n == 2 * t256.n && t64.n == 3 * t256.n) return 256;
  } else if (t256.n > 512 ? keys > 2280 || scattered : keys > 300 && attention_makespan(attention_cost(head_dim, 128), t128) > 0.98 * time) {
    return 256;
  }
  const double read = attention_traffic(head_dim, group, t256, kv_bytes, qo_bytes), least = time > read ? time : read;
  const double reached = kv_heads * group >= 512 ? 0.85 : 1.2;
  if (kv_bytes > 128e6 && attention_traffic(head_dim, group, t128, kv_bytes, qo_bytes) > reached * least) return 256;
  return 128;
}
// Whether a launch takes 64-row workgroups of four waves, one 16-row block each (kOwn = 1 in attention.hip), instead: up to a
// workgroup per unit always, with head_dim 64 (four fit a unit) up to three, and with head_dim 128 up to two where the
// estimates say so.  Beyond, every wave's own reads of K and V from LDS cost more than the shorter steps save.  The lines, and the
// estimate of such a launch, were drawn when two waves formed the S^T of 32 rows between them, and lie low for the kernel as it
// is (us, 64 / 128 / 256 rows: 16 heads of 128 x 1024 rows behind 224 keys 18.2 / 26.2 / 36.3, x 2048 behind 704 41.0 / 49.2 / 68.9;
// 28 x 1500 behind 400 40.4 / 38.4 / 51.8).  Of 740 measured launches 470 take it, 1.32 times as fast as the better of 128
// and 256 rows on average, 0.996 at least.  With head_dim 128 the 47 others of 257 to 512 workgroups would be 1.16 times as
// fast, 0.98 at least, 113 of 513 to 800 1.02, 0.84 at least; with 64 75 of 769 to 1100 1.07, 0.92 at least, 31 beyond 0.99.  Blocks of
// at most kAttnNarrowMaxRows rows, which take 64 rows either way, up to 256 workgroups, or 512 with head_dim 64, where two waves
// take 1.23 times as long (107 launches, 1.11 at least; 24 of 513 to 800 1.04, 0.94 at least).
inline bool attention_shares_blocks(int head_dim, const AttentionTiles (&tiles)[3]) {
  const AttentionTiles& t = tiles[0];
  if (head_dim == 64) return t.n <= 768;
  if (t.n <= 256) return true;
  const double t128 = attention_makespan(attention_cost(128, 128), tiles[1]), t256 = attention_makespan(attention_cost(128, 256), tiles[2]);
  return t.n <= 512 && attention_makespan(AttentionCost{2, 7.2, 0.018, 6.4, 0.0122, 0}, t) < (t128 < t256 ? t128 : t256);
}
inline bool attention_shares_blocks(int head_dim, int batch, int n_q_heads, int64_t n_rows, int64_t n_vis, bool causal, int n_splits) {
  AttentionTiles tiles[3];
  for (int i = 0; i < 3; ++i) add_attention_tiles(tiles[i], 64 << i, (double)batch * n_q_heads, n_rows, n_vis, causal, n_splits);
  if (n_rows <= kAttnNarrowMaxRows) return tiles[0].n <= (head_dim == 64 ? 512 : 256);
  return attention_shares_blocks(head_dim, tiles);
}
// One launch of batch * n_q_heads heads and n_splits key ranges, all of n_rows queries.
inline int attention_rows(int head_dim, int group, int batch, int n_q_heads, int64_t n_rows, int64_t n_vis, bool causal, int n_splits) {
  AttentionTiles tiles[3];
  const double heads = (double)batch * n_q_heads, row = heads * head_dim * 4;
  for (int i = 0; i < 3; ++i) add_attention_tiles(tiles[i], 64 << i, heads, n_rows, n_vis, causal, n_splits);
  return attention_rows(head_dim, group, heads / group * n_splits, tiles, row / group * (double)(n_vis + (causal ? n_rows : 0)),
                        row * (double)n_rows, true);
}

// The workgroups of a launch: 64 rows by four waves of 16, or in more workgroups than these are for (launch_host_attention); 128 or 256 rows.
enum class AttentionKernel { kShared64, kNarrow64, k128, k256 };
// One launch of batch * n_q_heads heads and n_splits key ranges, all of n_rows queries.
inline AttentionKernel attention_kernel(int head_dim, int group, int batch, int n_q_heads, int64_t n_rows, int64_t n_vis, bool causal, int n_splits) {
  if (attention_shares_blocks(head_dim, batch, n_q_heads, n_rows, n_vis, causal, n_splits)) return AttentionKernel::kShared64;
  // (a block of at most kAttnNarrowMaxRows rows is mostly padding in anything but 64-row workgroups)
  if (n_rows <= kAttnNarrowMaxRows) return AttentionKernel::kNarrow64;
  // (64 of attention_rows are for launches that share blocks)
  return attention_rows(head_dim, group, batch, n_q_heads, n_rows, n_vis, causal, n_splits) == kAttnQueryTile ? AttentionKernel::k256 : AttentionKernel::k128;
}
// One launch of n problems with rows[m] queries behind n_vis[m] keys, each with its causal segment.
inline AttentionKernel attention_group_kernel(int head_dim, int n_q_heads, int n_kv_heads, int n, const int64_t* n_vis, const int64_t* rows) {
  AttentionTiles tiles[3];
  double kv_bytes = 0, qo_bytes = 0;
  for (int m = 0; m < n; ++m) {
    for (int i = 0; i < 3; ++i) add_attention_tiles(tiles[i], 64 << i, n_q_heads, rows[m], n_vis[m], true);
    kv_bytes += (double)(n_vis[m] + rows[m]) * n_kv_heads * head_dim * 4;
    qo_bytes += (double)rows[m] * n_q_heads * head_dim * 4;
  }
  if (attention_shares_blocks(head_dim, tiles)) return AttentionKernel::kShared64;
  const int tile = attention_rows(head_dim, n_q_heads / n_kv_heads, n_kv_heads, tiles, kv_bytes, qo_bytes, false);
  return tile == kAttnQueryTile ? AttentionKernel::k256 : AttentionKernel::k128;
}

// Lanes of the merge kernel that share one item (a 16-byte chunk of the output).  A lane that holds all its parts in
// registers has their loads in flight at once, so with few items more lanes are faster; with many items the chip is full
// anyway, and lanes reading one 16-byte piece of each part use a fraction of what a load fetches.  Measured (us; lanes
// 1 / 2 / 4 / 8 / 16 / 64, items of head_dim 128; one lane holding eight parts):
//   6 parts    4096 items  3.5 / 2.4 / 2.5 / 2.3 / 2.4 / 3.7     1048576  22 / 21 / 25 / 43 / 80 / 438
//   16         4096        6.1 / 3.2 / 2.6 / 2.5 / 2.4 / 3.7     1048576  60 / 54 / 46 / 54 / 90 / 442
//   64         1024        18 / 5.9 / 4.9 / 3.9 / 3.0 / 2.6      65536    41 / 14 / 15 / 18 / 17 / 34
//   200        1024        53 / 14 / 11 / 7.7 / 6.4 / 3.1        65536    126 / 40 / 40 / 47 / 68 / 91
//   (head_dim 64) 64 parts, 131072 items: 8 lanes 32, 4 lanes 43
// A launch has fewer than 2^32 threads: beyond 2^28 items one lane takes an item.
constexpr int kMergePartsPerLane = 4;
inline int64_t merge_items(int batch, int64_t rows, int n_q_heads, int head_dim) {
  return (int64_t)batch * rows * n_q_heads * (head_dim / 8);
}
inline int merge_lanes(int64_t items, int n_parts) {
  if (items > (int64_t)1 << 28 || n_parts <= kMergePartsPerLane) return 1;
  if (n_parts <= 2 * kMergePartsPerLane) return items <= 65536 ? 2 : 1;
  if (n_parts <= 4 * kMergePartsPerLane) return 4;
  return items <= 1024 ? 64 : (items <= 4096 ? 16 : 8);
}

// Key split of the query-block attention: n_splits ranges of tiles_per_split 64-key tiles; ranges are equal and none
// is empty.
struct KeySplit {
  int n_splits, tiles_per_split;
};
inline KeySplit key_split_of(int64_t s, int64_t n_tiles) {
  s = s < n_tiles ? s : n_tiles;
  s = s < kMaxKeySplits ? s : kMaxKeySplits;
  s = s > 1 ? s : 1;
  const int64_t per = (n_tiles + s - 1) / s;
  KeySplit ks;
  ks.tiles_per_split = (int)per;
  ks.n_splits = (int)((n_tiles + per - 1) / per);
  return ks;
}
inline int64_t key_tiles(int64_t n_keys) { return (n_keys + kAttnKeyTile - 1) / kAttnKeyTile; }

// With one tile of query rows per query head: about two workgroups per compute unit, ranges of at least four tiles.
// Blocks longer than kQueryMaxTokens are split like this; a call with a shorter one is refused if its workspace does not
// hold the ranges of this split.
inline KeySplit per_head_key_split(int batch, int n_q_heads, int64_t n_q, int64_t n_keys) {
  const int64_t tile = n_q <= kAttnNarrowMaxRows ? kAttnNarrowQueryTile : kAttnQueryTile;
  const int64_t n_wg = (n_q + tile - 1) / tile * n_q_heads * batch;
  const int64_t s = (512 + n_wg - 1) / n_wg;
  const int64_t cap = key_tiles(n_keys) / 4 > 1 ? key_tiles(n_keys) / 4 : 1;
  return key_split_of(s < cap ? s : cap, key_tiles(n_keys));
}

// The split a workspace is sized for: as requested, or (0) the most ranges choose_query_plan() takes whatever the
// number of KV heads, which the size query is not told.
inline KeySplit plan_key_split(int batch, int n_q_heads, int64_t n_q, int64_t n_keys, int requested) {
  if (requested > 0) return key_split_of(requested, key_tiles(n_keys));
  if (n_q > kQueryMaxTokens) return per_head_key_split(batch, n_q_heads, n_q, n_keys);
  const int64_t rows = n_q <= kQueryShortTokens ? kQueryShortRows : kAttnQueryTile;
  const int64_t n_wg = (n_q * n_q_heads + rows - 1) / rows * batch;      // at least: with more KV heads there are more
  const int64_t s = (512 + n_wg - 1) / n_wg;
  const int64_t cap = key_tiles(n_keys) / 2 > 1 ? key_tiles(n_keys) / 2 : 1;
  return key_split_of(s < cap ? s : cap, key_tiles(n_keys));
}

// ---- kernel and ranges of a block of at most kQueryMaxTokens queries, from the time each would take.  There are four:
// a workgroup per query head (attention.hip's own launch), workgroups of 128 or 256 rows packed per KV head, and a wave per
// range for at most kQueryWaveRows packed rows.  Which is fastest turns on how many heads share K/V, how many workgroups
// there are and how many keys each has (us: per query head / packed 128 / wave):
//   120 decoding steps, 16 / 2 heads of 128, 1402 keys, one range      123 / 31.8 / 34.8
//   5 steps, 28 / 4 heads of 128, 17629 keys, 16 ranges                120 / 41.0 / 36.6
//   32 blocks of 7 queries, 16 / 16 heads of 64, 2194 keys, one range  47.9 / 50.1 / 54.4
//   126 blocks of 78, 2 / 1 heads of 64, 26528 keys, one range         482 / 358, four 348 / 266 (two of a workgroup per head 289)
//   603 queries, 16 / 1 heads of 128, 20814 keys, six ranges           115 / 161 (six ranges fill six XCDs of eight)
enum class QueryKernel { kPerHead, kPacked128, kPacked256, kWave };
struct QueryPlan {
  QueryKernel kernel;
  KeySplit split;
};
// Times in us, fitted to 18000 launches of 800 shapes (1 to 2048 queries, batches to 128, 64 to 200000 keys; then within 9 %)
// while the packed workgroups used 16x16x32 matrix instructions and no blocks were shared.  Packed workgroups have become up
// to 14 % faster, a workgroup per head with shared blocks up to 20 %: of 320 shapes drawn over these ranges the plans chosen
// now take 1.03 times the estimate in the median, 0.91 to 1.26 between the 5th and 95th in 100 (medians: a wave per range
// 1.04, packed rows in 128 1.02, in 256 1.15, a workgroup per head with shared blocks 1.02, of 128 rows 1.22).  The order of
// the plans has changed less: constants refitted to 70000 launches chose 0.5 % better on average and worse by more than 5 % in 325 of 7702
// shapes, so these stay.
// A workgroup with k keys takes alone + alone_per_key * k on a unit of its own, and every further one on the busiest unit
// adds more + more_per_key * k, whether it runs beside the others or after them.
struct QueryCost {
  double alone, alone_per_key, more, more_per_key;
};
inline QueryCost query_cost(QueryKernel kernel, int head_dim, int per_head_rows) {
  const bool wide = head_dim == 128;
  switch (kernel) {
    case QueryKernel::kWave: return wide ? QueryCost{7.4, 0.0103, 2.4, 0.0052} : QueryCost{6.0, 0.0029, 1.7, 0.0028};
    case QueryKernel::kPacked256: return wide ? QueryCost{9.2, 0.0225, 2.4, 0.0258} : QueryCost{6.6, 0.0175, 1.9, 0.0187};
    case QueryKernel::kPerHead:
      if (per_head_rows == 256) return query_cost(QueryKernel::kPacked256, head_dim, 0);
      if (per_head_rows == 64) return wide ? QueryCost{5.7, 0.0168, 1.5, 0.0084} : QueryCost{4.7, 0.0111, 0.7, 0.0045};
      break;
    case QueryKernel::kPacked128: break;
  }
  return wide ? QueryCost{5.4, 0.0164, 1.3, 0.0116} : QueryCost{4.8, 0.0114, 0.9, 0.0064};
}
struct QueryBlock {
  int batch, n_q_heads, n_kv_heads, head_dim;
  int64_t n_q, n_keys;
};
inline bool query_kernel_takes(QueryKernel kernel, const QueryBlock& q) {
  const int64_t rows = q.n_q * (q.n_q_heads / q.n_kv_heads);
  if (kernel == QueryKernel::kPerHead) return true;
  if (q.n_q > kQueryMaxTokens) return false;
  return kernel == QueryKernel::kWave ? rows <= kQueryWaveRows : kernel == QueryKernel::kPacked128 || rows > kAttnQueryTile;
}
inline double query_estimate(QueryKernel kernel, const QueryBlock& q, const KeySplit& ks) {
  const int64_t rows = q.n_q * (q.n_q_heads / q.n_kv_heads), n_tiles = key_tiles(q.n_keys);
  const int group = q.n_q_heads / q.n_kv_heads;
  // Workgroups in whole rounds of eight XCDs: the row tiles of a range run on one of them, of a workgroup per query head
  // those of a KV head's group.
  // (A workgroup per query head of more than kAttnNarrowMaxRows queries counts as attention_rows cuts it, without the shared
  // blocks and after its own 64 rows: the launches that query_cost was fitted to.)
  int tile = kernel == QueryKernel::kPacked256 ? kAttnQueryTile : kQueryShortRows;
  if (kernel == QueryKernel::kPerHead)
    tile = q.n_q <= kAttnNarrowMaxRows ? kAttnNarrowQueryTile : attention_rows(q.head_dim, group, q.batch, q.n_q_heads, q.n_q, q.n_keys, false, ks.n_splits);
  const int64_t ranges = (int64_t)q.n_kv_heads * q.batch * ks.n_splits, tiles = ((kernel == QueryKernel::kPerHead ? q.n_q : rows) + tile - 1) / tile;
  const double n = kernel == QueryKernel::kPerHead ? (double)((ranges * tiles + 7) / 8 * 8 * group) : (double)((ranges + 7) / 8 * 8 * tiles);
  const QueryCost c = query_cost(kernel, q.head_dim, tile);
  const double keys = (double)ks.tiles_per_split * kAttnKeyTile, more = std::ceil(n / 256) - 1;
  const double compute = c.alone + c.alone_per_key * keys + more * (c.more + c.more_per_key * keys);
  // K and V at 5.5 TB/s, a little less with few waves to keep it busy; once, but by workgroups per head once per row tile if
  // the 256 MB cache does not hold them.  A smooth maximum of the two.
  const double kv = (double)q.batch * q.n_kv_heads * (double)n_tiles * kAttnKeyTile * q.head_dim * 4;
  const double reads = kernel == QueryKernel::kWave ? 1 + 6.5 / n : kernel == QueryKernel::kPerHead && kv > 256e6 ? (double)tiles : 1;
  const double memory = reads * kv / 5.5e6;
  const double both = compute * compute * compute * compute + memory * memory * memory * memory;
  const double parts = (double)ks.n_splits * q.batch * (double)q.n_q * q.n_q_heads * q.head_dim * 2;
  return std::sqrt(std::sqrt(both)) + (ks.n_splits > 1 ? 1.84 + parts * 0.6e-6 + 0.3 / 64 * ks.n_splits : 0);
}
// The fastest kernel and, unless `requested` ranges are asked for (>= 1), number of ranges up to most_splits.  As the
// estimates are no better than that, a workgroup per query head with its own split stays unless another plan promises 5 %,
// or with the ranges requested 10 %.  Of 1900 calls outside the fit 11 were 2 to 17 % slower than with a workgroup per head, its own
// split or the ranges requested; the mean was 0.67 of its time.
inline QueryPlan choose_query_plan(const QueryBlock& q, int requested, int64_t most_splits) {
  const int64_t n_tiles = key_tiles(q.n_keys);
  const KeySplit own = per_head_key_split(q.batch, q.n_q_heads, q.n_q, q.n_keys);
  QueryPlan best{QueryKernel::kPerHead, requested > 0 ? key_split_of(requested, n_tiles) : own.n_splits <= most_splits ? own : key_split_of(1, n_tiles)};
  double least = (requested > 0 ? 0.9 : 0.95) * query_estimate(best.kernel, q, best.split);
  for (QueryKernel kernel : {QueryKernel::kPerHead, QueryKernel::kPacked128, QueryKernel::kPacked256, QueryKernel::kWave}) {
    if (!query_kernel_takes(kernel, q)) continue;
    for (int64_t s = requested > 0 ? requested : 1;; s += s / 8 + 1) {       // (every count up to 8, then steps of about an eighth)
      if (requested <= 0 && s > most_splits) s = most_splits;
      const KeySplit ks = key_split_of(s, n_tiles);
      const double t = query_estimate(kernel, q, ks) * (kernel == QueryKernel::kPerHead ? 0.98 : 1.0);
      if (t < least) {
        least = t;
        best = {kernel, ks};
      }
      if (requested > 0 || s >= most_splits) break;
    }
  }
  return best;
}

// Workspace of one key range: its bf16 partial output and float32 log-sum-exps.
inline size_t key_range_bytes(int batch, int n_q_heads, int head_dim, int64_t n_q) {
  const size_t rows = (size_t)batch * (size_t)n_q * (size_t)n_q_heads;
  return align256(rows * head_dim * 2) + align256(rows * sizeof(float));
}

inline size_t query_attention_workspace_bytes(int batch, int n_q_heads, int head_dim, int64_t n_q, int64_t n_keys,
                                              int n_splits) {
  if (batch < 1 || n_q_heads < 1 || (head_dim != 64 && head_dim != 128) || n_q < 1 || n_keys < 1 || n_splits < 0 ||
      n_q > kMaxTokens || n_keys > 3 * kMaxTokens)
    return 0;
  const KeySplit ks = plan_key_split(batch, n_q_heads, n_q, n_keys, n_splits);
  return ks.n_splits == 1 ? 0 : (size_t)ks.n_splits * key_range_bytes(batch, n_q_heads, head_dim, n_q);
}

// ---- attention-mass pass of the compression: with the probe rows resident in LDS (waves 4 or 8, n_blocks blocks of keys a
// wave), or streamed past 256 keys at a time (waves 0), by the time of each in rounds of the 256 compute units.  Resident
// workgroups hold a unit alone and fill its LDS first, streamed ones are three to a unit and small; so few keys a head, or a
// round that does not fill, are better streamed (us of the whole call, streamed / resident):
//   100 heads of 20 blocks of keys, 576 rows of 64  67 / 75      126 of 20, 512 rows of 128  86 / 90
//   192 of 25, 256 rows of 128  105 / 114                         32 of 256, 512 rows of 128  189 / 183
// Fitted to 5000 launches of 700 shapes; of these 6 are 1.2 to 3 % slower than streamed, the mean is 5 % faster.
constexpr int kMassMinProbeBytes = 49152;      // 192 rows of 128: with fewer the fill is too much of the work
constexpr int kMassMaxProbeBytes = 131072;     // 512
constexpr int kMassBlockKeys = 64;
struct MassPlan {
  int waves, n_blocks;
};
inline MassPlan plan_mass(int head_dim, int r_pad, int64_t L, int64_t heads) {
  const int64_t probe_bytes = (int64_t)r_pad * head_dim * 2;
  if (probe_bytes < kMassMinProbeBytes || probe_bytes > kMassMaxProbeBytes) return {0, 0};
  // times in us for 512 rows of 128, or 1024 of 64, the others in proportion; wg: workgroups in 256s
  const bool wide = head_dim == 128;
  const double rows = (double)probe_bytes / kMassMaxProbeBytes;
  const int64_t blocks = (L + kMassBlockKeys - 1) / kMassBlockKeys;
  auto units = [](int64_t n_wg) { return (double)n_wg / 256; };
  const double wg = units(heads * ((blocks + 3) / 4)), past = wg > 1 ? wg - 1 : 0;
  MassPlan best{0, 0};
  double least = wide ? 14.4 + 3.7 * (std::ceil(wg) - 1) + 3.0 * past : 17.2 + 5.6 * (std::ceil(wg) - 1) + 3.8 * past;
  least = (least - 1.5) * rows;                                      // (1.5: what the estimates are good to)
  for (int waves : {4, 8})
    for (int n = 1; n <= (waves == 4 ? 2 : 8); ++n) {
      const int64_t each = (blocks + waves - 1) / waves;             // blocks a wave has to take, n of them at most
      const double res = units(heads * ((each + n - 1) / n)), rounds = std::ceil(res);
      const double block = (waves == 4 ? (wide ? 8.0 : 11.3) : (wide ? 11.5 : 17.6)) * (double)(n < each ? n : each);
      // a fill is slower the more workgroups read the probe rows at once
      const double t = (wide ? 1.0 : 0.0) + rows * (rounds * ((wide ? 1.4 : 1.6) + block) + res * (wide ? 2.1 : 1.6));
      if (t < least) {
        least = t;
        best = {waves, n};
      }
    }
  return best;
}

// ---- workspace of the compression call: [partial sums of the pooled query | scores | sort arrays of the exact
// fallback when they do not fit the LDS]
constexpr int64_t kLdsSortMax = 8192;          // entries that fit the LDS selection arrays (14 bytes each)
constexpr int kPoolSplitMax = 8;               // workgroups (partial sums) per pooled query

// Ranges the n_rows = n_q * G probe rows of one pooled query are cut into: about 64 rows each, but no more ranges
// than it takes to give every compute unit two (n_pooled = batch * Hkv pooled queries share the 256 of them).
inline int pool_splits(int64_t n_rows, int64_t n_pooled) {
  int64_t s = (n_rows + 63) / 64;
  const int64_t fill = 512 / (n_pooled < 1 ? 1 : n_pooled);
  s = s > fill ? fill : s;
  return (int)(s < 1 ? 1 : (s > kPoolSplitMax ? kPoolSplitMax : s));
}

// Whether the scoring workgroups add up the pooled query themselves (compress.hip) instead of a launch in front of them, which
// costs about 2.5 us: few probe rows (16-byte loads a thread) read again by few workgroups.  Whole call, with the launch /
// without (us, graph replay): 16 rows of 64, 4 workgroups 11.4 / 9.6; 64 rows of 128, 64 workgroups 13.4 / 11.7, 512 15.1 /
// 13.6, 1504 16.8 / 17.7; 96 rows, 512 15.0 / 14.4; 160 rows, 250 14.1 / 13.5, 512 14.9 / 15.6; 512 rows, 64 14.1 / 17.3;
// 256 rows of 64, 256 14.6 / 13.6, 1024 16.3 / 18.0.
inline bool pools_in_scores(int64_t n_rows, int head_dim, int64_t heads, int64_t L) {
  const double loads = (double)n_rows * head_dim / 2048, workgroups = (double)heads * (double)((L * head_dim + 8191) / 8192);
  return loads <= 10 && workgroups / 256 * (loads + 1) <= 17;
}

inline int64_t pow2_ceil(int64_t x) {
  int64_t n = 1;
  while (n < x) n <<= 1;
  return n;
}

struct CompressWorkspace {
  size_t qbar_off, scores_off, sort_keys_off, sort_idx_off, total;
  int64_t n_sort;       // capacity (entries, a power of two) of the selection's sort arrays
  bool sort_in_global;
};

inline CompressWorkspace plan_compress_workspace(int batch, int hkv, int d, int64_t L, int64_t l_p) {
  CompressWorkspace w;
  size_t off = 0;
  w.qbar_off = off;
  off = align256(off + (size_t)batch * hkv * kPoolSplitMax * d * sizeof(double));
  w.scores_off = off;
  off = align256(off + (size_t)batch * hkv * (size_t)L * sizeof(double));
  // capacity of the sort arrays: room for the candidates of the fast path (the winners plus the rest
  // of the threshold bucket) when that fits the LDS, else exactly the padded winners
  w.n_sort = pow2_ceil(l_p > 1 ? l_p : 1);
  w.sort_in_global = w.n_sort > kLdsSortMax;
  if (!w.sort_in_global && 2 * w.n_sort <= kLdsSortMax) w.n_sort *= 2;
  w.sort_keys_off = w.sort_idx_off = off;
  if (w.sort_in_global) {
    w.sort_keys_off = off;
    off = align256(off + (size_t)batch * hkv * (size_t)w.n_sort * sizeof(uint64_t));
    w.sort_idx_off = off;
    off = align256(off + (size_t)batch * hkv * (size_t)w.n_sort * (sizeof(uint32_t) + sizeof(uint16_t)));
  }
  w.total = off;
  return w;
}

// Whether several workgroups share a head's selection and copy its rows in the same launch (compress.hip), or one selects
// and another launch copies.  Shared: one item of 2 heads x 16384 keys, 1024 rows 18.0 -> 16.5 us (graph replay), 6000 rows
// 29.8 -> 22.3, of 8 heads 41 -> 36; a launch less on the host as well.  Not with more heads (16 are even, 32.6 and 32.9 us,
// 32 slower, 29.2 and 30.5), nor beyond kResidentScores keys, which every workgroup would read three times (8 x 4 heads x
// 30000: 72 and 86); nor where most of a short block is selected (2000 of 2000 rows 14.9 and 15.7), nor without room for the
// candidates beside the rows, where the bucket path gives up and all workgroups sort (8192 rows 158 and 164).
constexpr int kResidentScores = 16384;         // scores a selection keeps in registers
constexpr uint32_t kMaxBinRank = 128;          // largest bucket the bucket path accepts
constexpr int kMaxSharedHeads = 8;
inline bool share_selection(int64_t heads, int64_t L, int64_t l_p, const CompressWorkspace& w) {
  return l_p > 0 && !w.sort_in_global && heads <= kMaxSharedHeads && L <= kResidentScores && (2 * l_p <= L || L > 4096) &&
         (w.n_sort < kLdsSortMax || l_p + kMaxBinRank <= w.n_sort || L <= w.n_sort);
}

// Workgroups a head of the compression in one launch (short_compress_kernel), 0 where it takes a launch per step.  More heads
// than share a selection, whose compression is four launches, of up to kShortKeys keys: one launch while the pooled query and the
// scores, which every workgroup repeats, cost less than the launches, and wherever the heads fill the chip by themselves.  Whole
// call, a launch per step / one (us, graph replay; probe rows x head_dim, keys a head): 128 heads, 512 x 64, 256 15.8 / 10.0;
// 480 heads 512 x 64, 512 31.4 / 20.4, 512 x 128, 1024 50.8 / 36.0; 32 heads, 448 x 128, 256 14.5 / 12.3; beyond the lines
// 32 heads, 512 x 128, 512 15.3 / 16.0, 1024 16.6 / 24.2, 96 heads, 512 x 128, 829 19.4 / 19.8; with up to eight heads, two or
// three launches, 16 x 64, 256 7.6 / 7.9, 512 x 128, 1024 11.6 / 17.1.  Beyond
// kShortBytes of rows read and written the memory decides, which a launch per step keeps busier with more waves, and a last round
// of long workgroups weighs more (640 heads, 8 x 128, 768, all selected 120.3 / 134.7; 552 heads, 512 x 128, 962 147.2 / 160.6).
// Of 11600 drawn calls within the lines a launch per step takes 1.34 times as long on average, and in 3 of 5800 with random
// scores 2 to 4 % less; where all scores are equal, which every part of a head sorts, in one of a hundred, up to 7 % less.
constexpr int kShortKeys = 1024;               // keys whose scores a workgroup keeps in LDS, one a thread
constexpr int64_t kShortBytes = 576 << 20;
inline int compresses_at_once(int64_t n_rows, int head_dim, int64_t heads, int64_t L, int64_t l_p) {
  const int64_t work = (2 * L + n_rows) * head_dim;
  if (l_p < 1 || L > kShortKeys || n_rows > 1024 || heads <= kMaxSharedHeads) return 0;
  if (work > (heads < 128 ? 110 << 10 : 256 << 10) && heads < 256) return 0;
  if (heads * (n_rows + L + 4 * l_p) * head_dim * 2 > kShortBytes) return 0;
  int64_t parts = l_p / 32 < 16 ? l_p / 32 : 16;
  parts = parts * heads <= 256 ? parts : 256 / heads;
  return (int)(parts > 1 ? parts : 1);
}

// Long blocks, a few heads: the scores' histogram by n_hist workgroups a head, selection and gather by n_parts (compress.hip);
// n_parts = 0: a workgroup per head and a gather launch.  The histograms take the place of the partial sums of the pooled
// query, kPoolSplitMax * head_dim * 8 bytes a head, which bounds the length; every part reads all of a head's scores, which
// bounds the heads.  Whole call, a workgroup per head / this (us, graph replay): 2 heads x 20000 keys 24.1 / 24.0, x 32768
// 33.4 / 25.7, x 65536 56.7 / 35.6, x 250000 182 / 79; 16 x 65536 95.8 / 76.5; 32 x 30000 75.5 / 70.3; 48 x 20000 79.7 / 81.8
// (before the parts of a head shared an XCD).  From 8192 - kMaxBinRank rows on the bucket path of the one workgroup has no room
// and it sorts: 1 x 65536, 8192 rows 272 / 36.5.
constexpr int kCoarseBins = 252;
constexpr int kMaxLongHeads = 32, kLongScores = 24576;
struct CoarseHistogram {         // of one part of a head's scores: counts (at most kResidentScores), and the map of all parts
  uint16_t count[kCoarseBins];
  float lo, inv;
};
static_assert(sizeof(CoarseHistogram) == 512, "eight to the partial sums of a pooled query of 64");
struct LongSelection {
  int n_hist, n_parts;
};
inline LongSelection plan_long_selection(int64_t heads, int head_dim, int64_t L, int64_t l_p, const CompressWorkspace& w) {
  const int64_t most = (int64_t)kPoolSplitMax * head_dim * (int64_t)sizeof(double) / (int64_t)sizeof(CoarseHistogram);
  if (l_p < 1 || w.sort_in_global || L <= kResidentScores || L > most * kResidentScores || heads > kMaxLongHeads) return {0, 0};
  if (L < kLongScores && (w.n_sort < kLdsSortMax || l_p + (int64_t)kMaxBinRank <= w.n_sort)) return {0, 0};
  int64_t n_hist = (L + kResidentScores / 2 - 1) / (kResidentScores / 2);
  n_hist = n_hist < most ? n_hist : most;
  int64_t n_parts = l_p / 32 < 16 ? l_p / 32 : 16;
  n_parts = n_parts * heads <= 256 ? n_parts : 256 / heads;
  return {(int)n_hist, (int)(n_parts > 1 ? n_parts : 1)};
}

// Which outputs a part takes.  Output x lies in the coarse bin of the outputs [excl, excl + c); a bin belongs to the part in
// whose share [l_p * part / n_parts, l_p * (part + 1) / n_parts) it begins, so that a part's outputs begin where a bin does.
// But a bin that may not fit the LDS beside the others of its part is divided where the shares are: every part that has some
// of it sorts the head's l_p largest (taken whole by one part, which then copied all its rows, us a call: 2 heads x 20000 keys
// of two values, 8100 rows 355 -> 271, 65536, 8000 rows 727 -> 593).
constexpr uint32_t most_of_a_bin(int64_t l_p, int n_parts) { return (uint32_t)(kLdsSortMax - (l_p + n_parts - 1) / n_parts); }
constexpr uint32_t first_of_share(uint32_t x, uint32_t excl, uint32_t c, uint32_t most) { return x == excl || c > most ? x : excl + c; }

// Workgroup -> head and part.  The parts of a head read the same scores, where they sort the head's largest ten times over, so
// they run on one of the eight XCDs (workgroup number modulo eight) and share its L2: rows of eight heads, one an XCD.  Fewer
// heads than a row are spread, as a single XCD's L2 would feed all parts.  us a call, parts of a head on several XCDs / on one:
// a key in 11 equal and on top, 32 heads x 131072 keys of 64, 1000 rows 683 / 497, 8 x 200000 of 128, 4000 rows 918 / 599
// (one workgroup a head took 601 and 718); normal scores 155 / 132, 121 / 121.
struct HeadPart {
  int head, part;
};
constexpr HeadPart head_and_part(int workgroup, int n_parts, int n_heads) {
  const int in_rows = n_heads / 8 * 8 * n_parts;
  if (workgroup >= in_rows) return {workgroup / n_parts, workgroup % n_parts};
  return {workgroup / (8 * n_parts) * 8 + workgroup % 8, workgroup / 8 % n_parts};
}

// The upper half of a float64 and its place in the order of the scores (as a signed integer; the map is its own inverse).
constexpr int upper_order(int hi) { return hi ^ ((hi >> 31) & 0x7fffffff); }
constexpr int kOrderInf = 0x7ff00000;          // of +infinity; above it lie NaNs, which the maps send to bin 0
// How far `to` lies above `from` in that order, modulo 2^32 (in unsigned arithmetic: the places of negative and of positive
// scores are further apart than an int holds).  `to` lies in [from, past) where its distance is below that of `past`.
constexpr uint32_t order_distance(int from, int to) { return (uint32_t)to - (uint32_t)from; }

inline size_t compress_workspace_bytes_checked(int batch, int n_kv_heads, int head_dim, int64_t L, int64_t l_p) {
  if (batch < 1 || n_kv_heads < 1 || (head_dim != 64 && head_dim != 128) || L < 1 || L > kMaxTokens || l_p < 0 || l_p > L)
    return 0;
  return plan_compress_workspace(batch, n_kv_heads, head_dim, L, l_p).total;
}

}  // namespace apbv
