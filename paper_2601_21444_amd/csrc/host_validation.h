// Host-side argument validation and planning of the C ABI (include/apbv.h).  Plain C++ with no HIP types, so that
// the rejection paths can be compiled alone with the host compiler and its sanitizers (tests/host/).  Everything
// here runs before any launch: a call that fails one of these checks enqueues nothing.
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <cmath>
#include "apbv.h"

namespace apbv {

constexpr int64_t kMaxTokens = (int64_t)1 << 24;
constexpr int kMaxKeySplits = 256;
constexpr int kAttnKeyTile = 64;            // keys per tile of the attention kernel
constexpr int kAttnQueryTile = 256;         // query rows per workgroup
constexpr int kAttnNarrowQueryTile = 64;    // ... of the variant used for query blocks of at most
constexpr int kAttnNarrowMaxRows = 128;     // this many rows
constexpr int kQueryMaxTokens = 2048;       // query blocks whose key-split launch packs the heads of a KV group into its rows
constexpr int kQueryShortTokens = 128;      // ... in tiles of kQueryShortRows rows up to here, of kAttnQueryTile above
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
// Blocks longer than kQueryMaxTokens are split like this; for shorter ones it is the fewest ranges the library's own
// choice may be cut down to when the workspace holds no more.
inline KeySplit per_head_key_split(int batch, int n_q_heads, int64_t n_q, int64_t n_keys) {
  const int64_t tile = n_q <= kAttnNarrowMaxRows ? kAttnNarrowQueryTile : kAttnQueryTile;
  const int64_t n_wg = (n_q + tile - 1) / tile * n_q_heads * batch;
  const int64_t s = (512 + n_wg - 1) / n_wg;
  const int64_t cap = key_tiles(n_keys) / 4 > 1 ? key_tiles(n_keys) / 4 : 1;
  return key_split_of(s < cap ? s : cap, key_tiles(n_keys));
}

// The split a workspace is sized for: as requested, or (0) the most ranges choose_key_split() takes whatever the
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

// The library's own choice for a block of at most kQueryMaxTokens queries, whose rows are packed per KV head.  For
// these kernels' purposes one workgroup per compute unit runs at a time (a second one shares the matrix pipe or the
// memory bandwidth), and the row tiles of a range run on one XCD of 32 compute units; a workgroup costs as much as kRangeOverhead key tiles before and after its keys (launch, cold
// instruction cache, first loads, epilogue), and every range adds its partial results to the merge.  In units of one
// 64-key tile (about 1 us): 64 queries of 16 / 2 heads over 16512 keys read 29.5 us at 16 ranges, 25.5 at 32, 27.8 at
// 64, 35.5 at 128; one query over 131072 keys 52.5 us at 32, 28.6 at 128, 29.7 at 256.
constexpr int kRangeOverhead = 8;
inline KeySplit choose_key_split(int batch, int n_q_heads, int n_kv_heads, int64_t n_q, int64_t n_keys) {
  const KeySplit most = plan_key_split(batch, n_q_heads, n_q, n_keys, 0);
  if (n_q > kQueryMaxTokens) return most;
  const int64_t rows = n_q * (n_q_heads / n_kv_heads);
  const int64_t tile = n_q <= kQueryShortTokens ? kQueryShortRows : kAttnQueryTile;
  const int64_t row_tiles = (rows + tile - 1) / tile, heads = (int64_t)n_kv_heads * batch;
  const int64_t n_tiles = key_tiles(n_keys);
  const double merge = (double)(rows * heads) / 5000.0;
  double best = 0.0;
  int64_t best_s = 1;
  for (int64_t s = 1; s <= most.n_splits; ++s) {
    const int64_t rounds = ((heads * s + 7) / 8 * row_tiles + 31) / 32;
    const double cost = (double)(rounds * ((n_tiles + s - 1) / s + kRangeOverhead)) + (s > 1 ? 4.0 + merge * (double)s : 0.0);
    if (s == 1 || cost < best) {
      best = cost;
      best_s = s;
    }
  }
  return key_split_of(best_s, n_tiles);
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

inline size_t compress_workspace_bytes_checked(int batch, int n_kv_heads, int head_dim, int64_t L, int64_t l_p) {
  if (batch < 1 || n_kv_heads < 1 || (head_dim != 64 && head_dim != 128) || L < 1 || L > kMaxTokens || l_p < 0 || l_p > L)
    return 0;
  return plan_compress_workspace(batch, n_kv_heads, head_dim, L, l_p).total;
}

}  // namespace apbv
