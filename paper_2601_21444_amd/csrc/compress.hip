// KV compression for gfx950 (Sec. 3.3; Alg. 1 "Identify Essential KVs" and "Send Block's Essential
// KVs"): score every local key, keep the l_p best per KV head, gather them.
//
// The score of key j for KV head v is the sum of the raw logits Q_qr[t, v*G+g] . K[j, v] over all
// query-block rows t and the G query heads of the group.  The sum is linear in the query, so it is
// evaluated as  q_bar[v] . K[j, v]  with the pooled query q_bar[v] = sum_t sum_g Q_qr[t, v*G+g]:
// one streaming pass over K, bound by HBM bandwidth.  Accumulation is in float64 so that the ranking
// agrees with a float64 evaluation (float32 accumulation flips near-equal neighbours).
//
// Launches on the caller's stream:
//   pool_query_kernel   partial sums of q_bar (float64), up to 8 row ranges per pooled query
//                                                                         [splits x Hkv x batch workgroups]
//   score_kernel        s[v, j], 16-byte coalesced reads of K rows; adds the partial sums of q_bar as it starts, or (few
//                       probe rows) the rows, without the launch in front; scores stored through to memory as it runs
//                                                                         [L/64 x Hkv x batch]
// then, for a few heads of at most 16384 keys,
//   select_gather_kernel  bucket sort by value of the scores above the l_p-th largest (exact fallback: radix select
//                       + bitonic sort), into (score descending, index ascending) order; K_c, V_c rows
//                                                                         [parts x Hkv x batch]
// for a few heads of longer blocks
//   coarse_histogram_kernel  counts of the scores per coarse bin          [n_hist x Hkv x batch]
//   long_select_gather_kernel  as above, over the coarse bins of a part   [parts x Hkv x batch]
// for many heads of at most 1024 keys, instead of all of these,
//   short_compress_kernel  every step in one launch                       [parts x Hkv x batch]
// and otherwise the same as two launches
//   select_kernel       the ordered indices                               [Hkv x batch]
//   gather_kernel       K_c, V_c rows                                     [l_p*Hkv/.. x batch]
#include <mutex>
#include "apbv_common.h"

namespace apbv {
namespace {

constexpr int kSelectThreads = 1024;

__device__ __forceinline__ double bf16_to_f64(uint32_t bits16) {
  return (double)__uint_as_float(bits16 << 16);
}

// A float64 moved across lanes by a DPP control (two 32-bit moves).  Controls: exchanges inside a quad, and
// rotations of a 16-lane row (lane i reads lane i-n of its row).
constexpr int kDppXor1 = 0xB1;    // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;    // quad_perm [2,3,0,1]
constexpr int kDppRor4 = 0x124;   // row_ror:4
constexpr int kDppRor8 = 0x128;   // row_ror:8
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  int lo = __double2loint(x), hi = __double2hiint(x);
  lo = __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xf, 0xf, false);
  hi = __builtin_amdgcn_update_dpp(0, hi, CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

// x plus that of the lane 16 or 32 away, in both.  (The swap of a register with itself leaves the lower group's value in both
// groups of the first result, the upper one's in those of the second.)
template <int AWAY>
__device__ __forceinline__ double add_rows(double x) {
  const uint32_t lo = (uint32_t)__double2loint(x), hi = (uint32_t)__double2hiint(x);
  auto swap = [](uint32_t w) { return AWAY == 16 ? __builtin_amdgcn_permlane16_swap(w, w, false, false) : __builtin_amdgcn_permlane32_swap(w, w, false, false); };
  const auto l = swap(lo), h = swap(hi);
  return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}

// ------------------------------------------------------------------------------------------------
// q_bar[b, v, c] = sum_g sum_t Q_qr[b, t, v*G+g, c]   (float64; the addends are bf16 so the sum is
// exact or within an ulp whatever the order).  The n_q * G probe rows of a (KV head, batch item) are
// cut into n_split equal ranges, one workgroup each (so that even a single item spreads over several
// compute units); a workgroup writes the partial sum of its range and the scoring kernel adds the
// partial sums in index order.  D/8 lanes per probe row (16-byte loads), T/(D/8) rows in flight (T = 1024 threads
// where a range is long enough to feed them four loads each, 256 otherwise).
template <int D, int T>
__global__ __launch_bounds__(T) void pool_query_kernel(View q, int64_t n_q, int group, double* qpart, int hkv, int n_split) {
  constexpr int KC = D / 8;
  constexpr int R = T / KC;                    // row groups
  __shared__ double part[T / 64][D];
  const int sp = blockIdx.x, v = blockIdx.y, b = blockIdx.z;
  const int c8 = threadIdx.x % KC, rg = threadIdx.x / KC;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bf16_t* base = q.ptr + (int64_t)b * q.sb + (int64_t)v * group * q.sh + 8 * c8;
  double acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0;
  const int n_rows = (int)(n_q * group);
  const int per = (n_rows + n_split - 1) / n_split;
  const int r_begin = sp * per, r_end = r_begin + per < n_rows ? r_begin + per : n_rows;
  // rows (t, g) in steps of R, four loads in flight; (t, g) advance without divisions in the loop
  const int dt = R / group, dg = R % group;
  int t = (r_begin + rg) / group, g = (r_begin + rg) % group;
  auto advance = [&]() {
    t += dt;
    g += dg;
    if (g >= group) {
      g -= group;
      ++t;
    }
  };
  for (int rr = r_begin + rg; rr < r_end; rr += 4 * R) {
    u32x4 x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      x[u] = u32x4{0u, 0u, 0u, 0u};                       // +0.0: adds nothing
      if (rr + u * R < r_end) x[u] = *reinterpret_cast<const u32x4*>(base + (int64_t)t * q.st + (int64_t)g * q.sh);
      advance();
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[2 * e] += bf16_to_f64(x[u][e] & 0xffffu);
        acc[2 * e + 1] += bf16_to_f64(x[u][e] >> 16);
      }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
#pragma unroll
    for (int m = KC; m < 64; m <<= 1) acc[e] += __shfl_xor(acc[e], m);
  }
  if (lane < KC) {
#pragma unroll
    for (int e = 0; e < 8; ++e) part[wave][8 * c8 + e] = acc[e];
  }
  __syncthreads();
  if (threadIdx.x < D) {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < T / 64; ++w) sum += part[w][threadIdx.x];
    qpart[(((int64_t)b * hkv + v) * n_split + sp) * D + threadIdx.x] = sum;
  }
}

// The sums of four rows over the LPR lanes of each, a reduce-scatter: after the two exchanges inside a quad each lane holds
// one row's sum over its quad, two rotations by 4 and 8 lanes finish it.  The last quad of a row's lanes (c >= LPR - 4) holds
// complete sums, this lane that of row *u.  Every row takes the same summation tree (the adds commute), so identical rows get
// identical scores.
template <int LPR>
__device__ __forceinline__ double reduce_rows(const double (&a)[4], int c, int* u) {
  const bool odd1 = (c & 1) != 0, odd2 = (c & 2) != 0;
  double keep0 = odd1 ? a[2] : a[0], keep1 = odd1 ? a[3] : a[1];
  keep0 += dpp_f64<kDppXor1>(odd1 ? a[0] : a[2]);
  keep1 += dpp_f64<kDppXor1>(odd1 ? a[1] : a[3]);
  double acc = odd2 ? keep1 : keep0;
  acc += dpp_f64<kDppXor2>(odd2 ? keep0 : keep1);
  acc += dpp_f64<kDppRor4>(acc);
  if (LPR == 16) acc += dpp_f64<kDppRor8>(acc);
  *u = (odd1 ? 2 : 0) + (odd2 ? 1 : 0);
  return acc;
}

// ------------------------------------------------------------------------------------------------
// s[b, v, j] = q_bar[b, v, :] . K[b, j, v, :].  D/8 lanes per key row, each lane 8 elements (one
// 16-byte load), fixed summation order per row so identical rows get identical scores.
// kPool: every workgroup adds the few probe rows of its pooled query itself, behind its key loads, and there is no launch
// for it (pools_in_scores: where).
template <int D, bool kPool>
__global__ __launch_bounds__(256) void score_kernel(View k, int64_t L, const double* __restrict__ qpart, int n_split,
                                                    double* __restrict__ s_ws, double* __restrict__ s_out,
                                                    int hkv, int rows_per_block, View q, int group) {
  constexpr int LPR = D / 8;               // lanes per row
  constexpr int RPS = 256 / LPR;           // rows per step of the workgroup
  constexpr int UNROLL = 4;
  static_assert(LPR == 8 || LPR == 16, "the cross-lane reduction below is written for 8 or 16 lanes per row");
  const int v = blockIdx.y, b = blockIdx.z;
  const int c = threadIdx.x % LPR;
  const int rsub = threadIdx.x / LPR;
  __shared__ double qs[D];
  __shared__ double rows[kPool ? RPS : 1][kPool ? D : 1];
  const double* qb = kPool ? nullptr : qpart + ((int64_t)b * hkv + v) * n_split * D;      // n_split partial sums of the pooled query
  const bf16_t* base = k.ptr + (int64_t)b * k.sb + (int64_t)v * k.sh + 8 * c;
  const int64_t out_base = ((int64_t)b * hkv + v) * L;
  const int64_t r_begin = (int64_t)blockIdx.x * rows_per_block;
  const int64_t r_end = (r_begin + rows_per_block < L) ? r_begin + rows_per_block : L;

  for (int64_t r0 = r_begin; r0 < r_end; r0 += RPS * UNROLL) {
    u32x4 x[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int64_t j = r0 + u * RPS + rsub;
      u32x4 z = {0u, 0u, 0u, 0u};
      if (j < r_end) z = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + j * k.st));
      x[u] = z;
    }
    // The pooled query reaches the lanes through LDS -- one 16-byte load by D/2 lanes per workgroup, behind the
    // key loads, instead of four loads per lane in front of them.
    if (kPool && r0 == r_begin) {
      const bf16_t* qrow = q.ptr + (int64_t)b * q.sb + (int64_t)v * group * q.sh + 8 * c;
      const int n_rows = (int)q.tokens * group;
      double sum[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) sum[e] = 0.0;
      for (int r = rsub; r < n_rows; r += 4 * RPS) {
        u32x4 y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int rr = r + u * RPS, t = rr / group;
          y[u] = u32x4{0u, 0u, 0u, 0u};                      // +0.0: adds nothing
          if (rr < n_rows) y[u] = *reinterpret_cast<const u32x4*>(qrow + (int64_t)t * q.st + (int64_t)(rr - t * group) * q.sh);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            sum[2 * e] += bf16_to_f64(y[u][e] & 0xffffu);
            sum[2 * e + 1] += bf16_to_f64(y[u][e] >> 16);
          }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) rows[rsub][8 * c + e] = sum[e];
      __syncthreads();
      if (threadIdx.x < D) {
        double t = 0.0;
#pragma unroll
        for (int r = 0; r < RPS; ++r) t += rows[r][threadIdx.x];
        qs[threadIdx.x] = t;
      }
      __syncthreads();
    }
    if (!kPool && r0 == r_begin) {
      if (threadIdx.x < D / 2) {
        // all partial sums are fetched before the first addition (independent loads), then added in index order
        double2 part[kPoolSplitMax];
#pragma unroll
        for (int sp = 0; sp < kPoolSplitMax; ++sp) {
          part[sp] = double2{0.0, 0.0};
          if (sp < n_split) part[sp] = *reinterpret_cast<const double2*>(qb + sp * D + 2 * threadIdx.x);
        }
        double2 t = part[0];
#pragma unroll
        for (int sp = 1; sp < kPoolSplitMax; ++sp)
          if (sp < n_split) {
            t.x += part[sp].x;
            t.y += part[sp].y;
          }
        qs[2 * threadIdx.x] = t.x;
        qs[2 * threadIdx.x + 1] = t.y;
      }
      __syncthreads();
    }
    double qv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) qv[e] = qs[8 * c + e];
    double a[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      double acc = 0.0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc = __builtin_fma(qv[2 * e], bf16_to_f64(x[u][e] & 0xffffu), acc);
        acc = __builtin_fma(qv[2 * e + 1], bf16_to_f64(x[u][e] >> 16), acc);
      }
      a[u] = acc;
    }
    int u;                                             // the row this lane ends up with
    const double acc = reduce_rows<LPR>(a, c, &u);
    const int64_t j = r0 + u * RPS + rsub;
    if (c >= LPR - 4 && j < r_end) {                   // the last quad of the row's lanes holds complete sums
      // written through to memory as the kernel runs (device-scope store): left to the write-back cache, the
      // scores of a large batch are flushed when the kernel ends, with nothing left to overlap the flush
      __hip_atomic_store(reinterpret_cast<long long*>(s_ws + out_base + j), __double_as_longlong(acc), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      if (s_out) s_out[out_base + j] = acc;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Order-preserving key: larger score <=> larger unsigned key; -0.0 and +0.0 map to the same key.
__device__ __forceinline__ uint64_t score_key(double s) {
  uint64_t b = (uint64_t)__double_as_longlong(s);
  if ((b << 1) == 0) b = 0;
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

// (key descending, index ascending)
__device__ __forceinline__ bool precedes(uint64_t ka, uint32_t ia, uint64_t kb, uint32_t ib) {
  return ka > kb || (ka == kb && ia < ib);
}

constexpr int kBins = 2048;                    // value buckets of the fast selection path

static_assert(kResidentScores == 16 * kSelectThreads, "sixteen scores a thread in registers");

struct SelectShared {
  uint32_t hist[kBins];       // entries per bucket
  uint32_t base[kBins];       // entries in higher buckets (output offset of the bucket)
  uint32_t fill[kBins];       // scatter cursor per bucket
  uint64_t prefix;
  uint32_t need, bucket, cnt, n_cand, t_bin, crowded, divided;
  int b_lo, b_hi;             // kParts: lowest and highest bucket of the part
  int order[2];               // long blocks: a part's range in the order of the scores, of the outputs
  uint32_t share[2];
  uint32_t wave_tot[kSelectThreads / 64];
  float red_lo[kSelectThreads / 64], red_hi[kSelectThreads / 64];
};

// Wave-wide combinations on the DPP data path (no LDS traffic): shifts inside the 16-lane rows, then lane 15 of
// a row into the next row and lane 31 into the upper half.  A lane whose source lies outside keeps `self`.
constexpr int kDppShr1 = 0x111, kDppShr2 = 0x112, kDppShr4 = 0x114, kDppShr8 = 0x118;   // row_shr:n
constexpr int kDppBcast15 = 0x142, kDppBcast31 = 0x143;
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_or_self(uint32_t self, uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)self, (int)x, CTRL, ROW_MASK, 0xf, false);
}

// Inclusive prefix sum over the 64 lanes of a wave.
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t x) {
  x += dpp_or_self<kDppShr1, 0xf>(0u, x);
  x += dpp_or_self<kDppShr2, 0xf>(0u, x);
  x += dpp_or_self<kDppShr4, 0xf>(0u, x);
  x += dpp_or_self<kDppShr8, 0xf>(0u, x);
  x += dpp_or_self<kDppBcast15, 0xa>(0u, x);
  x += dpp_or_self<kDppBcast31, 0xc>(0u, x);
  return x;
}

// op over the 64 lanes of a wave, the result in every lane (lane 63 collects it, one scalar read spreads it).
template <typename Op>
__device__ __forceinline__ uint32_t wave_reduce_bits(uint32_t x, Op op) {
  x = op(x, dpp_or_self<kDppShr1, 0xf>(x, x));
  x = op(x, dpp_or_self<kDppShr2, 0xf>(x, x));
  x = op(x, dpp_or_self<kDppShr4, 0xf>(x, x));
  x = op(x, dpp_or_self<kDppShr8, 0xf>(x, x));
  x = op(x, dpp_or_self<kDppBcast15, 0xa>(x, x));
  x = op(x, dpp_or_self<kDppBcast31, 0xc>(x, x));
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
__device__ __forceinline__ float wave_min(float x) {
  return __uint_as_float(wave_reduce_bits(__float_as_uint(x), [](uint32_t a, uint32_t b) {
    return __float_as_uint(fminf(__uint_as_float(a), __uint_as_float(b)));
  }));
}
__device__ __forceinline__ float wave_max(float x) {
  return __uint_as_float(wave_reduce_bits(__float_as_uint(x), [](uint32_t a, uint32_t b) {
    return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
  }));
}

// Inclusive scan of one value per thread over the whole workgroup (1024 threads); returns the
// inclusive prefix, *total gets the workgroup sum.  (wave_tot must not have been used since the last barrier.)
__device__ __forceinline__ uint32_t block_scan_incl(uint32_t x, SelectShared& sh, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t incl = wave_scan_incl(x);
  if (lane == 63) sh.wave_tot[wave] = incl;
  __syncthreads();
  // every wave scans the 16 totals itself, one a lane
  constexpr int kSelectWaves = kSelectThreads / 64;
  const uint32_t scan = wave_scan_incl(lane < kSelectWaves ? sh.wave_tot[lane] : 0u);
  const int w = __builtin_amdgcn_readfirstlane(wave);
  *total = (uint32_t)__builtin_amdgcn_readlane((int)scan, kSelectWaves - 1);
  return incl + (w > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)scan, w - 1) : 0u);
}

// Bitonic sort of n_sort (a power of two) entries into (key descending, index ascending) order.
__device__ __forceinline__ void bitonic_sort(uint64_t* skeys, uint32_t* sidx, int64_t n_sort64) {
  const uint32_t tid = threadIdx.x;
  const uint32_t n_sort = (uint32_t)n_sort64, half = n_sort >> 1;
  for (uint32_t k = 2; k <= n_sort; k <<= 1) {
    for (uint32_t j = k >> 1, lj = 31 - __builtin_clz(j); j > 0; j >>= 1, --lj) {
      for (uint32_t pidx = tid; pidx < half; pidx += kSelectThreads) {
        const uint32_t i = ((pidx >> lj) << (lj + 1)) | (pidx & (j - 1));
        const uint32_t q = i + j;
        const bool up = (i & k) == 0;          // this run is sorted "first precedes"
        const uint64_t ka = skeys[i], kb = skeys[q];
        const uint32_t ia = sidx[i], ib = sidx[q];
        const bool in_order = precedes(ka, ia, kb, ib);
        if (in_order != up) {
          skeys[i] = kb;
          skeys[q] = ka;
          sidx[i] = ib;
          sidx[q] = ia;
        }
      }
      __syncthreads();
    }
  }
}

// Fast path: a bucket sort by VALUE.  A monotone map sends every score to one of kBins buckets of equal width
// between the minimum and the maximum (computed in single precision: only the order matters).  A suffix scan of
// the bucket counts gives each bucket its output offset and finds the bucket that holds the l_p-th largest score;
// the entries of that bucket and of all higher ones are scattered into bucket-grouped order, and each entry then
// finds its rank inside its (small) bucket by direct comparison of the full 64-bit keys and indices.  Because the
// map is monotone, bucket order followed by (key descending, index ascending) inside a bucket is the global order,
// ties included.  Returns false (nothing written) if the candidates do not fit `cap` or a bucket is too crowded to
// rank by comparison; the caller then takes the exact radix path.
// kParts: n_parts workgroups share a head.  Each takes the buckets whose output offset lies in its share of the l_p
// outputs, scatters and ranks those alone, and leaves their indices in sh.fill, outputs [*out_first, *out_first +
// *n_out).  The histogram, and with it the decision to give up, is the same in every workgroup.
template <bool kParts, int kPer = kResidentScores / kSelectThreads>
__device__ __forceinline__ bool bucket_rank_select(const double* __restrict__ s, int64_t L, int64_t l_p, int64_t cap,
                                                   uint64_t* skeys, uint32_t* sidx, uint16_t* sbin,
                                                   int32_t* __restrict__ idx_out, SelectShared& sh, int part = 0,
                                                   int n_parts = 1, uint32_t* out_first = nullptr, uint32_t* n_out = nullptr) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool resident = kParts || L <= kResidentScores;      // (heads are shared only where the scores are resident)
  double sc[kPer];
  uint32_t bins[kPer];                                       // bucket | arrival order in the bucket << 11
  if (resident) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const uint32_t j = (uint32_t)tid + (uint32_t)u * kSelectThreads;
      sc[u] = j < (uint32_t)L ? *reinterpret_cast<const double*>(reinterpret_cast<const char*>(s) + (size_t)(j * 8u)) : 0.0;
    }
  }
  // minimum and maximum, in single precision (the conversion is monotone, which is all the map needs)
  float lo = INFINITY, hi = -INFINITY;
  if (resident) {
#pragma unroll
    for (int u = 0; u < kPer; ++u)
      if (tid + (int64_t)u * kSelectThreads < L) {
        const float x = (float)sc[u];
        lo = fminf(lo, x);
        hi = fmaxf(hi, x);
      }
  } else {
    for (int64_t j = tid; j < L; j += kSelectThreads) {
      const float x = (float)s[j];
      lo = fminf(lo, x);
      hi = fmaxf(hi, x);
    }
  }
  lo = wave_min(lo);
  hi = wave_max(hi);
  if (lane == 0) {
    sh.red_lo[wave] = lo;
    sh.red_hi[wave] = hi;
  }
  for (int i = tid; i < kBins; i += kSelectThreads) {
    sh.hist[i] = 0;
    sh.fill[i] = 0;
  }
  if (tid == 0) {
    sh.crowded = 0;
    if (kParts) {
      sh.b_lo = kBins;
      sh.b_hi = -1;
    }
  }
  __syncthreads();
  lo = wave_min(sh.red_lo[lane % (kSelectThreads / 64)]);     // (16 waves' values, one a lane: a loop over them costs 0.6 us)
  hi = wave_max(sh.red_hi[lane % (kSelectThreads / 64)]);
  const float inv = (float)kBins / (hi - lo);
  if (!(inv > 0.0f) || !(inv < 1.0e30f)) return false;       // all scores equal in single precision (or range overflow)
  // rounding, subtraction of lo, multiplication by a positive constant and truncation are all monotone
  auto bin_of = [&](double x) {
    const int b = (int)(((float)x - lo) * inv);
    return (uint32_t)(b > kBins - 1 ? kBins - 1 : b);
  };
  // histogram; the count an atomic returns is the entry's arrival order inside its bucket, kept (with the bucket)
  // for the scatter below so that the resident case needs no second pass of atomics
  if (resident) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      bins[u] = 0;
      if (tid + (int64_t)u * kSelectThreads < L) {
        const uint32_t b = bin_of(sc[u]);
        bins[u] = b | (atomicAdd(&sh.hist[b], 1u) << 11);
      }
    }
  } else {
    for (int64_t j = tid; j < L; j += kSelectThreads) atomicAdd(&sh.hist[bin_of(s[j])], 1u);
  }
  __syncthreads();
  // thread t owns buckets kBins-1-2t and kBins-2-2t (descending): suffix counts by an inclusive scan
  const int b0 = kBins - 1 - 2 * tid, b1 = kBins - 2 - 2 * tid;
  const uint32_t c0 = sh.hist[b0], c1 = sh.hist[b1];
  uint32_t total;
  const uint32_t incl = block_scan_incl(c0 + c1, sh, &total);
  const uint32_t excl = incl - (c0 + c1);
  sh.base[b0] = excl;
  sh.base[b1] = excl + c0;
  if (kParts) {
    const uint32_t from = (uint32_t)(l_p * part / n_parts), to = (uint32_t)(l_p * (part + 1) / n_parts);
    const bool in0 = c0 != 0 && excl >= from && excl < to, in1 = c1 != 0 && excl + c0 >= from && excl + c0 < to;
    if (in0 || in1) {
      atomicMin(&sh.b_lo, in1 ? b1 : b0);
      atomicMax(&sh.b_hi, in0 ? b0 : b1);
    }
  }
  if (excl < (uint32_t)l_p && (uint32_t)l_p <= incl) {
    const bool first = (uint32_t)l_p <= excl + c0;
    sh.t_bin = first ? b0 : b1;
    sh.n_cand = first ? excl + c0 : incl;
  }
  __syncthreads();
  const uint32_t n_cand = sh.n_cand;
  const int t_bin = (int)sh.t_bin;
  if ((int64_t)n_cand > cap) return false;
  // a candidate bucket too crowded to rank by comparison: seen by every thread after the scatter's barrier
  if ((b0 >= t_bin && c0 > kMaxBinRank) || (b1 >= t_bin && c1 > kMaxBinRank)) sh.crowded = 1;
  // the candidates this workgroup ranks: those of buckets [b_lo, b_hi], positions from `first` on
  const int b_lo = kParts ? sh.b_lo : t_bin, b_hi = kParts ? sh.b_hi : kBins - 1;
  const bool none = kParts && b_hi < 0;
  const uint32_t first = kParts && !none ? sh.base[b_hi] : 0;
  const uint32_t n_loc = none ? 0 : (kParts ? sh.base[b_lo] + sh.hist[b_lo] - first : n_cand);
  // scatter the candidates into bucket-grouped order.  Every wave walks all kPer iterations for the few lanes
  // that hold a candidate, so the body is two stores (index, raw score); key and bucket follow below.
  if (resident && kParts) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const uint32_t j = (uint32_t)tid + (uint32_t)u * kSelectThreads;
      const int b = (int)(bins[u] & (uint32_t)(kBins - 1));
      if (j < (uint32_t)L && b >= b_lo && b <= b_hi) {
        const uint32_t pos = sh.base[b] - first + (bins[u] >> 11);
        sidx[pos] = j;
        skeys[pos] = (uint64_t)__double_as_longlong(sc[u]);
      }
    }
  } else if (resident) {
    // Every bucket offset is fetched before the first store.  Lanes without a candidate all read one and the
    // same word (a broadcast), so that only the few candidates' reads can collide on an LDS bank.
    uint32_t pos[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const uint32_t b = bins[u] & (uint32_t)(kBins - 1);
      pos[u] = sh.base[(int)b >= t_bin ? b : (uint32_t)(kBins - 1)] + (bins[u] >> 11);
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const uint32_t j = (uint32_t)tid + (uint32_t)u * kSelectThreads;
      if (j < (uint32_t)L && (int)(bins[u] & (uint32_t)(kBins - 1)) >= t_bin) {
        sidx[pos[u]] = j;
        skeys[pos[u]] = (uint64_t)__double_as_longlong(sc[u]);
      }
    }
  } else {
    for (int64_t j = tid; j < L; j += kSelectThreads) {
      const double x = s[j];
      const uint32_t b = bin_of(x);
      if ((int)b >= t_bin) {
        const uint32_t pos = sh.base[b] + atomicAdd(&sh.fill[b], 1u);
        sidx[pos] = (uint32_t)j;
        skeys[pos] = (uint64_t)__double_as_longlong(x);
      }
    }
  }
  __syncthreads();
  // the owner of a candidate position turns the raw score into its key and bucket, in place
  for (uint32_t pos = tid; pos < n_loc; pos += kSelectThreads) {
    const double x = __longlong_as_double((long long)skeys[pos]);
    skeys[pos] = score_key(x);
    sbin[pos] = (uint16_t)bin_of(x);
  }
  __syncthreads();
  if (sh.crowded) return false;
  // rank inside the bucket, write the index at its final position
  for (uint32_t pos = tid; pos < n_loc; pos += kSelectThreads) {
    const uint32_t b = sbin[pos];
    const uint32_t begin = sh.base[b] - first, cnt = sh.hist[b];
    const uint64_t key = skeys[pos];
    const uint32_t idx = sidx[pos];
    uint32_t rank = 0;
    const uint32_t end = begin + cnt;                        // cnt >= 1: the entry itself
    for (uint32_t q = begin; q < end; q += 4) {              // four entries' reads in flight
      uint64_t kq[4];
      uint32_t iq[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t qq = q + e < end ? q + e : end - 1;
        kq[e] = skeys[qq];
        iq[e] = sidx[qq];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) rank += (q + e < end && precedes(kq[e], iq[e], key, idx)) ? 1u : 0u;
    }
    if (first + begin + rank < (uint32_t)l_p) {
      idx_out[first + begin + rank] = (int32_t)idx;
      if (kParts) sh.fill[begin + rank] = idx;                // (the scatter's cursors are done with)
    }
  }
  if (kParts) {
    *out_first = first;
    *n_out = first + n_loc < (uint32_t)l_p ? n_loc : (uint32_t)l_p - first;
  }
  return true;
}

// Exact path for any input: radix select of the l_p-th largest key, most significant byte first, then
// collection of the l_p winners (ties at the threshold by ascending index).
// kByWaves: where ties have to be told apart by index, each wave reads a range of keys, instead of each thread, which reads a
// line of memory a lane.  For long blocks, whose exact path runs in many workgroups at once: equal scores, us a call, 2 heads
// x 65536, 2000 rows 558 -> 529, 32 x 131072, 1000 rows 1343 -> 1140.  In the other kernels, whose exact path lies in the
// midst of code that is fetched once, it moves what lies behind: 154 -> 147 for 2 x 16384 equal scores, but up to 2 % of every
// call of blocks of 4000 keys.
template <bool kByWaves>
__device__ __forceinline__ void radix_collect(const double* __restrict__ s, int64_t L, int64_t l_p, uint64_t* skeys,
                                              uint32_t* sidx, SelectShared& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // after 8 passes `prefix` is the l_p-th largest key and `need` says how many keys equal to it belong
  // to the result
  uint64_t prefix = 0;
  uint32_t need = (uint32_t)l_p;
  uint32_t bucket = 0;           // number of keys equal to the final prefix
  for (int pass = 0; pass < 8; ++pass) {
    const int shift = 56 - 8 * pass;
    __syncthreads();
    if (tid < 256) sh.hist[tid] = 0;
    __syncthreads();
    for (int64_t j = tid; j < L; j += kSelectThreads) {
      const uint64_t key = score_key(s[j]);
      if (pass == 0 || (key >> (shift + 8)) == prefix) atomicAdd(&sh.hist[(key >> shift) & 255], 1u);
    }
    __syncthreads();
    if (wave == 0) {
      // lane l owns digits 255-4l .. 252-4l (descending); find the digit holding the need-th largest
      uint32_t c4[4], tot = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        c4[q] = sh.hist[255 - 4 * lane - q];
        tot += c4[q];
      }
      const uint32_t incl = wave_scan_incl(tot);
      uint32_t excl = incl - tot;
      if (excl < need && need <= incl) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (excl < need && need <= excl + c4[q]) {
            sh.prefix = (prefix << 8) | (uint64_t)(255 - 4 * lane - q);
            sh.need = need - excl;
            sh.bucket = c4[q];
          }
          excl += c4[q];
        }
      }
    }
    __syncthreads();
    prefix = sh.prefix;
    need = sh.need;
    bucket = sh.bucket;
  }
  const uint64_t kth = prefix;
  const uint32_t n_gt = (uint32_t)l_p - need;     // keys strictly above the threshold

  if (tid == 0) sh.cnt = 0;
  __syncthreads();
  if (bucket == need) {
    // every key equal to the threshold is taken: no ordering constraint while collecting
    for (int64_t j = tid; j < L; j += kSelectThreads) {
      const uint64_t key = score_key(s[j]);
      if (key >= kth) {
        const uint32_t pos = atomicAdd(&sh.cnt, 1u);
        skeys[pos] = key;
        sidx[pos] = (uint32_t)j;
      }
    }
  } else if constexpr (!kByWaves) {
    // more equal keys than needed: take the `need` lowest indices.  Each thread scans a contiguous
    // index range; an exclusive scan of the per-thread tie counts gives each tie its rank by index.
    const int64_t chunk = (L + kSelectThreads - 1) / kSelectThreads;
    const int64_t lo = (int64_t)tid * chunk, hi = (lo + chunk < L) ? lo + chunk : L;
    uint32_t n_eq = 0;
    for (int64_t j = lo; j < hi; ++j) n_eq += (score_key(s[j]) == kth);
    uint32_t total;
    uint32_t rank = block_scan_incl(n_eq, sh, &total) - n_eq;
    for (int64_t j = lo; j < hi; ++j) {
      const uint64_t key = score_key(s[j]);
      if (key > kth) {
        const uint32_t pos = atomicAdd(&sh.cnt, 1u);
        skeys[pos] = key;
        sidx[pos] = (uint32_t)j;
      } else if (key == kth) {
        if (rank < need) {
          skeys[n_gt + rank] = key;
          sidx[n_gt + rank] = (uint32_t)j;
        }
        ++rank;
      }
    }
  } else {
    // more equal keys than needed: as above, a contiguous range per wave, 64 keys side by side
    constexpr int kWaves = kSelectThreads / 64;
    const int64_t span = (L + kSelectThreads - 1) / kSelectThreads * 64;
    const int64_t lo = wave * span, hi = lo + span < L ? lo + span : L;
    uint32_t n_eq = 0;
    for (int64_t j0 = lo; j0 < hi; j0 += 64) {
      const int64_t j = j0 + lane;
      n_eq += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(j < hi && score_key(s[j]) == kth));
    }
    if (lane == 0) sh.wave_tot[wave] = n_eq;
    __syncthreads();
    uint32_t rank = 0;                          // ties in front of the range, then of its next 64 keys
#pragma unroll
    for (int w = 0; w < kWaves; ++w) rank += w < wave ? sh.wave_tot[w] : 0u;
    for (int64_t j0 = lo; j0 < hi; j0 += 64) {
      const int64_t j = j0 + lane;
      const uint64_t key = j < hi ? score_key(s[j]) : 0;
      const bool tie = j < hi && key == kth;
      const uint64_t ties = __builtin_amdgcn_ballot_w64(tie);
      if (key > kth) {
        const uint32_t pos = atomicAdd(&sh.cnt, 1u);
        skeys[pos] = key;
        sidx[pos] = (uint32_t)j;
      } else if (tie) {
        const uint32_t at = rank + __builtin_amdgcn_mbcnt_hi((uint32_t)(ties >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ties, 0u));
        if (at < need) {
          skeys[n_gt + at] = key;
          sidx[n_gt + at] = (uint32_t)j;
        }
      }
      rank += (uint32_t)__builtin_popcountll(ties);
    }
  }
}

// One workgroup per (KV head, batch item).  skeys/sidx hold `cap` entries (LDS or global).
template <bool kGlobalSort>
__global__ __launch_bounds__(kSelectThreads) void select_kernel(const double* __restrict__ s_ws, int64_t L, int64_t l_p,
                                                                int64_t cap, int32_t* __restrict__ idx_out,
                                                                uint64_t* gkeys, uint32_t* gidx, int hkv) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  __shared__ SelectShared sh;

  const int v = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x;
  const int64_t head = (int64_t)b * hkv + v;
  const double* s = s_ws + head * L;
  uint64_t* skeys;
  uint32_t* sidx;
  if (kGlobalSort) {
    skeys = gkeys + head * cap;
    sidx = reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(gidx) + head * cap * 6);   // [cap] u32 + [cap] u16
  } else {
    skeys = reinterpret_cast<uint64_t*>(dyn);
    sidx = reinterpret_cast<uint32_t*>(dyn + cap * sizeof(uint64_t));
  }

  uint16_t* sbin = reinterpret_cast<uint16_t*>(sidx + cap);
  if (bucket_rank_select<false>(s, L, l_p, cap, skeys, sidx, sbin, idx_out + head * l_p, sh)) return;
  radix_collect<false>(s, L, l_p, skeys, sidx, sh);
  int64_t n_sort = 1;
  while (n_sort < l_p) n_sort <<= 1;
  __syncthreads();
  for (int64_t i = l_p + tid; i < n_sort; i += kSelectThreads) {   // padding sorts last
    skeys[i] = 0;
    sidx[i] = 0xffffffffu;
  }
  __syncthreads();
  bitonic_sort(skeys, sidx, n_sort);
  for (int64_t i = tid; i < l_p; i += kSelectThreads) idx_out[head * l_p + i] = (int32_t)sidx[i];
}

// ------------------------------------------------------------------------------------------------
// K_c[b, i, v, :] = K[b, idx[b, v, i], v, :], same for V.  One thread per 16-byte chunk.
template <int D>
__global__ __launch_bounds__(256) void gather_kernel(View k, View v, const int32_t* __restrict__ idx, int64_t l_p, int hkv,
                                                     int64_t L, bf16_t* __restrict__ k_c, bf16_t* __restrict__ v_c) {
  constexpr int KC = D / 8;
  const int b = blockIdx.y;
  const int64_t item = (int64_t)blockIdx.x * 256 + threadIdx.x;      // over l_p * hkv * KC
  const int64_t n_items = l_p * hkv * KC;
  if (item >= n_items) return;
  const int c = (int)(item % KC);
  const int64_t row = item / KC;            // i * hkv + head
  const int head = (int)(row % hkv);
  const int64_t i = row / hkv;
  const int64_t j = idx[((int64_t)b * hkv + head) * l_p + i];
  if (j < 0 || j >= L) return;              // never read outside the block, whatever idx holds
  const int64_t dst = (((int64_t)b * l_p + i) * hkv + head) * D + 8 * c;
  const u32x4 kk = *reinterpret_cast<const u32x4*>(k.ptr + (int64_t)b * k.sb + j * k.st + (int64_t)head * k.sh + 8 * c);
  const u32x4 vv = *reinterpret_cast<const u32x4*>(v.ptr + (int64_t)b * v.sb + j * v.st + (int64_t)head * v.sh + 8 * c);
  // (the compressed block is written once and read by another kernel or a copy engine: keep it out of the caches)
  __builtin_nontemporal_store(kk, reinterpret_cast<u32x4*>(k_c + dst));
  __builtin_nontemporal_store(vv, reinterpret_cast<u32x4*>(v_c + dst));
}

// K_c, V_c rows first .. first + n_out - 1 of a head from the token indices in `rows` (LDS), by one workgroup.
template <int D>
__device__ __forceinline__ void copy_rows(const View& k, const View& v, const uint32_t* rows, uint32_t first, uint32_t n_out, int b, int head, int hkv, int64_t l_p,
                                          bf16_t* __restrict__ k_c, bf16_t* __restrict__ v_c) {
  constexpr int KC = D / 8;
  const bf16_t* kb = k.ptr + (int64_t)b * k.sb + (int64_t)head * k.sh;
  const bf16_t* vb = v.ptr + (int64_t)b * v.sb + (int64_t)head * v.sh;
  for (uint32_t item = threadIdx.x; item < n_out * KC; item += kSelectThreads) {
    const uint32_t i = item / KC, c = item % KC;
    const int64_t j = rows[i];
    const int64_t dst = (((int64_t)b * l_p + first + i) * hkv + head) * D + 8 * c;
    const u32x4 kk = *reinterpret_cast<const u32x4*>(kb + j * k.st + 8 * c);
    const u32x4 vv = *reinterpret_cast<const u32x4*>(vb + j * v.st + 8 * c);
    __builtin_nontemporal_store(kk, reinterpret_cast<u32x4*>(k_c + dst));
    __builtin_nontemporal_store(vv, reinterpret_cast<u32x4*>(v_c + dst));
  }
}

// Selection and gather in one launch, n_parts workgroups per (KV head, batch item).  A head's selection alone leaves all
// but one compute unit idle, and a gather launched behind it waits for the launch; here every workgroup repeats the part
// that needs all scores (load, minimum and maximum, histogram, scan) and shares the rest: it scatters and ranks its own
// buckets and copies the rows it has found.  The exact path, where it is needed, runs in every workgroup, each copying
// its share of the rows.  Two heads of 16384 scores and 1024 rows: 9.8 + 2.4 us and the gap between -> 10.5 us, of which
// 2.4 load the scores, 3.6 are minimum and maximum, histogram and scan (issue-bound, repeated), 0.8 the copy.
// kPer: scores a thread holds.  Every loop over them is unrolled, and steps without a score are neither free to issue nor to
// fetch, so short blocks take a shorter body: whole call with 16 a thread / as many as it takes (us, graph replay): 512 keys
// 9.9 / 8.0, 1000 (8 heads) 11.4 / 9.6, 2048 13.3 / 11.8, 4096 14.0 / 12.7, 8192 14.3 / 13.5.
constexpr int kMaxSelectParts = 16;
static_assert(kLdsSortMax / kMaxSelectParts + 1 + (int64_t)kMaxBinRank <= kBins && 64 + (int64_t)kMaxBinRank <= kBins,
              "a part's share of the outputs and one bucket more fit sh.fill");

// The exact path of a shared selection: every workgroup sorts the head's l_p largest and writes its share of the indices, outputs
// [*first, *first + *n_out), which it returns.
__device__ __forceinline__ const uint32_t* exact_share(const double* __restrict__ s, int64_t L, int64_t l_p, uint64_t* skeys, uint32_t* sidx,
                                                       int32_t* __restrict__ idx, SelectShared& sh, int part, int n_parts, uint32_t* first, uint32_t* n_out) {
  const int tid = threadIdx.x;
  radix_collect<false>(s, L, l_p, skeys, sidx, sh);
  int64_t n_sort = 1;
  while (n_sort < l_p) n_sort <<= 1;
  __syncthreads();
  for (int64_t i = l_p + tid; i < n_sort; i += kSelectThreads) {   // padding sorts last
    skeys[i] = 0;
    sidx[i] = 0xffffffffu;
  }
  __syncthreads();
  bitonic_sort(skeys, sidx, n_sort);
  *first = (uint32_t)(l_p * part / n_parts);
  *n_out = (uint32_t)(l_p * (part + 1) / n_parts) - *first;
  const uint32_t* rows = sidx + *first;
  for (uint32_t i = tid; i < *n_out; i += kSelectThreads) idx[*first + i] = (int32_t)rows[i];
  return rows;
}

template <int D, int kPer>
__global__ __launch_bounds__(kSelectThreads) void select_gather_kernel(const double* __restrict__ s_ws, View k, View v, int64_t L, int64_t l_p,
                                                                       int64_t cap, int32_t* __restrict__ idx_out, int hkv,
                                                                       bf16_t* __restrict__ k_c, bf16_t* __restrict__ v_c) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  __shared__ SelectShared sh;
  const int part = blockIdx.x, n_parts = gridDim.x, head = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x;
  const int64_t h = (int64_t)b * hkv + head;
  const double* s = s_ws + h * L;
  int32_t* idx = idx_out + h * l_p;
  uint64_t* skeys = reinterpret_cast<uint64_t*>(dyn);
  uint32_t* sidx = reinterpret_cast<uint32_t*>(dyn + cap * sizeof(uint64_t));
  uint16_t* sbin = reinterpret_cast<uint16_t*>(sidx + cap);
  uint32_t first = 0, n_out = 0;
  const uint32_t* rows = sh.fill;
  if (!bucket_rank_select<true, kPer>(s, L, l_p, cap, skeys, sidx, sbin, idx, sh, part, n_parts, &first, &n_out))
    rows = exact_share(s, L, l_p, skeys, sidx, idx, sh, part, n_parts, &first, &n_out);
  __syncthreads();
  copy_rows<D>(k, v, rows, first, n_out, b, head, hkv, l_p, k_c, v_c);
}

// ------------------------------------------------------------------------------------------------
// Selection of long blocks (more scores than a workgroup keeps in registers), a few heads: a histogram by several workgroups
// per head, then selection and gather by several.  One workgroup that reads a head's scores three times, and the gather, took
// 46 of the call's 57 us (one item of 2 heads x 65536 keys, 2000 rows); these take 6.5 and 17, of which 8 read the scores
// (512 KB at what one unit's cache delivers), 1.2 find the bins' bounds and 5 are the buckets, the ranking and the copy.
//
// The coarse map is linear between the smallest and a quarter past the largest of a fixed sample of the head's scores, clamped
// at both ends: monotone, and the same in every workgroup without one that has seen all scores.  It looks at the upper 32
// bits of a score only, so that a bin is a range of these, ordered as signed integers, and the many scores outside a
// workgroup's bins cost one comparison each.
constexpr int kSampleScores = 4096;            // in lines of sixteen
constexpr int kSubBins = 8;                    // LDS bins per coarse bin while counting (fewer collisions)

__device__ __forceinline__ int clamped_bin(float y, int bins) { return (int)fminf(fmaxf(y, 0.0f), (float)(bins - 1)); }      // NaN: 0

__device__ __forceinline__ float upper_value(int hi) { return (float)__hiloint2double(hi, 0); }

// The smallest place in the order whose coarse bin is at least b, kOrderInf + 1 for the one past the last: 64 probes a round,
// one a lane.
__device__ __forceinline__ int first_of_bin(int b, float lo, float inv) {
  const int lane = threadIdx.x & 63;
  int64_t a = upper_order((int)0xfff00000), z = (int64_t)kOrderInf + 1;      // from -infinity
  while (a < z) {
    const int64_t step = (z - a + 63) / 64, probe = a + lane * step;
    const bool there = probe >= z || clamped_bin((upper_value(upper_order((int)probe)) - lo) * inv, kCoarseBins) >= b;
    const uint64_t mask = __builtin_amdgcn_ballot_w64(there);
    if (mask == 0) {
      a += 63 * step + 1;
    } else {
      const int n = __builtin_ctzll(mask);
      const int64_t to = a + n * step;
      if (n > 0) a += (n - 1) * step + 1;
      z = to < z ? to : z;
    }
  }
  return (int)z;
}

// Smallest and largest of a value per thread over the workgroup, in every thread.
__device__ __forceinline__ void block_range(float& lo, float& hi, float* red_lo, float* red_hi) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  lo = wave_min(lo);
  hi = wave_max(hi);
  if (lane == 0) {
    red_lo[wave] = lo;
    red_hi[wave] = hi;
  }
  __syncthreads();
  lo = wave_min(red_lo[lane % (kSelectThreads / 64)]);
  hi = wave_max(red_hi[lane % (kSelectThreads / 64)]);
}

// Counts of one part of a head's scores per coarse bin.  Grid (parts, Hkv, batch); a part has at most kResidentScores.
__global__ __launch_bounds__(kSelectThreads) void coarse_histogram_kernel(const double* __restrict__ s_ws, int64_t L, int hkv, CoarseHistogram* __restrict__ out) {
  __shared__ uint32_t hist[kCoarseBins * kSubBins];
  __shared__ float red_lo[kSelectThreads / 64], red_hi[kSelectThreads / 64];
  const int tid = threadIdx.x, part = blockIdx.x, n_parts = gridDim.x;
  const int64_t head = (int64_t)blockIdx.z * hkv + blockIdx.y;
  const double* s = s_ws + head * L;
  const int64_t per = (L + n_parts - 1) / n_parts, begin = part * per, end = begin + per < L ? begin + per : L;
  constexpr int kPer = kResidentScores / kSelectThreads, kSample = kSampleScores / kSelectThreads;
  const int* upper = reinterpret_cast<const int*>(s) + 1;        // of score j: upper[2 * j]
  int smp[kSample], sc[kPer];
#pragma unroll
  for (int u = 0; u < kSample; ++u) {
    const int i = tid + u * kSelectThreads;
    smp[u] = upper[2 * ((int64_t)(i / 16) * (L / (kSampleScores / 16)) + i % 16)];
  }
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int64_t j = begin + tid + u * kSelectThreads;
    sc[u] = j < end ? upper[2 * j] : 0;
  }
  for (int i = tid; i < kCoarseBins * kSubBins; i += kSelectThreads) hist[i] = 0;
  float lo = INFINITY, hi = -INFINITY;
#pragma unroll
  for (int u = 0; u < kSample; ++u) {
    const float x = upper_value(smp[u]);
    lo = fminf(lo, x);
    hi = fmaxf(hi, x);
  }
  block_range(lo, hi, red_lo, red_hi);
  float inv = (float)kCoarseBins / ((hi - lo) * 1.25f);
  if (!(inv > 0.0f) || !(inv < 1.0e30f)) inv = 0.0f;            // equal, or not finite: no map
#pragma unroll
  for (int u = 0; u < kPer; ++u)
    if (begin + tid + u * kSelectThreads < end) atomicAdd(&hist[clamped_bin((upper_value(sc[u]) - lo) * inv * (float)kSubBins, kCoarseBins * kSubBins)], 1u);
  __syncthreads();
  CoarseHistogram* o = out + head * n_parts + part;
  if (tid < kCoarseBins) {
    uint32_t n = 0;
#pragma unroll
    for (int i = 0; i < kSubBins; ++i) n += hist[tid * kSubBins + i];
    o->count[tid] = (uint16_t)n;
  }
  if (tid == 0) {
    o->lo = lo;
    o->inv = inv;
  }
}

// Grid (parts, Hkv, batch).  Every workgroup adds the parts' histograms and takes the coarse bins whose output offset lies in
// its share of the l_p outputs; it collects the scores of those bins, all it has to know of the others being their number,
// sorts them by buckets as bucket_rank_select does, over their own range, and copies the rows.  Where they are too alike for
// that it sorts them whole; where a bin of its share may be too large for the LDS (most_of_a_bin) it sorts the head's l_p
// largest, and takes its outputs from there.
template <int D>
__global__ __launch_bounds__(kSelectThreads) void long_select_gather_kernel(const double* __restrict__ s_ws, View k, View v, int64_t L, int64_t l_p, int n_hist,
                                                                            const CoarseHistogram* __restrict__ coarse, int32_t* __restrict__ idx_out, int hkv,
                                                                            bf16_t* __restrict__ k_c, bf16_t* __restrict__ v_c) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  __shared__ SelectShared sh;
  constexpr int kItems = (int)(kLdsSortMax / kSelectThreads);
  const int n_parts = gridDim.x, n_heads = hkv * gridDim.z;
  int part = blockIdx.x, head = blockIdx.y, b = blockIdx.z;
  if (n_heads >= 8) {                                        // (fewer are not dealt otherwise, and the divisions take 0.2 to 0.3 us)
    const HeadPart at = head_and_part(part + n_parts * (head + hkv * b), n_parts, n_heads);
    part = at.part;
    head = at.head % hkv;
    b = at.head / hkv;
  }
  const int tid = threadIdx.x;
  const int64_t h = (int64_t)b * hkv + head;
  const double* s = s_ws + h * L;
  int32_t* idx = idx_out + h * l_p;
  uint64_t* skeys = reinterpret_cast<uint64_t*>(dyn);
  uint32_t* sidx = reinterpret_cast<uint32_t*>(dyn + kLdsSortMax * sizeof(uint64_t));
  uint16_t* sbin = reinterpret_cast<uint16_t*>(sidx + kLdsSortMax);

  // ---- the upper halves of the scores, sixteen a thread at a time: the first travel while the bins are found
  constexpr uint32_t kLoads = 16, kStep = kLoads * kSelectThreads;
  const uint32_t n_keys = (uint32_t)L;                       // (32-bit offsets: 64-bit ones were most of the loop's instructions)
  const char* upper = reinterpret_cast<const char*>(s) + 4;
  int hi[kLoads];
  auto load = [&](uint32_t j0) {                             // (past the end: the last score, not taken)
#pragma unroll
    for (uint32_t u = 0; u < kLoads; ++u) {
      const uint32_t j = j0 + u * kSelectThreads;
      hi[u] = *reinterpret_cast<const int*>(upper + (size_t)((j < n_keys ? j : n_keys - 1) * 8u));
    }
  };
  load(tid);

  // ---- the workgroup's coarse bins: thread t has bin kCoarseBins - 1 - t, descending
  const CoarseHistogram* ch = coarse + h * n_hist;
  const float lo = ch->lo, inv = ch->inv;
  const uint32_t from = (uint32_t)(l_p * part / n_parts), to = (uint32_t)(l_p * (part + 1) / n_parts);
  if (tid == 0) {
    sh.b_lo = kCoarseBins;
    sh.b_hi = -1;
    sh.divided = 0;
    sh.cnt = 0;
    sh.crowded = 0;
  }
  for (int i = tid; i < kBins; i += kSelectThreads) sh.hist[i] = 0;
  uint32_t c = 0;
  if (tid < kCoarseBins)
    for (int q = 0; q < n_hist; ++q) c += ch[q].count[kCoarseBins - 1 - tid];
  uint32_t total;
  __syncthreads();
  const uint32_t excl = block_scan_incl(c, sh, &total) - c, most = most_of_a_bin(l_p, n_parts);
  if (c != 0) {                                              // (output l_p lies in a bin too: L > l_p)
    if (excl <= from && from < excl + c) sh.share[0] = first_of_share(from, excl, c, most);
    if (excl <= to && to < excl + c) sh.share[1] = first_of_share(to, excl, c, most);
    if (c > most && excl < to && from < excl + c) sh.divided = 1;
    if (excl >= from && excl < to) {
      atomicMin(&sh.b_lo, kCoarseBins - 1 - tid);
      atomicMax(&sh.b_hi, kCoarseBins - 1 - tid);
    }
  }
  if (tid < kCoarseBins) sh.fill[kCoarseBins - 1 - tid] = excl + c;
  __syncthreads();
  const int b_lo = sh.b_lo, b_hi = sh.b_hi;
  const bool exact = sh.divided != 0;                        // (always where there is no map: all scores are in bin 0)
  const uint32_t first = sh.share[0], end = sh.share[1] < (uint32_t)l_p ? sh.share[1] : (uint32_t)l_p;
  if (first >= end) return;                                  // all of the share lies in a bin that begins before it
  const uint32_t n_out = end - first, n_loc = exact ? 0 : sh.fill[b_lo] - first;      // at most kLdsSortMax
  uint32_t n_sort = 0;                                       // entries left to sort by comparison exchanges, if any
  __syncthreads();

  if (!exact) {
    // ---- collect the indices of the bins' scores, in any order.  Bin 0, where NaNs are counted too, is never one of them: with
    // an output it has at least L - l_p + 1 scores, more than the LDS sorts.
    static_assert(kResidentScores >= 2 * kLdsSortMax, "L > kResidentScores, l_p <= kLdsSortMax: at least L - l_p + 1 scores");
    if (tid < 128) {
      const int bound = first_of_bin(tid < 64 ? b_lo : b_hi + 1, lo, inv);
      if ((tid & 63) == 0) sh.order[tid >> 6] = bound;
    }
    __syncthreads();
    const int lowest = sh.order[0];
    const uint32_t width = order_distance(lowest, sh.order[1]);
    for (uint32_t j0 = tid; j0 < n_keys; j0 += kStep) {
      uint32_t hits = 0;                                     // (few: their stores are one short loop behind the comparisons)
#pragma unroll
      for (uint32_t u = 0; u < kLoads; ++u) hits |= (uint32_t)(order_distance(lowest, upper_order(hi[u])) < width) << u;
      const uint32_t left = (n_keys - j0 + kSelectThreads - 1) / kSelectThreads;
      if (left < kLoads) hits &= (1u << left) - 1;
      if (j0 + kStep < n_keys) load(j0 + kStep);              // travels while the hits are stored
      while (hits != 0) {
        const uint32_t pos = atomicAdd(&sh.cnt, 1u);
        if (pos < n_loc) sidx[pos] = j0 + (uint32_t)__builtin_ctz(hits) * kSelectThreads;      // (always: the same map counted them)
        hits &= hits - 1;
      }
    }
    __syncthreads();
    // ---- buckets of equal width over the collected scores; every thread holds up to kItems of them
    double x[kItems];
    uint32_t ix[kItems], bin[kItems];                        // bucket | arrival order << 11
    float lo2 = INFINITY, hi2 = -INFINITY;
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
      const uint32_t pos = tid + u * kSelectThreads;
      x[u] = 0.0;
      ix[u] = bin[u] = 0;
      if (pos < n_loc) {
        ix[u] = sidx[pos];
        x[u] = s[ix[u]];
      }
    }
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
      if (tid + u * kSelectThreads < n_loc) {
        lo2 = fminf(lo2, (float)x[u]);
        hi2 = fmaxf(hi2, (float)x[u]);
      }
    }
    block_range(lo2, hi2, sh.red_lo, sh.red_hi);
    float inv2 = (float)kBins / (hi2 - lo2);
    if (!(inv2 > 0.0f) || !(inv2 < 1.0e30f)) inv2 = 0.0f;    // all alike: one bucket
#pragma unroll
    for (int u = 0; u < kItems; ++u)
      if (tid + u * kSelectThreads < n_loc) {
        const uint32_t q = (uint32_t)clamped_bin(((float)x[u] - lo2) * inv2, kBins);
        bin[u] = q | (atomicAdd(&sh.hist[q], 1u) << 11);
      }
    __syncthreads();
    const int b0 = kBins - 1 - 2 * tid, b1 = kBins - 2 - 2 * tid;
    const uint32_t c0 = sh.hist[b0], c1 = sh.hist[b1];
    const uint32_t before = block_scan_incl(c0 + c1, sh, &total) - (c0 + c1);
    sh.base[b0] = before;
    sh.base[b1] = before + c0;
    if (c0 > kMaxBinRank || c1 > kMaxBinRank) sh.crowded = 1;
    __syncthreads();
    if (sh.crowded != 0) {
      // too many alike to rank by comparison: what was collected is sorted as it is
#pragma unroll
      for (int u = 0; u < kItems; ++u) {
        const uint32_t pos = tid + u * kSelectThreads;
        if (pos < n_loc) skeys[pos] = score_key(x[u]);       // (sidx[pos] is ix[u])
      }
      n_sort = n_loc;
    } else {
#pragma unroll
      for (int u = 0; u < kItems; ++u)
        if (tid + u * kSelectThreads < n_loc) {
          const uint32_t q = bin[u] & (uint32_t)(kBins - 1), pos = sh.base[q] + (bin[u] >> 11);
          skeys[pos] = score_key(x[u]);
          sidx[pos] = ix[u];
          sbin[pos] = (uint16_t)q;
        }
      __syncthreads();
      uint32_t out_pos[kItems];
#pragma unroll
      for (int u = 0; u < kItems; ++u) {
        const uint32_t pos = tid + u * kSelectThreads;
        out_pos[u] = n_out;
        if (pos >= n_loc) continue;
        const uint32_t q = sbin[pos], begin = sh.base[q], end = begin + sh.hist[q];
        const uint64_t key = skeys[pos];
        const uint32_t index = sidx[pos];
        uint32_t rank = 0;
        for (uint32_t e = begin; e < end; ++e) rank += precedes(skeys[e], sidx[e], key, index) ? 1u : 0u;
        out_pos[u] = begin + rank;
        ix[u] = index;
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kItems; ++u)
        if (out_pos[u] < n_out) {
          sidx[out_pos[u]] = ix[u];
          idx[first + out_pos[u]] = (int32_t)ix[u];
        }
    }
  }
  const uint32_t* rows = sidx;
  if (__builtin_expect(exact, 0)) {
    radix_collect<true>(s, L, l_p, skeys, sidx, sh);
    n_sort = (uint32_t)l_p;
    rows = sidx + first;
  }
  if (n_sort > 0) {
    int64_t n_padded = 1;
    while (n_padded < n_sort) n_padded <<= 1;
    __syncthreads();
    for (int64_t i = n_sort + tid; i < n_padded; i += kSelectThreads) {   // padding sorts last
      skeys[i] = 0;
      sidx[i] = 0xffffffffu;
    }
    __syncthreads();
    bitonic_sort(skeys, sidx, n_padded);
    for (uint32_t i = tid; i < n_out; i += kSelectThreads) idx[first + i] = (int32_t)rows[i];
  }
  __syncthreads();
  copy_rows<D>(k, v, rows, first, n_out, b, head, hkv, l_p, k_c, v_c);
}

// ------------------------------------------------------------------------------------------------
// Short blocks: pooled query, scores, selection and gather in one launch (compresses_at_once: where).  A launch that waits
// for another costs more than what a unit's workgroup does in each step of a short block, so every workgroup adds up the
// pooled query and scores all keys of its head itself, into LDS, and then shares the selection and the rows as above.  Bound
// by the latencies of its steps and by what one unit's cache delivers, (probe rows + keys) * D * 2 bytes a workgroup.  Two
// workgroups a unit leave 64 registers, and 12 bytes a lane go to scratch; with the registers it asks for (70), one a unit, 447
// calls take 1.09 times as long, 0.86 to 1.54 times.
template <int D>
__global__ __launch_bounds__(kSelectThreads, 8) void short_compress_kernel(View q, View k, View v, int L, int64_t l_p, int group, int hkv, double* __restrict__ s_out,
                                                                        int32_t* __restrict__ idx_out, bf16_t* __restrict__ k_c, bf16_t* __restrict__ v_c) {
  constexpr int LPR = D / 8;                   // lanes per row
  constexpr int RPS = kSelectThreads / LPR;    // rows per step of the workgroup
  constexpr int kWaves = kSelectThreads / 64;
  constexpr int UNROLL = 4;
  static_assert(LPR == 8 || LPR == 16, "the cross-lane reduction below is written for 8 or 16 lanes per row");
  static_assert(kShortKeys == kSelectThreads, "one score a thread");
  static_assert(kShortKeys + (int)kMaxBinRank <= kBins, "the outputs of a head's only part and one bucket more fit sh.fill");
  __shared__ SelectShared sh;
  __shared__ double qs[D], scores[kShortKeys];
  __shared__ __attribute__((aligned(16))) unsigned char buf[kWaves * D * 8 > kShortKeys * 14 ? kWaves * D * 8 : kShortKeys * 14];
  double(*qpart)[D] = reinterpret_cast<double(*)[D]>(buf);                  // until the pooled query is complete
  uint64_t* skeys = reinterpret_cast<uint64_t*>(buf);                       // from then on
  uint32_t* sidx = reinterpret_cast<uint32_t*>(buf + kShortKeys * 8);
  uint16_t* sbin = reinterpret_cast<uint16_t*>(buf + kShortKeys * 12);

  const int part = blockIdx.x, n_parts = gridDim.x, head = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = tid % LPR, rsub = tid / LPR;
  const bf16_t* kb = k.ptr + (int64_t)b * k.sb + (int64_t)head * k.sh + 8 * c;
  auto load = [&](int r0, u32x4(&x)[UNROLL]) {
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int j = r0 + u * RPS + rsub;
      x[u] = u32x4{0u, 0u, 0u, 0u};
      if (j < L) x[u] = *reinterpret_cast<const u32x4*>(kb + (int64_t)j * k.st);
    }
  };
  u32x4 x[UNROLL];
  load(0, x);                                  // travel while the pooled query is added up

  // ---- the pooled query: rows (t, g) in steps of RPS, which advance without divisions
  {
    const bf16_t* qb = q.ptr + (int64_t)b * q.sb + (int64_t)head * group * q.sh + 8 * c;
    const int n_rows = (int)q.tokens * group, dt = RPS / group, dg = RPS % group;
    int t = rsub / group, g = rsub % group;
    double sum[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[e] = 0.0;
    for (int r = rsub; r < n_rows; r += UNROLL * RPS) {
      u32x4 y[UNROLL];
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        y[u] = u32x4{0u, 0u, 0u, 0u};
        if (r + u * RPS < n_rows) y[u] = *reinterpret_cast<const u32x4*>(qb + (int64_t)t * q.st + (int64_t)g * q.sh);
        t += dt;
        g += dg;
        if (g >= group) {
          g -= group;
          ++t;
        }
      }
#pragma unroll
      for (int u = 0; u < UNROLL; ++u)
        if (r + u * RPS < n_rows) {            // (whole waves without a row skip the additions)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            sum[2 * e] += bf16_to_f64(y[u][e] & 0xffffu);
            sum[2 * e + 1] += bf16_to_f64(y[u][e] >> 16);
          }
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (LPR == 8) sum[e] += dpp_f64<kDppRor8>(sum[e]);
      sum[e] = add_rows<16>(sum[e]);
      sum[e] = add_rows<32>(sum[e]);
    }
    if (lane < LPR) {
#pragma unroll
      for (int e = 0; e < 8; ++e) qpart[wave][8 * c + e] = sum[e];
    }
    __syncthreads();
    if (tid < D) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) s += qpart[w][tid];
      qs[tid] = s;
    }
    __syncthreads();
  }

  // ---- the scores, by the same sums as score_kernel's
  double qv[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) qv[e] = qs[8 * c + e];
  for (int r0 = 0; r0 < L; r0 += RPS * UNROLL) {
    double a[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      a[u] = 0.0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        a[u] = __builtin_fma(qv[2 * e], bf16_to_f64(x[u][e] & 0xffffu), a[u]);
        a[u] = __builtin_fma(qv[2 * e + 1], bf16_to_f64(x[u][e] >> 16), a[u]);
      }
    }
    load(r0 + RPS * UNROLL, x);
    int u;
    const double acc = reduce_rows<LPR>(a, c, &u);
    const int j = r0 + u * RPS + rsub;
    if (c >= LPR - 4 && j < L) scores[j] = acc;
  }
  __syncthreads();
  const int64_t h = (int64_t)b * hkv + head;
  if (s_out && part == 0 && tid < L) s_out[h * L + tid] = scores[tid];

  // ---- selection and gather, as in select_gather_kernel
  int32_t* idx = idx_out + h * l_p;
  uint32_t first = 0, n_out = 0;
  const uint32_t* rows = sh.fill;
  if (!bucket_rank_select<true, 1>(scores, L, l_p, kShortKeys, skeys, sidx, sbin, idx, sh, part, n_parts, &first, &n_out))
    rows = exact_share(scores, L, l_p, skeys, sidx, idx, sh, part, n_parts, &first, &n_out);
  __syncthreads();
  copy_rows<D>(k, v, rows, first, n_out, b, head, hkv, l_p, k_c, v_c);
}

// Scratch of the entry point that takes no workspace (apbv_compress_kv_noalloc): a fixed array in the code object,
// one copy per GPU at that GPU's own address.  In host code the array's name is only a handle for the symbol lookup
// below; kernels and launch code use the looked-up device address.
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// Per-device one-time set-up (the library's only state): the selection kernel's dynamic-LDS limit, which is a
// per-device property of the loaded code object, and the device address of `scratch`.
constexpr int kMaxDevices = 64;
struct DeviceState {
  bool ready = false;
  void* scratch_ptr = nullptr;
};
std::mutex g_state_mutex;
DeviceState g_state[kMaxDevices];

template <int D>
bool allow_select_lds() {
  for (const void* f : {reinterpret_cast<const void*>(&select_gather_kernel<D, 1>), reinterpret_cast<const void*>(&select_gather_kernel<D, 2>),
                        reinterpret_cast<const void*>(&select_gather_kernel<D, 4>), reinterpret_cast<const void*>(&select_gather_kernel<D, 8>),
                        reinterpret_cast<const void*>(&select_gather_kernel<D, 12>), reinterpret_cast<const void*>(&select_gather_kernel<D, 16>)})
    if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kLdsSortMax * 14)) != hipSuccess) return false;
  return true;
}

apbv_status device_state(DeviceState& out) {
  int device = -1;
  if (hipGetDevice(&device) != hipSuccess || device < 0) return APBV_ERR_LAUNCH;
  if (device >= kMaxDevices) return APBV_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_state_mutex);
  DeviceState& st = g_state[device];
  if (!st.ready) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&select_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)(kLdsSortMax * 14)) != hipSuccess)
      return APBV_ERR_LAUNCH;
    if (!allow_select_lds<64>() || !allow_select_lds<128>()) return APBV_ERR_LAUNCH;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&long_select_gather_kernel<64>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kLdsSortMax * 14)) != hipSuccess ||
        hipFuncSetAttribute(reinterpret_cast<const void*>(&long_select_gather_kernel<128>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kLdsSortMax * 14)) != hipSuccess)
      return APBV_ERR_LAUNCH;
    if (!prepare_matrix_scores()) return APBV_ERR_LAUNCH;
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return APBV_ERR_LAUNCH;
    st.scratch_ptr = ptr;
    st.ready = true;
  }
  out = st;
  return APBV_OK;
}

}  // namespace

size_t compress_workspace_bytes(int batch, int hkv, int d, int64_t L, int64_t l_p) {
  return plan_compress_workspace(batch, hkv, d, L, l_p).total;
}

apbv_status launch_compress(const CompressParams& p_in, hipStream_t stream) {
  CompressParams p = p_in;
  const CompressWorkspace w = plan_compress_workspace(p.batch, p.hkv, p.d, p.L, p.l_p);
  if (p.reducer != APBV_REDUCE_SUM) {
    const apbv_status ok = check_matrix_scores(p);
    if (ok != APBV_OK) return ok;
  }
  DeviceState dev;
  const apbv_status ds = device_state(dev);
  if (ds != APBV_OK) return ds;
  if (p.use_static_scratch) {
    // the workspace is this GPU's copy of the static array: every such call on the GPU shares it
    if (p.reducer != APBV_REDUCE_SUM || w.total > kStaticScratchBytes) return APBV_ERR_WORKSPACE;
    p.workspace = dev.scratch_ptr;
    p.workspace_bytes = kStaticScratchBytes;
  }
  if (p.workspace_bytes < w.total) return APBV_ERR_WORKSPACE;
  unsigned char* ws = static_cast<unsigned char*>(p.workspace);
  double* qbar = reinterpret_cast<double*>(ws + w.qbar_off);
  double* scores = reinterpret_cast<double*>(ws + w.scores_off);
  Launcher launch(stream);

  if (p.reducer != APBV_REDUCE_SUM) {
    // the non-linear reductions form the logit matrix on the matrix cores (score_matrix.hip); their row
    // statistics live behind the selection workspace
    const size_t stats_off = align_up(w.total, 256);
    const size_t stats_bytes = matrix_scores_workspace_bytes(p.reducer, p.batch, p.hkv, p.q_probe.tokens * p.group, p.L);
    if (p.workspace_bytes < stats_off + stats_bytes) return APBV_ERR_WORKSPACE;
    const apbv_status st = launch_matrix_scores(p, scores, ws + stats_off, stream);
    if (st != APBV_OK) return st;
  } else if (const int parts = compresses_at_once(p.q_probe.tokens * p.group, p.d, (int64_t)p.hkv * p.batch, p.L, p.l_p); parts > 0) {
    auto compress = [&](auto kernel) {
      launch(kernel, dim3((unsigned)parts, p.hkv, p.batch), dim3(kSelectThreads), 0, p.q_probe, p.k, p.v, (int)p.L, p.l_p, p.group, p.hkv, p.scores_out, p.idx_out, p.k_c, p.v_c);
    };
    p.d == 128 ? compress(short_compress_kernel<128>) : compress(short_compress_kernel<64>);
    return launch.status();
  } else {
    const int64_t n_rows = p.q_probe.tokens * p.group;
    const bool pooled = pools_in_scores(n_rows, p.d, (int64_t)p.hkv * p.batch, p.L);
    const int n_split = pool_splits(n_rows, (int64_t)p.batch * p.hkv);
    if (!pooled) {
      // pooled query, as n_split partial sums
      const int64_t rows_per_split = (n_rows + n_split - 1) / n_split;
      const bool wide = rows_per_split >= 4 * 1024 / (p.d / 8);
      const dim3 pool_grid(n_split, p.hkv, p.batch);
      if (p.d == 128 && wide)
        launch(pool_query_kernel<128, 1024>, pool_grid, dim3(1024), 0, p.q_probe, p.q_probe.tokens, p.group, qbar, p.hkv, n_split);
      else if (p.d == 128)
        launch(pool_query_kernel<128, 256>, pool_grid, dim3(256), 0, p.q_probe, p.q_probe.tokens, p.group, qbar, p.hkv, n_split);
      else if (wide)
        launch(pool_query_kernel<64, 1024>, pool_grid, dim3(1024), 0, p.q_probe, p.q_probe.tokens, p.group, qbar, p.hkv, n_split);
      else
        launch(pool_query_kernel<64, 256>, pool_grid, dim3(256), 0, p.q_probe, p.q_probe.tokens, p.group, qbar, p.hkv, n_split);
    }
    // scores: one outer iteration per workgroup: 4 rows in flight per thread, many small workgroups
    const int rows_per_block = 4 * 256 / (p.d / 8);
    dim3 grid((unsigned)((p.L + rows_per_block - 1) / rows_per_block), p.hkv, p.batch);
    auto score = [&](auto kernel) { launch(kernel, grid, dim3(256), 0, p.k, p.L, qbar, n_split, scores, p.scores_out, p.hkv, rows_per_block, p.q_probe, p.group); };
    if (p.d == 128)
      pooled ? score(score_kernel<128, true>) : score(score_kernel<128, false>);
    else
      pooled ? score(score_kernel<64, true>) : score(score_kernel<64, false>);
  }
  // (a few heads' selection is shared by several workgroups each, in parts of at least 32 rows, and copies its rows too)
  int64_t n_parts = p.l_p / 32 < kMaxSelectParts ? p.l_p / 32 : kMaxSelectParts;
  n_parts = n_parts > 1 ? n_parts : 1;
  if (share_selection((int64_t)p.hkv * p.batch, p.L, p.l_p, w)) {
    const dim3 grid((unsigned)n_parts, p.hkv, p.batch);
    const size_t dyn = (size_t)w.n_sort * 14;
    auto select = [&](auto kernel) { launch(kernel, grid, dim3(kSelectThreads), dyn, scores, p.k, p.v, p.L, p.l_p, w.n_sort, p.idx_out, p.hkv, p.k_c, p.v_c); };
    auto select_up_to = [&](auto per) {
      constexpr int kPer = decltype(per)::value;
      p.d == 128 ? select(select_gather_kernel<128, kPer>) : select(select_gather_kernel<64, kPer>);
    };
    switch ((p.L + kSelectThreads - 1) / kSelectThreads) {
      case 1: select_up_to(std::integral_constant<int, 1>{}); break;
      case 2: select_up_to(std::integral_constant<int, 2>{}); break;
      case 3: case 4: select_up_to(std::integral_constant<int, 4>{}); break;
      case 5: case 6: case 7: case 8: select_up_to(std::integral_constant<int, 8>{}); break;
      case 9: case 10: case 11: case 12: select_up_to(std::integral_constant<int, 12>{}); break;
      default: select_up_to(std::integral_constant<int, 16>{});
    }
  } else if (const LongSelection plan = plan_long_selection((int64_t)p.hkv * p.batch, p.d, p.L, p.l_p, w); plan.n_parts > 0) {
    // the histograms lie where the partial sums of the pooled queries were
    CoarseHistogram* coarse = reinterpret_cast<CoarseHistogram*>(ws + w.qbar_off);
    launch(coarse_histogram_kernel, dim3((unsigned)plan.n_hist, p.hkv, p.batch), dim3(kSelectThreads), 0, scores, p.L, p.hkv, coarse);
    const dim3 grid((unsigned)plan.n_parts, p.hkv, p.batch);
    const size_t dyn = (size_t)kLdsSortMax * 14;
    if (p.d == 128)
      launch(long_select_gather_kernel<128>, grid, dim3(kSelectThreads), dyn, scores, p.k, p.v, p.L, p.l_p, plan.n_hist, coarse, p.idx_out, p.hkv, p.k_c, p.v_c);
    else
      launch(long_select_gather_kernel<64>, grid, dim3(kSelectThreads), dyn, scores, p.k, p.v, p.L, p.l_p, plan.n_hist, coarse, p.idx_out, p.hkv, p.k_c, p.v_c);
  } else if (p.l_p > 0) {
    // select + order
    if (w.sort_in_global) {
      launch(select_kernel<true>, dim3(p.hkv, p.batch), dim3(kSelectThreads), 0, scores, p.L, p.l_p, w.n_sort, p.idx_out, reinterpret_cast<uint64_t*>(ws + w.sort_keys_off), reinterpret_cast<uint32_t*>(ws + w.sort_idx_off), p.hkv);
    } else {
      const size_t dyn = (size_t)w.n_sort * 14;
      launch(select_kernel<false>, dim3(p.hkv, p.batch), dim3(kSelectThreads), dyn, scores, p.L, p.l_p, w.n_sort, p.idx_out, nullptr, nullptr, p.hkv);
    }
    // gather
    const int64_t n_items = p.l_p * p.hkv * (p.d / 8);
    dim3 grid((unsigned)((n_items + 255) / 256), p.batch);
    if (p.d == 128)
      launch(gather_kernel<128>, grid, dim3(256), 0, p.k, p.v, p.idx_out, p.l_p, p.hkv, p.L, p.k_c, p.v_c);
    else
      launch(gather_kernel<64>, grid, dim3(256), 0, p.k, p.v, p.idx_out, p.l_p, p.hkv, p.L, p.k_c, p.v_c);
  }
  return launch.status();
}

}  // namespace apbv
