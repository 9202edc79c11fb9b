// Attention of a short query block over a long key axis for gfx950 (Eq. 5, and a decoding step): the launches of
// apbv_query_attention other than attention.hip's own (choose_query_plan picks one of four).  Operation, mask, softmax
// and MFMA mapping are those of attention.hip; what differs is how the work is cut.
//
// Rows.  The G query heads that share a KV head are G more rows of one problem: row r = i * G + g of (batch item, KV
// head) is query i of head kvh * G + g.  A decoding step of one query then fills G of a 16-row MFMA block and reads
// every key once, where one workgroup per query head read them G times and computed 63 padding rows of 64.
//
// Keys.  At most 32 rows per KV head are bound by HBM, and need many loads in flight rather than a shared tile: every
// WAVE walks its own range of the key axis with its own LDS rings (two 32-key tiles of K and of V, filled by LDS-direct
// loads) and no barrier: the rings' order is kept by counting the wave's own loads.  The waves of a workgroup take
// consecutive ranges of the same rows and combine their results in LDS at the end (float32), so a workgroup writes one
// partial result per row.  One query over 133120 keys, 16 / 2 heads of 128 (136 MB): 94 -> 24.1 us, 5.7 TB/s.
//
// More rows have matrix work to do and share their tiles among the waves: packed_attention.hip.  With the merge, against a
// workgroup per query head: 64 queries x 16 / 2 heads over 131072 keys 88 -> 70 us, 17 queries x 28 / 4 over 2 x 5000 keys 32 -> 15 us;
// this kernel with two blocks of rows per wave was slower than a workgroup per query head on the first (125 / 106 us).
#include "apbv_common.h"
#include "attention_tiles.h"

namespace apbv {
namespace {

// Waves per workgroup: as many as have room for their rings below 64 KB (the reach of an LDS-direct load).
template <int D>
struct QueryShape {
  using T = Tile<D, 1>;                                    // a tile is loaded and read by one wave
  static constexpr int kRingBytes = 4 * T::TILE_BYTES;     // [K0 | K1 | V0 | V1] of one wave
  static constexpr int kWaves = 65536 / kRingBytes;
};

// Work item: the at most 16*NQ rows of (batch item b, KV head kvh), key range `split`.
template <int D, int NQ>
__device__ __forceinline__ void query_workgroup(const AttnParams& p, const int b, const int kvh, const int split) {
  using S = QueryShape<D>;
  using T = typename S::T;
  constexpr int W = S::kWaves;
  constexpr int kRows = 16 * NQ;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[W][S::kRingBytes];
  static_assert(sizeof(lds) <= 65536, "LDS-direct loads reach the first 64 KB");
  static_assert(kRows * D * 4 <= S::kRingBytes, "a wave's float32 result fits its rings");

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15;
  const int lg = lane >> 4;
  const int n_rows = (int)p.L * p.group;                   // at most kRows

  Segs ks, vs;
  key_segments(p, b, kvh, ks, vs);

  // ---- the wave's tiles [tb, te): an equal share of the workgroup's range (planned in 64-key units)
  auto last_key = [&](int64_t i) { return (i + p.n_vis < p.s_kv - 1) ? i + p.n_vis : p.s_kv - 1; };
  const int64_t n_vis_tiles = last_key(p.L - 1) / kBN + 1;
  const int64_t per_split = (int64_t)p.tiles_per_split * (64 / kBN);
  const int64_t s_begin = split * per_split < n_vis_tiles ? split * per_split : n_vis_tiles;
  const int64_t s_end = s_begin + per_split < n_vis_tiles ? s_begin + per_split : n_vis_tiles;
  const int per_wave = (int)((s_end - s_begin + W - 1) / W);
  const int tb = __builtin_amdgcn_readfirstlane((int)(s_begin + wave * per_wave < s_end ? s_begin + wave * per_wave : s_end));
  const int te = __builtin_amdgcn_readfirstlane((int)(tb + per_wave < s_end ? tb + per_wave : s_end));
  const int t_mask = __builtin_amdgcn_readfirstlane((int)((last_key(0) + 1) / kBN));   // first tile with a key some row cannot see

  // ---- the rings: K(t), V(t) live in slot (t - tb) & 1
  TileStream<D, 1, false> kst;
  TileStream<D, 1, true> vst;
  kst.init(ks, p.s_kv, 0, lane, tb);
  vst.init(vs, p.s_kv, 0, lane, tb);
  const unsigned char* ring = lds[wave];
  const uint32_t ring_addr = __builtin_amdgcn_readfirstlane(lds_addr(ring));
  auto k_slot = [&](int s) { return ring + s * T::TILE_BYTES; };
  auto v_slot = [&](int s) { return ring + (2 + s) * T::TILE_BYTES; };
  auto issue_k = [&](int s) { kst.issue_until(ring_addr + s * T::TILE_BYTES, te - 1); };
  auto issue_v = [&](int s) { vst.issue_until(ring_addr + (2 + s) * T::TILE_BYTES, te - 1); };
  if (tb < te) {
#pragma unroll 1
    for (int i = 0; i < 2; ++i) issue_k(i);
    issue_v(0);
  }

  // ---- Q^T fragments; this lane's rows 16*nq + li
  bf16x8 qf[T::KSD][NQ];
  int jlast[NQ];                                           // last visible virtual key of each row
#pragma unroll
  for (int nq = 0; nq < NQ; ++nq) {
    const int r = 16 * nq + li < n_rows ? 16 * nq + li : n_rows - 1;
    const int i = r / p.group;
    const int h = kvh * p.group + r % p.group;
    jlast[nq] = (int)last_key(i);
    const bf16_t* qrow = p.q.ptr + (int64_t)b * p.q.sb + (int64_t)h * p.q.sh + i * p.q.st;
#pragma unroll
    for (int c = 0; c < T::KSD; ++c) qf[c][nq] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(qrow + 32 * c + 8 * lg));
  }

  // ---- per-lane LDS read offsets (attention.hip: K rows as the A operand of S^T, V transposed as that of O^T)
  int k_off[T::KSD], v_off[T::DBN];
#pragma unroll
  for (int c = 0; c < T::KSD; ++c) k_off[c] = li * T::ROW_BYTES + (((4 * c + lg) ^ T::fk(li)) << 4);
  {
    const int row = 4 * lg + (li >> 2);
#pragma unroll
    for (int d = 0; d < T::DBN; ++d)
      v_off[d] = row * T::ROW_BYTES + (((2 * d + ((li & 3) >> 1)) ^ T::fv(row)) << 4) + (li & 1) * 8;
  }

  f32x4 o[T::DBN][NQ];
  float m_ref[NQ], m_sub[NQ], s_far[NQ], l_run[NQ];        // as in attention.hip
#pragma unroll
  for (int nq = 0; nq < NQ; ++nq) {
#pragma unroll
    for (int d = 0; d < T::DBN; ++d) o[d][nq] = f32x4{0.f, 0.f, 0.f, 0.f};
    m_ref[nq] = s_far[nq] = -INFINITY;
    m_sub[nq] = l_run[nq] = 0.f;
  }
  const float inv_scale_log2 = 1.0f / p.scale_log2;

  typedef f32x4 STile[2][NQ];
  auto qk = [&](const unsigned char* kt, STile& s) {
#pragma unroll
    for (int c = 0; c < T::KSD; ++c)
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) {
        const bf16x8 a = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(kt + mb * 16 * T::ROW_BYTES + k_off[c]));
#pragma unroll
        for (int nq = 0; nq < NQ; ++nq)
          s[mb][nq] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[c][nq], c == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[mb][nq], 0, 0, 0);
      }
  };
  // mask, this lane's largest logit per row, and the reference maximum (moved only past the threshold)
  auto settle = [&](STile& s, int t) {
    if (t >= t_mask) {
#pragma unroll
      for (int nq = 0; nq < NQ; ++nq) {
        const int jrel = jlast[nq] - t * kBN;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (16 * mb + 4 * lg + r > jrel) s[mb][nq][r] = -INFINITY;
      }
    }
    float lm[NQ];
    bool far = false;
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq) {
      float mx = __builtin_fmaxf(s[0][nq][0], s[0][nq][1]);
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int r = (mb == 0 ? 2 : 0); r < 4; ++r) mx = __builtin_fmaxf(mx, s[mb][nq][r]);
      lm[nq] = mx;
      far = far || mx > s_far[nq];
    }
    if (__builtin_amdgcn_ballot_w64(far) != 0) {
#pragma unroll
      for (int nq = 0; nq < NQ; ++nq) {
        float mx = lm[nq];
        {
          auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
          mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
        }
        {
          auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
          mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
        }
        const float m_new = fmaxf(m_ref[nq], mx * p.scale_log2);
        const float alpha = m_new > -INFINITY ? __builtin_amdgcn_exp2f(m_ref[nq] - m_new) : 1.f;
        m_ref[nq] = m_new;
        m_sub[nq] = m_new > -INFINITY ? m_new : 0.f;
        s_far[nq] = (m_new + kRescaleThreshold) * inv_scale_log2;
        l_run[nq] *= alpha;
#pragma unroll
        for (int d = 0; d < T::DBN; ++d) o[d][nq] *= alpha;
      }
    }
  };
  auto probabilities = [&](const STile& s, u32x4 (&pw)[NQ]) {
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq)
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          f32x2 xy = {__builtin_amdgcn_exp2f(__builtin_fmaf(s[mb][nq][e], p.scale_log2, -m_sub[nq])),
                      __builtin_amdgcn_exp2f(__builtin_fmaf(s[mb][nq][e + 1], p.scale_log2, -m_sub[nq]))};
          const bf16x2 c = __builtin_convertvector(xy, bf16x2);
          l_run[nq] = __builtin_amdgcn_fdot2_f32_bf16(c, bf16x2{(__bf16)1.0f, (__bf16)1.0f}, l_run[nq], false);
          pw[nq][2 * mb + (e >> 1)] = __builtin_bit_cast(uint32_t, c);
        }
  };
  auto pv = [&](const unsigned char* vt, const u32x4 (&pw)[NQ]) {
#pragma unroll
    for (int d = 0; d < T::DBN; ++d) {
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((APBV_LDS(s16x4))(vt + v_off[d]));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((APBV_LDS(s16x4))(vt + 16 * T::ROW_BYTES + v_off[d]));
      const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
      for (int nq = 0; nq < NQ; ++nq)
        o[d][nq] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, pw[nq]), o[d][nq], 0, 0, 0);
    }
  };

  // ---- key loop.  At the top of step t S^T(t) is in registers and settled, and the loads of K(t+1), V(t) are
  // outstanding in that order; the slots of K(t) and V(t-1) are free (every LDS read of them has returned: lgkmcnt 0)
  // and take K(t+2), V(t+1).  S^T(t+1) is formed on the matrix pipe beside the exponentials of tile t.  Past the range's
  // end the last tile is requested again (and its S^T formed, never used): one body for all steps.  The code is kept
  // short on purpose: a launch starts with a cold instruction cache, and straight-line code runs at about 1 byte/ns.
  STile s_cur, s_nxt;
  auto step = [&](int t, auto slot, STile& sc, STile& sn) {
    constexpr int a = decltype(slot)::value;               // (t - tb) & 1
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    issue_k(a);
    issue_v(a ^ 1);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * T::LOADS) : "memory");         // V(t), K(t+2), V(t+1) may be outstanding
    u32x4 pw[NQ];
    qk(k_slot(a ^ 1), sn);
    probabilities(sc, pw);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * T::LOADS) : "memory");         // K(t+2), V(t+1)
    pv(v_slot(a), pw);
    if (t + 1 < te) settle(sn, t + 1);
  };
  if (tb < te) {
    __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0), known to the compiler: Q and the first tiles
    qk(k_slot(0), s_cur);
    settle(s_cur, tb);
    for (int t = tb;; t += 2) {
      step(t, std::integral_constant<int, 0>{}, s_cur, s_nxt);
      if (t + 1 >= te) break;
      step(t + 1, std::integral_constant<int, 1>{}, s_nxt, s_cur);
      if (t + 2 >= te) break;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // no load into the rings is left when they are reused below
  }

  // ---- combine the waves' results: every wave scales its O by exp2(m - M) / (sum of all), M the rows' maximum over
  // the waves, and the scaled results are added.  Row r of the tile: m at stat[r], l at stat[kRows + r] of each wave.
  float l_tot[NQ];
#pragma unroll
  for (int nq = 0; nq < NQ; ++nq) {
    float x = l_run[nq];
    {
      auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
      x = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    }
    {
      auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
      x = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    }
    l_tot[nq] = x;
  }
  float* stat = reinterpret_cast<float*>(lds[wave]);
  __syncthreads();
  if (lg == 0) {
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq) {
      stat[16 * nq + li] = m_ref[nq];
      stat[kRows + 16 * nq + li] = l_tot[nq];
    }
  }
  __syncthreads();
  float factor[NQ];
#pragma unroll
  for (int nq = 0; nq < NQ; ++nq) {
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) m = fmaxf(m, reinterpret_cast<const float*>(lds[w])[16 * nq + li]);
    const float m0 = m > -INFINITY ? m : 0.f;              // a row without any visible key in the range: all weights 0
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float* sw = reinterpret_cast<const float*>(lds[w]);
      l = __builtin_fmaf(sw[kRows + 16 * nq + li], __builtin_amdgcn_exp2f(sw[16 * nq + li] - m0), l);
    }
    factor[nq] = l > 0.f ? __builtin_amdgcn_exp2f(m_ref[nq] - m0) / l : 0.f;
    const int r = 16 * nq + li;
    if (p.lse != nullptr && wave == 0 && lg == 0 && r < n_rows) {
      const int i = r / p.group;
      const int h = kvh * p.group + r % p.group;
      p.lse[(int64_t)split * p.split_stride_lse + ((int64_t)b * p.hq + h) * p.L + i] =
          l > 0.f ? (m + __builtin_amdgcn_logf(l)) * 0.6931471805599453f : -INFINITY;
    }
  }
  __syncthreads();
  // O as float32 [row][D], the 16-byte chunks of a row swizzled by the row so that 16 rows' chunks spread over the banks
  constexpr int kChunks = D / 4;
  {
    f32x4* mine = reinterpret_cast<f32x4*>(lds[wave]);
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq)
#pragma unroll
      for (int d = 0; d < T::DBN; ++d) mine[(16 * nq + li) * kChunks + ((4 * d + lg) ^ li)] = o[d][nq] * factor[nq];
  }
  __syncthreads();
  for (int item = threadIdx.x; item < kRows * (D / 8); item += 64 * W) {
    const int row = item / (D / 8), c = item % (D / 8);
    if (row >= n_rows) break;
    f32x4 x0 = {0.f, 0.f, 0.f, 0.f}, x1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const f32x4* src = reinterpret_cast<const f32x4*>(lds[w]) + row * kChunks;
      x0 += src[(2 * c) ^ (row & 15)];
      x1 += src[(2 * c + 1) ^ (row & 15)];
    }
    u32x4 y;
    y.x = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{x0.x, x0.y}), bf16x2));
    y.y = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{x0.z, x0.w}), bf16x2));
    y.z = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{x1.x, x1.y}), bf16x2));
    y.w = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{x1.z, x1.w}), bf16x2));
    const int i = row / p.group;
    const int h = kvh * p.group + row % p.group;
    *reinterpret_cast<u32x4*>(p.out + (int64_t)split * p.split_stride_out + (((int64_t)b * p.L + i) * p.hq + h) * D + 8 * c) = y;
  }
}

// One workgroup per (batch item, KV head, key range).
template <int D, int NQ>
__global__ __launch_bounds__(64 * QueryShape<D>::kWaves, D == 128 ? 1 : 2) void query_attention_kernel(const AttnParams p) {
  const int split = blockIdx.x % p.n_splits, bh = blockIdx.x / p.n_splits;
  query_workgroup<D, NQ>(p, bh / p.hkv, bh % p.hkv, split);
}

template <int D, int NQ>
apbv_status launch_query_variant(const AttnParams& p, hipStream_t stream) {
  const int64_t n_blocks = (int64_t)p.batch * p.hkv * p.n_splits;
  if (n_blocks > 0x7fffffff) return APBV_ERR_UNSUPPORTED;
  Launcher launch(stream);
  launch(query_attention_kernel<D, NQ>, dim3((unsigned)n_blocks), dim3(64 * QueryShape<D>::kWaves), 0, p);
  return launch.status();
}

template <int D>
apbv_status launch_query_rows(const AttnParams& p, hipStream_t stream) {
  const int64_t rows = p.L * p.group;
  if (rows <= 16) return launch_query_variant<D, 1>(p, stream);
  if (rows <= kQueryWaveRows) return launch_query_variant<D, 2>(p, stream);
  return APBV_ERR_UNSUPPORTED;
}

}  // namespace

apbv_status launch_query_attention(const AttnParams& p, int head_dim, QueryKernel kernel, hipStream_t stream) {
  switch (kernel) {
    case QueryKernel::kPerHead: return launch_host_attention(p, head_dim, stream);
    case QueryKernel::kPacked128: return launch_packed_attention(p, head_dim, kQueryShortRows, stream);
    case QueryKernel::kPacked256: return launch_packed_attention(p, head_dim, kAttnQueryTile, stream);
    case QueryKernel::kWave: break;
  }
  if (head_dim == 128) return launch_query_rows<128>(p, stream);
  if (head_dim == 64) return launch_query_rows<64>(p, stream);
  return APBV_ERR_UNSUPPORTED;
}

}  // namespace apbv
