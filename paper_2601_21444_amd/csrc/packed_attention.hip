// Attention of a query block whose heads of a KV group are packed into the rows, for gfx950 (Eq. 5): the workgroups of
// apbv_query_attention for more rows per KV head than one wave takes.  Row r = i * G + g of (batch item, KV head) is query i
// of head kvh * G + g, so a key is read once for all heads that share it.  Operation, mask, softmax and key loop are
// those of attention.hip; the matrix instruction is not.
//
// Such launches are cut into as many key ranges as it takes to give every compute unit one workgroup, one wave a SIMD.
// There a 16x16x32 matrix instruction and the vector instructions of its wave add up (16 + 4.2 n cycles, measured); under
// a 32x32x16 one (32 cycles) four to five vector instructions are free.  MFMA mapping (v_mfma_f32_32x32x16_bf16; with
// c = lane % 32, h = lane / 32: A is 32x16 with the lane holding row c, k-slots 8h..8h+7; B is 16x32 with the lane holding
// column c, the same k-slots; D is 32x32 with the lane holding column c, register i row 8(i/4) + 4h + i%4):
//   S^T = K Q^T   : A = 32 keys x 16 head-dim columns, B = Q^T in registers: a lane holds 16 keys of ONE row.
//   O^T = V^T P^T : B = registers 8m..8m+7 of S^T for the m-th 16 keys (slot 8h + e: key 16m + 8(e/4) + 4h + e%4);
//                   A = V^T by two transposing reads of four consecutive keys each.
// Bound by the sum of what a lone wave issues (about 750 cycles a tile of 32 keys from resident LDS, 1100 with the loads and
// barriers, of which 520 are matrix instructions) and the start and end of the workgroups (6 to 7 us).  Per call with the merge, workgroups of
// 16x16x32 / these (us): 64 queries x 16 / 2 heads of 128 over 16512 keys 22.7 / 20.4, 17 x 28 / 4 over 2 x 4150 17.3 / 15.1,
// 64 x 8 / 2 of 64 over 16512 13.2 / 11.6, 300 x 8 / 2 of 64, two items, over 5100 21.2 / 19.0; where HBM or power bounds
// them they are equal (512 x 16 / 2 over 100000 338 / 337).  Results against float64 are as before (same stages and widths).
#include "apbv_common.h"
#include "attention_tiles.h"

namespace apbv {
namespace {

constexpr int kPackedRing = 4;      // K tiles, and V tiles, resident in LDS


__device__ __forceinline__ f32x16 mfma32(const bf16x8 a, const bf16x8 b, const f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Work item: the 32*W rows from row tile `rt` of (batch item b, KV head kvh), key range `split`.
template <int D, int W>
__device__ __forceinline__ void packed_workgroup(const AttnParams& p, const int rt, const int b, const int kvh, const int split) {
  using T = Tile<D, W, true>;
  constexpr int kRows = 32 * W;
  constexpr int KS = D / 16;                 // matrix instructions of S^T
  constexpr int DB = D / 32;                 // 32-row blocks of O^T, two matrix instructions each
  __shared__ __attribute__((aligned(1024))) unsigned char k_lds[kPackedRing][T::TILE_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char v_lds[kPackedRing][T::TILE_BYTES];
  static_assert(2 * kPackedRing * T::TILE_BYTES <= 65536, "LDS-direct loads reach the first 64 KB");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 31, hh = lane >> 5;

  const int n_rows = (int)p.L * p.group;
  const int r0 = rt * kRows, rw = r0 + wave * 32;             // first row of the workgroup, of the wave
  auto query_of = [&](int r) { return (int)((uint32_t)(r < n_rows ? r : n_rows - 1) / (uint32_t)p.group); };
  const int row = rw + c < n_rows ? rw + c : n_rows - 1;
  const int qi = query_of(row), head = kvh * p.group + (row - qi * p.group);

  Segs ks, vs;
  key_segments(p, b, kvh, ks, vs);

  // ---- Q^T fragments (B operand of S^T): elements 16*kk + 8*hh .. +7 of the lane's row
  bf16x8 qf[KS];
  {
    const bf16_t* qrow = p.q.ptr + (int64_t)b * p.q.sb + (int64_t)head * p.q.sh + (int64_t)qi * p.q.st + 8 * hh;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) qf[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(qrow + 16 * kk));
  }

  // ---- per-lane LDS read offsets.  K: row c, 16-byte chunk (2*kk + hh) ^ fk(c).  V: within a 16-lane group source lane s
  // addresses key row 4*hh + s/4 (+ 16m + 8 for the second four keys, as immediates), head-dim columns
  // 32*db + 16*(group % 2) + 4*(s%4) .. +3
  int k_off[KS], v_off[DB];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) k_off[kk] = c * T::ROW_BYTES + (((2 * kk + hh) ^ T::fk(c)) << 4);
  {
    const int s = lane & 15, vrow = 4 * hh + (s >> 2);
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      const int chunk = 4 * db + 2 * ((lane >> 4) & 1) + ((s & 3) >> 1);
      v_off[db] = vrow * T::ROW_BYTES + ((chunk ^ T::fv(vrow)) << 4) + (s & 1) * 8;
    }
  }

  // ---- online softmax state of the lane's row (attention.hip); the two lane halves hold disjoint keys
  f32x16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
  float m_ref = -INFINITY, m_sub = 0.f, s_far = -INFINITY, l_run = 0.f;
  const float inv_scale_log2 = 1.0f / p.scale_log2;

  // ---- tiles: the workgroup walks [t_begin, n_tiles), the wave computes [t_begin, n_w), masked from t_mask on
  const int s_kv = (int)p.s_kv, n_vis = (int)p.n_vis;         // at most 3 * 2^24
  auto last_key = [&](int i) { return i + n_vis < s_kv - 1 ? i + n_vis : s_kv - 1; };
  const int n_tiles_vis = last_key(query_of(r0 + kRows - 1)) / kBN + 1;
  const int64_t per_split = (int64_t)p.tiles_per_split * (64 / kBN), begin = split * per_split;
  const int t_begin = __builtin_amdgcn_readfirstlane((int)(begin < n_tiles_vis ? begin : n_tiles_vis));
  const int n_tiles = __builtin_amdgcn_readfirstlane((int)(begin + per_split < n_tiles_vis ? begin + per_split : n_tiles_vis));
  const int t_last_wave = last_key(query_of(rw + 31)) / kBN;
  const int n_w = __builtin_amdgcn_readfirstlane(t_last_wave + 1 < n_tiles ? t_last_wave + 1 : n_tiles);
  const int t_mask = __builtin_amdgcn_readfirstlane((last_key(query_of(rw)) + 1) / kBN);
  const int jlast = last_key(qi);

  typedef u32x4 PTile[2];
  typedef bf16x8 KFrags[KS];
  auto read_k = [&](const unsigned char* kt, int kk) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(kt + k_off[kk])); };
  auto load_k = [&](const unsigned char* kt, KFrags& kf) {
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) kf[kk] = read_k(kt, kk);
  };
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  auto apply_mask = [&](f32x16& s, int t) {
    const int jrel = jlast - t * kBN;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (8 * (i / 4) + 4 * hh + i % 4 > jrel) s[i] = -INFINITY;
  };
  auto lane_max = [&](const f32x16& s) {
    float mx = __builtin_fmaxf(s[0], s[1]);
#pragma unroll
    for (int i = 2; i < 16; ++i) mx = __builtin_fmaxf(mx, s[i]);
    return mx;
  };
  // lazy rescaling (attention.hip)
  auto advance_reference = [&](float lm) {
    if (__builtin_amdgcn_ballot_w64(lm > s_far) != 0) {
      auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(lm), __float_as_uint(lm), false, false);
      const float mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
      const float m_new = fmaxf(m_ref, mx * p.scale_log2);
      const float alpha = m_new > -INFINITY ? __builtin_amdgcn_exp2f(m_ref - m_new) : 1.f;
      m_ref = m_new;
      m_sub = m_new > -INFINITY ? m_new : 0.f;
      s_far = (m_new + kRescaleThreshold) * inv_scale_log2;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
    }
  };

  // ---- one tile: finishes tile t (S^T in sc, V at vt) while it forms S^T of tile t+1 (K fragments in kf) into sn and takes
  // its lane maximum.  First the KS matrix instructions of S^T, then DB of O^T for the first 16 keys, then DB for the second;
  // the exponentials run beside the first two groups, pair by pair (stages F scale and subtract, E exp2, C round, D row
  // sum), the first four pairs done before the second group needs them.
  auto tile = [&](auto prefetch_k, KFrags& kf, const unsigned char* kt_after, const unsigned char* vt, const f32x16& sc, f32x16& sn, float& lm, auto&& between) {
    constexpr bool kPrefetchK = decltype(prefetch_k)::value;
    constexpr int kMfma = KS + 2 * DB, kExp = KS + DB;
    float xf[8][2];
    uint32_t cw[8];
    PTile pw;
    s16x4 vf[2][DB][2];
    auto stage_f = [&](int pi) {
      xf[pi][0] = __builtin_fmaf(sc[2 * pi], p.scale_log2, -m_sub);
      xf[pi][1] = __builtin_fmaf(sc[2 * pi + 1], p.scale_log2, -m_sub);
    };
    auto stage_e = [&](int pi) {
      xf[pi][0] = __builtin_amdgcn_exp2f(xf[pi][0]);
      xf[pi][1] = __builtin_amdgcn_exp2f(xf[pi][1]);
    };
    auto stage_c = [&](int pi) {
      f32x2 xy = {xf[pi][0], xf[pi][1]};
      cw[pi] = __builtin_bit_cast(uint32_t, __builtin_convertvector(xy, bf16x2));
      pw[pi >> 2][pi & 3] = cw[pi];
    };
    auto stage_d = [&](int pi) {
      l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, cw[pi]), bf16x2{(__bf16)1.0f, (__bf16)1.0f}, l_run, false);
    };
    static_for<kMfma>([&](auto I) {
      constexpr int i = I;
      if constexpr (i < KS) {
        sn = mfma32(kf[i], qf[i], i == 0 ? zero : sn);
        constexpr int v0 = (4 * DB * i) / KS, v1 = (4 * DB * (i + 1)) / KS;
        static_for<v1 - v0>([&](auto J) {
          constexpr int r = v0 + J, m = r / (2 * DB), db = r / 2 % DB, half = r % 2;
          vf[m][db][half] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((APBV_LDS(s16x4))(vt + (16 * m + 8 * half) * T::ROW_BYTES + v_off[db]));
        });
      } else {
        constexpr int m = (i - KS) / DB, db = (i - KS) % DB;
        const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(vf[m][db][0], vf[m][db][1], 0, 1, 2, 3, 4, 5, 6, 7));
        o[db] = mfma32(a, __builtin_bit_cast(bf16x8, pw[m]), o[db]);
        if constexpr (kPrefetchK) {
          constexpr int k0 = (KS * (i - KS)) / (2 * DB), k1 = (KS * (i - KS + 1)) / (2 * DB);
          static_for<k1 - k0>([&](auto J) { kf[k0 + J] = read_k(kt_after, k0 + J); });
        }
      }
      if constexpr (i < kExp) {
        constexpr int s0 = (16 * i) / kExp, s1 = (16 * (i + 1)) / kExp;
        static_for<s1 - s0>([&](auto J) {
          constexpr int sl = s0 + J, pi = sl / 2;
          if constexpr (sl % 2 == 0) {
            stage_f(pi);
            if constexpr (pi > 0) stage_c(pi - 1);
          } else {
            stage_e(pi);
            if constexpr (pi > 0) stage_d(pi - 1);
          }
        });
        if constexpr (i == kExp - 1) {
          stage_c(7);
          stage_d(7);
        }
      } else {
        constexpr int m0 = (8 * (i - kExp)) / DB, m1 = (8 * (i - kExp + 1)) / DB;
        static_for<m1 - m0>([&](auto J) {
          constexpr int m = m0 + J;
          if constexpr (m == 0)
            lm = __builtin_fmaxf(sn[0], sn[1]);
          else
            lm = __builtin_fmaxf(lm, __builtin_fmaxf(sn[2 * m], sn[2 * m + 1]));
        });
      }
      between(I, std::integral_constant<int, kMfma>{});
    });
  };

  TileStream<D, W, false, true> kst;
  TileStream<D, W, true, true> vst;
  kst.init(ks, p.s_kv, wave, lane, t_begin);
  vst.init(vs, p.s_kv, wave, lane, t_begin);
  const uint32_t k_ring = lds_addr(k_lds[0]), v_ring = lds_addr(v_lds[0]);
  // The Q fragments are in (vmcnt 0, known to the compiler): from here on only tile loads are outstanding.
  __builtin_amdgcn_s_waitcnt(0x0F70);
  auto arrive = [&]() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  auto nothing = [](auto, auto) {};
  // the loads of two K and two V tiles, spread over the matrix instructions of a tile
  auto load_tiles = [&](uint32_t k0, uint32_t k1, uint32_t v0, uint32_t v1) {
    return [&, k0, k1, v0, v1](auto I, auto N) {
      constexpr int n = 4 * T::IPW, from = n * decltype(I)::value / decltype(N)::value, to = n * (decltype(I)::value + 1) / decltype(N)::value;
      static_for<to - from>([&](auto J) {
        constexpr int j = from + J, which = j / T::IPW, u = j % T::IPW;
        if constexpr (which < 2)
          kst.issue_in_run(which == 0 ? k0 : k1, u, n_tiles - 1);
        else
          vst.issue_in_run(which == 2 ? v0 : v1, u, n_tiles - 1);
      });
    };
  };
  f32x16 s_a = zero, s_b = zero;
  if (t_begin < n_tiles) {
    kst.issue(k_ring);
    arrive();
    if (t_begin + 1 < n_tiles) kst.issue(k_ring + T::TILE_BYTES);
    if (t_begin + 2 < n_tiles) kst.issue(k_ring + 2 * T::TILE_BYTES);
    vst.issue(v_ring);
    if (t_begin + 1 < n_tiles) vst.issue(v_ring + T::TILE_BYTES);
    if (t_begin < n_w) {
      KFrags kf;
      load_k(k_lds[0], kf);
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) s_a = mfma32(kf[kk], qf[kk], s_a);
      if (t_begin >= t_mask) apply_mask(s_a, t_begin);
      advance_reference(lane_max(s_a));
    }
  }

  // ---- key loop (attention.hip): with r = t - t_begin, K(t) and V(t) live in slot r % 4, K one tile ahead of V in the
  // computation, one barrier per two tiles.
  int t = t_begin;
  const int t_pipe_end = n_w < t_mask ? n_w : t_mask;
  while (t < n_tiles) {
    int n_hot = 0;
    if (t + 4 < t_pipe_end && kst.t_next == t + 3 && vst.t_next == t + 2) {
      // whole rounds that start at t' with t' + 4 < t_pipe_end; their loads K(t'+3..t'+6), V(t'+2..t'+5) must lie in the
      // streams' current runs, or past the last tile, which is then loaded again (into slots nobody reads)
      n_hot = (t_pipe_end - 1 - t) / 4;
      const int by_k = kst.run_left() / 4, by_v = vst.run_left() / 4;
      if (kst.run_end < n_tiles) n_hot = n_hot < by_k ? n_hot : by_k;
      if (vst.run_end < n_tiles) n_hot = n_hot < by_v ? n_hot : by_v;
    }
    KFrags kf;
    float lm;
    for (int r = 0; r < n_hot; ++r, t += 4) {
      arrive();
      load_k(k_lds[1], kf);
      tile(std::true_type{}, kf, k_lds[2], v_lds[0], s_a, s_b, lm, load_tiles(k_ring + 3 * T::TILE_BYTES, k_ring, v_ring + 2 * T::TILE_BYTES, v_ring + 3 * T::TILE_BYTES));
      advance_reference(lm);
      tile(std::false_type{}, kf, nullptr, v_lds[1], s_b, s_a, lm, nothing);
      advance_reference(lm);
      arrive();
      load_k(k_lds[3], kf);
      tile(std::true_type{}, kf, k_lds[0], v_lds[2], s_a, s_b, lm, load_tiles(k_ring + T::TILE_BYTES, k_ring + 2 * T::TILE_BYTES, v_ring, v_ring + T::TILE_BYTES));
      advance_reference(lm);
      tile(std::false_type{}, kf, nullptr, v_lds[3], s_b, s_a, lm, nothing);
      advance_reference(lm);
    }
    if (t >= n_tiles) break;
    // one round of the general kind; past the wave's last tile S^T is formed from whatever the slot holds, and not used (ring
    // slots computed instead of written out were 4 % slower, 64 queries x 16 / 2 heads over 16512 keys 20.4 -> 21.3 us)
    auto step = [&](int tt, const unsigned char* kt_next, const unsigned char* vt, f32x16& sc, f32x16& sn) {
      if (tt >= n_w) return;
      load_k(kt_next, kf);
      tile(std::false_type{}, kf, nullptr, vt, sc, sn, lm, nothing);
      if (tt + 1 < n_w) {
        if (tt + 1 >= t_mask) {
          apply_mask(sn, tt + 1);
          lm = lane_max(sn);
        }
        advance_reference(lm);
      }
    };
    arrive();
    if (t + 3 < n_tiles) kst.issue(k_ring + 3 * T::TILE_BYTES);
    if (t + 4 < n_tiles) kst.issue(k_ring);
    if (t + 2 < n_tiles) vst.issue(v_ring + 2 * T::TILE_BYTES);
    if (t + 3 < n_tiles) vst.issue(v_ring + 3 * T::TILE_BYTES);
    step(t, k_lds[1], v_lds[0], s_a, s_b);
    step(t + 1, k_lds[2], v_lds[1], s_b, s_a);
    if (t + 2 >= n_tiles) break;
    arrive();
    if (t + 5 < n_tiles) kst.issue(k_ring + T::TILE_BYTES);
    if (t + 6 < n_tiles) kst.issue(k_ring + 2 * T::TILE_BYTES);
    if (t + 4 < n_tiles) vst.issue(v_ring);
    if (t + 5 < n_tiles) vst.issue(v_ring + T::TILE_BYTES);
    step(t + 2, k_lds[3], v_lds[2], s_a, s_b);
    step(t + 3, k_lds[0], v_lds[3], s_b, s_a);
    t += 4;
  }

  // ---- normalise, round, store.  A lane holds 4 of every 8 columns of its row; the halves exchange so that each stores 16
  // bytes of every other 8.
  auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
  const float l_tot = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;         // a key range may leave a row without any visible key
  const bool live = rw + c < n_rows;
  bf16_t* orow = p.out + (int64_t)split * p.split_stride_out + (((int64_t)b * p.L + qi) * p.hq + head) * D + 8 * hh;
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int q = 0; q < 4; q += 2) {
      u32x4 y;
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        auto word = [&](int g) {
          f32x2 xy = {o[db][4 * g + 2 * w] * inv, o[db][4 * g + 2 * w + 1] * inv};
          return __builtin_bit_cast(uint32_t, __builtin_convertvector(xy, bf16x2));
        };
        auto ex = __builtin_amdgcn_permlane32_swap(word(q), word(q + 1), false, false);
        y[w] = ex[0];
        y[2 + w] = ex[1];
      }
      if (live) *reinterpret_cast<u32x4*>(orow + 32 * db + 8 * q) = y;
    }
  if (p.lse != nullptr && hh == 0 && live)
    p.lse[(int64_t)split * p.split_stride_lse + ((int64_t)b * p.hq + head) * p.L + qi] =
        l_tot > 0.f ? (m_ref + __builtin_amdgcn_logf(l_tot)) * 0.6931471805599453f : -INFINITY;
}

// The row tiles of one (batch item, KV head, key range) read the same keys: they run back to back on one XCD.
template <int D, int W>
__global__ __launch_bounds__(64 * W, 8 / W) void packed_attention_kernel(const AttnParams p, const int n_rtiles, const int n_ranges) {
  const int slot = blockIdx.x / kXcds;
  const int range = (slot / n_rtiles) * kXcds + blockIdx.x % kXcds;      // (batch item, KV head, split)
  if (range >= n_ranges) return;
  const int split = range % p.n_splits, bh = range / p.n_splits;
  packed_workgroup<D, W>(p, slot % n_rtiles, bh / p.hkv, bh % p.hkv, split);
}

template <int W>
apbv_status launch_packed_variant(const AttnParams& p, int head_dim, hipStream_t stream) {
  const int64_t n_rtiles = (p.L * p.group + 32 * W - 1) / (32 * W);
  const int64_t n_ranges = (int64_t)p.batch * p.hkv * p.n_splits;
  const int64_t n_blocks = (n_ranges + kXcds - 1) / kXcds * kXcds * n_rtiles;
  if (n_blocks > 0x7fffffff) return APBV_ERR_UNSUPPORTED;
  Launcher launch(stream);
  if (head_dim == 128)
    launch(packed_attention_kernel<128, W>, dim3((unsigned)n_blocks), dim3(64 * W), 0, p, (int)n_rtiles, (int)n_ranges);
  else if (head_dim == 64)
    launch(packed_attention_kernel<64, W>, dim3((unsigned)n_blocks), dim3(64 * W), 0, p, (int)n_rtiles, (int)n_ranges);
  else
    return APBV_ERR_UNSUPPORTED;
  return launch.status();
}

}  // namespace

// The rows of a KV group's heads together, in workgroups of kQueryShortRows or kAttnQueryTile rows.
apbv_status launch_packed_attention(const AttnParams& p, int head_dim, int rows, hipStream_t stream) {
  static_assert(kQueryShortRows == 32 * 4 && kAttnQueryTile == 32 * 8, "the tile sizes the host-side planning assumes");
  return rows == kAttnQueryTile ? launch_packed_variant<8>(p, head_dim, stream) : launch_packed_variant<4>(p, head_dim, stream);
}

}  // namespace apbv
