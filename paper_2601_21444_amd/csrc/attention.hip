// Fused host attention for gfx950 (Eq. 4 by the definition of Eq. 1): one pass of online-softmax
// attention of the local query block over the concatenated keys [anchor | passing | local].
//
// Mask.  The three KV segments are walked as ONE virtual key axis j in [0, n_vis + L): anchor and
// passing keys (j < n_vis) are visible to every query and local key j - n_vis is visible to query i iff
// j - n_vis <= i, so the whole mask is the single test  j <= i + n_vis  (a causal mask shifted by
// n_vis).  Without a local segment (partial attention of a query block over context keys only, merged
// later by log-sum-exp) the bound is simply the last key.  Key tiles that lie entirely above that
// diagonal are never visited, and only tiles that touch it pay for the comparison.
//
// Tiling.  A workgroup of 8 waves (two per SIMD, one workgroup per CU) owns 256 consecutive query
// positions of one query head; each wave owns 32 of them.  Key tiles of 32 virtual keys are copied
// global -> LDS by the LDS-direct load (global_load_lds_dwordx4: no VGPR staging, no VALU work) into rings
// of four K and four V tiles, one barrier per two tiles.  Both are stored row-major [32][D] with an XOR
// swizzle of their 16-byte chunks; the swizzle is applied on the global side (which chunk a lane
// fetches), because an LDS-direct load always writes lane l's 16 bytes at base + 16*l.
//
// MFMA mapping (v_mfma_f32_16x16x32_bf16; with g = lane/16, i = lane%16: A is 16x32 with the lane
// holding row i, k-slots 8g..8g+7; B is 32x16 with the lane holding column i, the same k-slots; D is
// 16x16 with the lane holding column i, rows 4g..4g+3).  The 16x16x32 shape moves half the accumulator
// bytes per flop of the 32x32x16 one; on this power-limited part that is worth a higher clock.
//   S^T = K Q^T  : A = 16 key rows x 32 head-dim columns (one 16-byte LDS read per lane, used for both
//                  16-query blocks of the wave), B = Q^T kept in registers.  A lane then holds, for each of
//                  its two queries (i and 16 + i of the wave), keys 16*mb + 4g + r of the tile (mb = 0, 1).
//   O^T = V^T P^T: B = P^T straight from the S^T accumulator registers (rounded to bf16), no LDS round
//                  trip.  That fixes which key sits in which k-slot (slot 8g + e: key
//                  16 (e/4) + 4g + e%4); A = V^T is fetched to match with two transposing LDS
//                  reads (ds_read_b64_tr_b16: within 16 lanes, lane i receives element i%4 of the 8
//                  bytes addressed by lanes i/4, 4+i/4, 8+i/4, 12+i/4), each delivering 4 consecutive
//                  keys of one head-dim column.
//
// Softmax.  exp2 domain with the scale folded in.  The exponents of a row are taken against a reference that only moves when
// some logit of its 16-row block exceeds its row's by more than 2^5; then the references of the block become their rows'
// maxima, and O and the row sums are rescaled.  What is subtracted lies kReferenceBias above the reference, so that such a
// logit's probability is 2 or more, and nothing but the probabilities has to be looked at: bit 14 of a bf16 says so, and
// the words that hold a tile's are or-ed together (six instructions a tile; the maxima of the logits, which told it before,
// took fourteen).  If a bit is set, the block's probabilities are formed again from the logits, which are kept until then.  bf16
// and float32 have the exponents to spare: what underflows is 2^-121 of the row's maximum.  us, maxima of the logits / this:
// 28 heads of 128, three problems of up to 16384 rows 6064 / 5910, 16 heads x 16384 rows behind 9216 keys 1859 / 1807, 2 x 28
// heads x 3001 rows 181.1 / 179.4, 2 heads of 64, three problems of 16219 rows 255.5 / 247.3.  A probability equal to the
// reference is not rounded, so the sooner it moves the closer the results: relative errors against float64 of 300 rows of
// unit-variance logits with 2^2, 2^5, 2^8 1.86e-3, 2.03e-3, 2.11e-3 (2^8 for 32 rows at a time, as it was: 2.11e-3); every
// move costs, and times grow from 2^4 down (28 heads of 128 as above, both blocks of a wave moving together, at 2^2 / 2^3 / 2^4 / 2^5 / 2^8: 6142 / 6077 / 6039 / 6036 / 6014).
// Row sums are one more matrix instruction per query block and tile, with ones in place of V^T: it adds the probabilities
// P^T of all 32 keys to what every lane of the row holds.  Eight two-element dot products on the vector ALU did it before,
// of about 60 vector instructions a tile, and exchanges between the lane groups at the end.  us, dot products / this: 28
// heads of 128, three problems of up to 16384 rows 6243 / 6188, 2 x 28 heads x 3001 rows 185.1 / 182.3, 2 heads of 64, three
// problems of 16219 rows 270.5 / 258.6.
//
// Software pipeline.  The steps of a tile form a chain (S^T -> exp -> P^T -> O^T); done tile
// after tile a wave alternates between the matrix pipe and the vector ALU, and every LDS fragment read
// is waited for where it is issued.  Here, while the matrix pipe computes S^T of tile t+1, the vector
// ALU exponentiates tile t and the V^T operands of tile t are read; while it accumulates O^T of tile t,
// the K fragments of tile t+2 are read.  K therefore
// runs one tile ahead of V in LDS, and no LDS read is consumed in the phase that issues it.  Tiles that
// touch the mask diagonal, and the few rounds around a segment boundary, take the plain sequence.
//
// Key split.  For a short query block (few query tiles) the key axis can be cut into n_splits ranges of
// tiles_per_split tiles, one workgroup each; every range writes a normalised partial result and
// its log-sum-exp, merged afterwards (Eq. 5's merge).  n_splits = 1 is the plain kernel.
//
// Launch.  One workgroup per (query tile, query head, batch item), heaviest query tiles first.  The
// linear workgroup id is decoded so that the G query heads that share a KV head run on the same XCD
// (workgroup id modulo 8) back to back and stream the same K/V tiles through that XCD's L2.
#include "apbv_common.h"
#include "attention_tiles.h"

namespace apbv {
namespace {

constexpr int kWaves = 8;          // waves per workgroup of the main variant: 256 query rows
constexpr int kWavesNarrow = 2;    // of the variants for less work than fills the chip with 256-row workgroups: 64
constexpr int kWavesShort = 4;     // and 128 query rows
constexpr int kBM = 32 * kWaves;   // query rows per workgroup (main variant)
constexpr float kNoReference = -3.402823466e38f;      // what is subtracted in a row that has seen no visible key: below every logit
constexpr int kRing = 4;           // K tiles, and V tiles, resident in LDS

// One workgroup's work: row tile `qt` of batch item b and query head (kvh, g), key range `split`.
// kOwn: 16-row blocks per wave.  Two share every K and V fragment that is read; one is for launches that leave SIMDs empty: a
// wave alone on its SIMD does not overlap its matrix and vector instructions (16 + 4.2 n cycles for one 16x16x32 and n vector
// instructions, measured), so its time is their sum, half of what it is with two.  Results are the same bit for bit.  Four
// waves of one block, against two waves of two blocks / two waves that finish 16 rows each but form S^T of all 32 (as the
// reference was one for a block before) / now (us): 16 heads of 128 x 1024 rows behind 224 keys 29.3 / 22.2 / 18.2, 2 heads
// of 64 x 512 rows behind 160 12.8 / 10.9 / 9.0.
template <int D, int W, int kOwn>
__device__ __forceinline__ void attention_workgroup(const AttnParams& p, const int qt, const int b, const int kvh,
                                                    const int g, const int split) {
  using T = Tile<D, W>;
  constexpr int kRows = 16 * kOwn * W;        // query rows of the workgroup
  __shared__ __attribute__((aligned(1024))) unsigned char k_lds[kRing][T::TILE_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char v_lds[kRing][T::TILE_BYTES];
  // the LDS destination of an LDS-direct load travels in M0, which addresses the first 64 KB of the workgroup's LDS
  static_assert(2 * kRing * T::TILE_BYTES <= 65536, "the K/V tile rings must lie below 64 KB of LDS");
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: keeps LDS tile addresses in SGPRs
  const int li = lane & 15;       // query column / A-operand row within a 16-block
  const int lg = lane >> 4;       // lane group: k-slots 8 lg .. 8 lg + 7, accumulator rows 4 lg .. 4 lg + 3

  const int h = kvh * p.group + g;
  const int64_t i0 = (int64_t)qt * kRows;               // first row of the workgroup
  const int64_t iw = i0 + wave * 16 * kOwn;             // first row of the wave

  Segs ks, vs;
  key_segments(p, b, kvh, ks, vs);

  // ---- Q^T fragments (B operand of S^T), kept in registers for the whole key loop.
  bf16x8 qf[T::KSD][kOwn];
#pragma unroll
  for (int nq = 0; nq < kOwn; ++nq) {
    const int64_t i = iw + 16 * nq + li, r = i < p.L ? i : p.L - 1;
    const bf16_t* qrow = p.q.ptr + (int64_t)b * p.q.sb + (int64_t)h * p.q.sh + r * p.q.st;
#pragma unroll
    for (int c = 0; c < T::KSD; ++c) qf[c][nq] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(qrow + 32 * c + 8 * lg));
  }

  // ---- per-lane LDS read offsets
  // K (A operand of S^T): row 16*mb + li, 16-byte chunk (4*c + lg) ^ fk(row); fk does not depend on mb
  int k_off[T::KSD];
#pragma unroll
  for (int c = 0; c < T::KSD; ++c) k_off[c] = li * T::ROW_BYTES + (((4 * c + lg) ^ T::fk(li)) << 4);
  // V (A operand of O^T, transposing read): within a 16-lane group, source lane s addresses key row 4*lg + s/4
  // (+ 16 for the second half of the k-slots, as an immediate; fv does not depend on it), head-dim columns
  // 16*d + 4*(s%4) .. +3
  int v_off[T::DBN];
  {
    const int row = 4 * lg + (li >> 2);
#pragma unroll
    for (int d = 0; d < T::DBN; ++d) {
      const int chunk = 2 * d + ((li & 3) >> 1);
      v_off[d] = row * T::ROW_BYTES + ((chunk ^ T::fv(row)) << 4) + (li & 1) * 8;
    }
  }

  // ---- online softmax state.  Per lane: kOwn queries; the four lane groups hold different head-dim rows of O, and the same sums.
  f32x4 o[T::DBN][kOwn];
#pragma unroll
  for (int d = 0; d < T::DBN; ++d)
#pragma unroll
    for (int nq = 0; nq < kOwn; ++nq) o[d][nq] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_sub[kOwn];                         // what the exponent subtracts: the row's reference + kReferenceBias
  f32x4 l_run[kOwn];                         // [0]: running sum of the bf16-rounded probabilities of the row (the other three are not used)
#pragma unroll
  for (int nq = 0; nq < kOwn; ++nq) {
    m_sub[nq] = kNoReference;
    l_run[nq] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});

  // Keys the workgroup / this wave can see at all.
  // Query i sees the virtual keys 0 .. min(i + n_vis, s_kv - 1); the second bound only matters when there is no
  // causal segment (s_kv == n_vis: every key visible to every query).
  auto last_key = [&](int64_t i) { return (i + p.n_vis < p.s_kv - 1) ? i + p.n_vis : p.s_kv - 1; };
  const int64_t i_last_wg = (i0 + kRows - 1 < p.L - 1) ? i0 + kRows - 1 : p.L - 1;
  const int n_tiles_vis = (int)(last_key(i_last_wg) / kBN) + 1;      // tiles the workgroup can see into
  // key split (partial results merged afterwards): this workgroup walks tiles [t_begin, n_tiles) only; the split is
  // planned in 64-key units
  const int64_t per_split = (int64_t)p.tiles_per_split * (64 / kBN);
  const int64_t t_begin64 = (int64_t)split * per_split;
  const int t_begin = (int)(t_begin64 < n_tiles_vis ? t_begin64 : n_tiles_vis);
  const int n_tiles = (int)(t_begin64 + per_split < n_tiles_vis ? t_begin64 + per_split : n_tiles_vis);
  const int t_last_wave = (int)(last_key(iw + 16 * kOwn - 1) / kBN);     // last tile any row of the wave can see into
  const int n_w = t_last_wave + 1 < n_tiles ? t_last_wave + 1 : n_tiles;     // the wave computes tiles [t_begin, n_w)
  const int t_mask_wave = (int)((last_key(iw) + 1) / kBN);    // first tile with a key some row of the wave cannot see
  int jrel0[kOwn];                                            // last visible virtual key of each row
#pragma unroll
  for (int nq = 0; nq < kOwn; ++nq) jrel0[nq] = (int)last_key(iw + 16 * nq + li);

  typedef f32x4 STile[2][kOwn];      // S^T of one tile: [16-key block][16-query block]
  typedef u32x4 PTile[kOwn];         // P^T of one tile as the B operand of O^T: [16-query block], four 32-bit words

  auto read_k = [&](const unsigned char* kt, int mb, int c) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(kt + mb * 16 * T::ROW_BYTES + k_off[c]));
  };
  auto read_vt = [&](const unsigned char* vt, int d) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((APBV_LDS(s16x4))(vt + v_off[d]));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((APBV_LDS(s16x4))(vt + 16 * T::ROW_BYTES + v_off[d]));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  // ---- S^T = K Q^T of one tile
  auto qk = [&](const unsigned char* kt, STile& s) {
#pragma unroll
    for (int c = 0; c < T::KSD; ++c)
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) {
        const bf16x8 a = read_k(kt, mb, c);
#pragma unroll
        for (int nq = 0; nq < kOwn; ++nq)
          s[mb][nq] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[c][nq], c == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[mb][nq], 0, 0, 0);
      }
  };

  // ---- mask of a tile that reaches above the wave's first diagonal element
  auto apply_mask = [&](STile& s, int t) {
#pragma unroll
    for (int nq = 0; nq < kOwn; ++nq) {
      const int jrel_max = jrel0[nq] - t * kBN;          // last visible key of this query, tile-relative
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (16 * mb + 4 * lg + r > jrel_max) s[mb][nq][r] = -INFINITY;
    }
  };

  // ---- probabilities of the tile for query block nq: exp2 of the scaled logits minus the reference, rounded to bf16
  // (the PV operand).
  auto exp_block = [&](const STile& s, int nq, PTile& pw) {
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        f32x2 xy = {__builtin_amdgcn_exp2f(__builtin_fmaf(s[mb][nq][e], p.scale_log2, -m_sub[nq])),
                    __builtin_amdgcn_exp2f(__builtin_fmaf(s[mb][nq][e + 1], p.scale_log2, -m_sub[nq]))};
        pw[nq][2 * mb + (e >> 1)] = __builtin_bit_cast(uint32_t, __builtin_convertvector(xy, bf16x2));
      }
  };

  // ---- lazy rescaling: where a probability of a 16-row block is 2 or more, the references of the block's rows become their
  // largest logits of the tile, where these are larger, and the probabilities are formed again.  (A row that has not seen a
  // visible key has kNoReference: hidden keys give exp2(-inf) = 0, the first visible one +inf.)
  auto asks = [&](const u32x4& pw) {       // lanes with such a probability
    return __builtin_amdgcn_ballot_w64(((pw[0] | pw[1] | pw[2] | pw[3]) & 0x40004000u) != 0);
  };
  auto tile_reference = [&](const STile& s, int nq) {      // the row's largest logit of the tile + kReferenceBias
    float mx = s[0][nq][0];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int r = (mb == 0 ? 1 : 0); r < 4; ++r) mx = __builtin_fmaxf(mx, s[mb][nq][r]);
    {
      auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    }
    {
      auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    }
    return __builtin_fmaf(mx, p.scale_log2, kReferenceBias);
  };
  auto move_reference = [&](const STile& s, int nq, PTile& pw) {
    const float m_new = fmaxf(m_sub[nq], tile_reference(s, nq));
    const float alpha = __builtin_amdgcn_exp2f(m_sub[nq] - m_new);
    m_sub[nq] = m_new;
    l_run[nq][0] *= alpha;
#pragma unroll
    for (int d = 0; d < T::DBN; ++d) o[d][nq] *= alpha;
    exp_block(s, nq, pw);
  };
  // Only the blocks that ask take these steps, behind a branch each.  In the hot loop these lie inside one for both, which is 1 %
  // faster at 256 rows; the plain sequence, which is there several times, would take 20 to 52 bytes of scratch so.
  // Both blocks stepping together, branch-free, and the first tile behind the branch too, as it was, against this (us; queries of
  // 12 times unit variance, and of unit variance): 2 x 28 heads x 3001 rows 208.5 / 197.0, 175.8 / 174.8; 16 heads x 8192 rows behind
  // 2560 keys 409.3 / 388.7, 357.9 / 357.9; 28 x 8192 behind 4096 908.0 / 871.1, 801.1 / 801.3; 8 heads of 64 x 8192 behind 1000
  // 122.1 / 115.0, 104.3 / 104.2; of one tile, 23 blocks of a row x 28 heads of 128 10.6 / 10.0.
  auto settle_reference = [&](auto hot, const STile& s, PTile& pw) {
    if constexpr (decltype(hot)::value) {
      uint64_t moves[kOwn], some = 0;
#pragma unroll
      for (int nq = 0; nq < kOwn; ++nq) some |= moves[nq] = asks(pw[nq]);
      if (__builtin_expect(some == 0, 1)) return;
#pragma unroll
      for (int nq = 0; nq < kOwn; ++nq)
        if (moves[nq] != 0) move_reference(s, nq, pw);
    } else {
#pragma unroll
      for (int nq = 0; nq < kOwn; ++nq)
        if (__builtin_expect(asks(pw[nq]) != 0, 0)) move_reference(s, nq, pw);
    }
  };

  // ---- row sums += 1 P^T
  auto add_sums = [&](int nq, const u32x4& pw) {
    l_run[nq] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, __builtin_bit_cast(bf16x8, pw), l_run[nq], 0, 0, 0);
  };

  // ---- O^T += V^T P^T for the 32 keys of the tile
  auto pv = [&](const unsigned char* vt, const PTile& pw) {
#pragma unroll
    for (int nq = 0; nq < kOwn; ++nq) add_sums(nq, pw[nq]);
#pragma unroll
    for (int d = 0; d < T::DBN; ++d) {
      const bf16x8 a = read_vt(vt, d);
#pragma unroll
      for (int nq = 0; nq < kOwn; ++nq)
        o[d][nq] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, pw[nq]), o[d][nq], 0, 0, 0);
    }
  };

  // ---- plain sequence, for the first tile and for tiles on the mask diagonal
  auto prepare = [&](const unsigned char* kt, int t, STile& s) {       // S^T, mask
    qk(kt, s);
    if (t >= t_mask_wave) apply_mask(s, t);
  };
  auto finish = [&](const unsigned char* vt, const STile& s) {          // probabilities, reference, O^T
    PTile pw;
#pragma unroll
    for (int nq = 0; nq < kOwn; ++nq) exp_block(s, nq, pw);
    settle_reference(std::false_type{}, s, pw);
    pv(vt, pw);
  };

  // ---- pipelined body: finishes tile t (S^T in sc, V tile at vt) while it prepares tile t+1 (K fragments already
  // in kf, S^T into sn).  No LDS read is waited for where it is issued: the K fragments of a tile are read one phase
  // ahead, the V^T operands of phase B during phase A.
  //   phase A: S^T(t+1) on the matrix pipe from kf; the exponentials of tile t on the vector ALU; the V^T operands of
  //            tile t read into vf; then the reference, should a probability ask for it
  //   phase B: O^T(t) from vf; with kPrefetchK the K fragments of tile t+2 (at kt_after, landed since the
  //            last barrier) read into kf
  typedef bf16x8 KFrags[2 * T::KSD];        // [c][mb]
  auto load_k = [&](const unsigned char* kt, KFrags& kf) {
#pragma unroll
    for (int c = 0; c < T::KSD; ++c)
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) kf[2 * c + mb] = read_k(kt, mb, c);
  };
  auto pipelined = [&](auto prefetch_k, KFrags& kf, const unsigned char* kt_after, const unsigned char* vt,
                       const STile& sc, STile& sn) {
    constexpr bool kPrefetchK = decltype(prefetch_k)::value;
    // The source lists each matrix instruction with its share of the vector and LDS instructions; the compiler's own
    // scheduler keeps that interleaving (pinning it with scheduling fences was measured 3 % slower).
    // exponential pipeline of tile t, one pair of probabilities at a time: pair pi = (nq, mb, first/second two rows);
    // stages F (scale and subtract), E (exp2), C (round to bf16 into the B operand word)
    constexpr int kPairs = 4 * kOwn;
    float xf[kPairs][2];
    PTile pw;
    auto stage_f = [&](int pi) {
      const int nq = pi >> 2, mb = (pi >> 1) & 1, e = 2 * (pi & 1);
      xf[pi][0] = __builtin_fmaf(sc[mb][nq][e], p.scale_log2, -m_sub[nq]);
      xf[pi][1] = __builtin_fmaf(sc[mb][nq][e + 1], p.scale_log2, -m_sub[nq]);
    };
    auto stage_e = [&](int pi) {
      xf[pi][0] = __builtin_amdgcn_exp2f(xf[pi][0]);
      xf[pi][1] = __builtin_amdgcn_exp2f(xf[pi][1]);
    };
    auto stage_c = [&](int pi) {
      const int nq = pi >> 2, mb = (pi >> 1) & 1;
      f32x2 xy = {xf[pi][0], xf[pi][1]};
      pw[nq][2 * mb + (pi & 1)] = __builtin_bit_cast(uint32_t, __builtin_convertvector(xy, bf16x2));
    };
    // ---- phase A: one slice per matrix instruction of S^T(t+1)
    s16x4 vlo[T::DBN], vhi[T::DBN];
    constexpr int nA = 2 * kOwn * T::KSD;          // matrix instructions of phase A
    static_for<nA>([&](auto I) {
      constexpr int i = I;
      constexpr int c = i / (2 * kOwn), nq = (i / 2) % kOwn, mb = i % 2;
      sn[mb][nq] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[2 * c + mb], qf[c][nq],
                                                           c == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sn[mb][nq], 0, 0, 0);
      // the slices of the exponential pipeline are spread evenly over the nA matrix instructions
      constexpr int s0 = (2 * kPairs * i) / nA, s1 = (2 * kPairs * (i + 1)) / nA;
      static_for<s1 - s0>([&](auto J) {
        constexpr int sl = s0 + J, pi = sl / 2;
        if constexpr (sl % 2 == 0) {
          stage_f(pi);
          if constexpr (pi > 0) stage_c(pi - 1);
        } else {
          stage_e(pi);
        }
      });
      // ... and the 2 DBN transposing reads of the V^T operands of phase B
      constexpr int r0 = (2 * T::DBN * i) / nA, r1 = (2 * T::DBN * (i + 1)) / nA;
      static_for<r1 - r0>([&](auto J) {
        constexpr int r = r0 + J, d = r / 2;
        if constexpr (r % 2 == 0)
          vlo[d] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((APBV_LDS(s16x4))(vt + v_off[d]));
        else
          vhi[d] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((APBV_LDS(s16x4))(vt + 16 * T::ROW_BYTES + v_off[d]));
      });
    });
    stage_c(kPairs - 1);
    settle_reference(std::true_type{}, sc, pw);
    // ---- phase B: one slice per matrix instruction of O^T(t)
    constexpr int nB = kOwn * T::DBN, nK = kPrefetchK ? 2 * T::KSD : 0;
    static_for<nB>([&](auto I) {
      constexpr int i = I;
      constexpr int d = i / kOwn, nq = i % kOwn;
      if constexpr (d == 0) add_sums(nq, pw[nq]);
      const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(vlo[d], vhi[d], 0, 1, 2, 3, 4, 5, 6, 7));
      o[d][nq] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, pw[nq]), o[d][nq], 0, 0, 0);
      // the K fragments of tile t+2
      constexpr int k0 = (nK * i) / nB, k1 = (nK * (i + 1)) / nB;
      static_for<k1 - k0>([&](auto J) {
        constexpr int k = k0 + J;
        kf[k] = read_k(kt_after, k % 2, k / 2);
      });
    });
  };

  // One tile step of the wave in the plain sequence: K(t+1) is at kt_next, V(t) at vt, S^T(t) in sc; leaves S^T(t+1)
  // in sn.
  auto step = [&](int t, const unsigned char* kt_next, const unsigned char* vt, STile& sc, STile& sn) {
    if (t >= n_w) return;
    finish(vt, sc);
    if (t + 1 < n_w) prepare(kt_next, t + 1, sn);
  };

  // ---- key loop.  With r = t - t_begin, K(t) and V(t) live in slot r % 4 of their rings, and K runs one tile ahead
  // of V in the computation.  One barrier per two tiles: after the barrier in front of tiles t, t+1 the tiles K(t+1),
  // K(t+2), V(t), V(t+1) have landed, everyone is done with K(t-1), K(t), V(t-2), V(t-1), and the loads of K(t+3),
  // K(t+4), V(t+2), V(t+3) go into those slots.
  TileStream<D, W, false> kst;
  TileStream<D, W, true> vst;
  kst.init(ks, p.s_kv, wave, lane, t_begin);
  vst.init(vs, p.s_kv, wave, lane, t_begin);
  uint32_t ka[kRing], va[kRing];
#pragma unroll
  for (int i = 0; i < kRing; ++i) {
    ka[i] = lds_addr(k_lds[i]);
    va[i] = lds_addr(v_lds[i]);
  }
  // The Q fragments are in (vmcnt 0, other counters untouched): from here on only tile loads are
  // outstanding, and the compiler knows it need not wait for vector memory inside the loop.
  __builtin_amdgcn_s_waitcnt(0x0F70);
  STile s_a, s_b;
  if (t_begin < n_tiles) {
    kst.issue(ka[0]);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (t_begin + 1 < n_tiles) kst.issue(ka[1]);
    if (t_begin + 2 < n_tiles) kst.issue(ka[2]);
    vst.issue(va[0]);
    if (t_begin + 1 < n_tiles) vst.issue(va[1]);
    if (t_begin < n_w) {
      prepare(k_lds[0], t_begin, s_a);
#pragma unroll
      for (int nq = 0; nq < kOwn; ++nq) m_sub[nq] = fmaxf(m_sub[nq], tile_reference(s_a, nq));   // every row's first move: nothing to rescale
    }
  }
  // loads of the two barrier intervals of a four-tile round that starts at tile t
  auto issue_first = [&](int t) {
    if (t + 3 < n_tiles) kst.issue(ka[3]);
    if (t + 4 < n_tiles) kst.issue(ka[0]);
    if (t + 2 < n_tiles) vst.issue(va[2]);
    if (t + 3 < n_tiles) vst.issue(va[3]);
  };
  auto issue_second = [&](int t) {
    if (t + 5 < n_tiles) kst.issue(ka[1]);
    if (t + 6 < n_tiles) kst.issue(ka[2]);
    if (t + 4 < n_tiles) vst.issue(va[0]);
    if (t + 5 < n_tiles) vst.issue(va[1]);
  };
  auto arrive = [&]() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's share of the tiles needed next has landed
    __syncthreads();                                  // ... everyone's has, and everyone is done with the slots reloaded now
  };
  int t = t_begin;
  const int t_pipe_end = n_w < t_mask_wave ? n_w : t_mask_wave;
  while (t < n_tiles) {
    // Rounds in which all four tiles and their successors are fully visible to the wave and every tile to be
    // loaded lies inside the streams' current runs: the pipelined body and unconditional loads, no tests.  (A round
    // loads K(t+3..t+6) and V(t+2..t+5).  Waves leave this loop at different rounds; every round of either kind
    // passes the same two barriers.)
    int n_hot = 0;
    if (t + 4 < t_pipe_end && t + 6 < n_tiles && kst.t_next == t + 3 && vst.t_next == t + 2) {
      const int by_mask = (t_pipe_end - 4 - t + 3) / 4;      // rounds that start at t' with t' + 4 < t_pipe_end
      const int by_end = (n_tiles - 6 - t + 3) / 4;          // ... and load existing tiles only: t' + 6 < n_tiles
      const int by_k = kst.run_left() / 4, by_v = vst.run_left() / 4;
      n_hot = by_mask < by_end ? by_mask : by_end;
      n_hot = n_hot < by_k ? n_hot : by_k;
      n_hot = n_hot < by_v ? n_hot : by_v;
    }
    KFrags kf;
    for (int r = 0; r < n_hot; ++r, t += 4) {
      arrive();
      load_k(k_lds[1], kf);
      kst.issue_in_run(ka[3]);
      kst.issue_in_run(ka[0]);
      vst.issue_in_run(va[2]);
      vst.issue_in_run(va[3]);
      pipelined(std::true_type{}, kf, k_lds[2], v_lds[0], s_a, s_b);
      pipelined(std::false_type{}, kf, nullptr, v_lds[1], s_b, s_a);
      arrive();
      load_k(k_lds[3], kf);
      kst.issue_in_run(ka[1]);
      kst.issue_in_run(ka[2]);
      vst.issue_in_run(va[0]);
      vst.issue_in_run(va[1]);
      pipelined(std::true_type{}, kf, k_lds[0], v_lds[2], s_a, s_b);
      pipelined(std::false_type{}, kf, nullptr, v_lds[3], s_b, s_a);
    }
    if (t >= n_tiles) break;
    // One round of the general kind: tiles on the mask diagonal, the wave's last tiles, rounds the wave only sits
    // through, loads that cross a segment boundary or stop at the last tile.
    arrive();
    issue_first(t);
    step(t, k_lds[1], v_lds[0], s_a, s_b);
    step(t + 1, k_lds[2], v_lds[1], s_b, s_a);
    if (t + 2 >= n_tiles) break;
    arrive();
    issue_second(t);
    step(t + 2, k_lds[3], v_lds[2], s_a, s_b);
    step(t + 3, k_lds[0], v_lds[3], s_b, s_a);
    t += 4;
  }

  // ---- epilogue: normalise, round to bf16, store; optional log-sum-exp.  (The lane's place is asked for anew, so that no
  // register holds it through the key loop.)
  const int lane_out = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), lg_out = lane_out >> 4;
#pragma unroll
  for (int nq = 0; nq < kOwn; ++nq) {
    const float l_tot = l_run[nq][0];
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;     // a key split may leave a row without any visible key
    const int64_t i = iw + 16 * nq + (lane_out & 15);
    if (i < p.L) {
      bf16_t* orow = p.out + (int64_t)split * p.split_stride_out + (((int64_t)b * p.L + i) * p.hq + h) * D;
#pragma unroll
      for (int d = 0; d < T::DBN; ++d) {
        f32x2 x01 = {o[d][nq][0] * inv, o[d][nq][1] * inv};
        f32x2 x23 = {o[d][nq][2] * inv, o[d][nq][3] * inv};
        bf16x2 c01 = __builtin_convertvector(x01, bf16x2);
        bf16x2 c23 = __builtin_convertvector(x23, bf16x2);
        u32x2 w;
        w.x = __builtin_bit_cast(uint32_t, c01);
        w.y = __builtin_bit_cast(uint32_t, c23);
        *reinterpret_cast<u32x2*>(orow + 16 * d + 4 * lg_out) = w;
      }
      if (p.lse != nullptr && lg_out == 0)
        p.lse[(int64_t)split * p.split_stride_lse + ((int64_t)b * p.hq + h) * p.L + i] =
            l_tot > 0.f ? (m_sub[nq] + __builtin_amdgcn_logf(l_tot)) * 0.6931471805599453f : -INFINITY;
    }
  }
}

// Work items are numbered heaviest first, `period` consecutive ones (the KV heads, batch items and key ranges of one
// query tile) being equally heavy, and are dealt to the XCDs eight at a time.  Dealt always in the same direction,
// XCD 0 would get the heaviest item of every row of eight and XCD 7 the lightest -- 4 to 12 % more work for the one
// than for the other with a causal block.  Odd rows are therefore dealt in the opposite direction, in whole groups of
// `period` XCDs where that divides eight, so that an XCD keeps serving the same KV head (its L2 holds that head's
// K/V), item by item otherwise.
__device__ __forceinline__ int deal(int row, int xcd, int period) {
  if (row & 1) {
    const int s = (period < kXcds && kXcds % period == 0) ? period : (period % kXcds == 0 ? kXcds : 1);
    xcd = (kXcds / s - 1 - xcd / s) * s + xcd % s;
  }
  return row * kXcds + xcd;
}

// The place of this workgroup's item among its XCD's (rows of `group` workgroups, one item each), -1 without one: of the last
// row some XCDs have no item, and arrange those they have.
template <int D, int W, int kOwn>
__device__ __forceinline__ int arranged_slot(int slot, int group, int period, int n_items, int arrangements) {
  const int n_all = gridDim.x / kXcds;
  const bool all = deal(n_all / group - 1, blockIdx.x % kXcds, period) < n_items;
  const int n = all ? n_all : n_all - group;
  return slot < n ? arrange_workgroup(slot, n, workgroups_per_unit(D, W, kOwn), all ? arrangements % 4 : arrangements / 4) : -1;
}

// ---- workgroup -> (query tile, head, batch, key range); the heads of one KV group share an XCD
template <int D, int W, int kOwn = 2>
__global__ __launch_bounds__(64 * W, 2) void host_attention_kernel(const AttnParams p, const int n_qtiles,
                                                                   const int n_items, const int arrangements) {
  const int xcd = blockIdx.x % kXcds;
  int slot = blockIdx.x / kXcds;
  if (W != kWavesNarrow && arrangements != 0) {
    slot = arranged_slot<D, W, kOwn>(slot, p.group, p.batch * p.hkv * p.n_splits, n_items, arrangements);
    if (slot < 0) return;
  }
  const int item_split = deal(slot / p.group, xcd, p.batch * p.hkv * p.n_splits);
  if (item_split >= n_items) return;
  const int split = item_split % p.n_splits;     // key ranges of one item share nothing: spread them over the XCDs
  const int item = item_split / p.n_splits;
  const int g = slot % p.group;
  const int bh = p.batch * p.hkv;
  const int qt = n_qtiles - 1 - item / bh;       // heaviest query tiles first
  const int b = (item % bh) / p.hkv;
  const int kvh = (item % bh) % p.hkv;
  attention_workgroup<D, W, kOwn>(p, qt, b, kvh, g, split);
}

// ---- several attention problems of different lengths in one launch (the two virtual hosts and the anchor
// block of a physical host, Alg. 1 / Sec. 4.3): one workgroup per entry of the merged heaviest-first order of
// all (problem, query tile) pairs, per KV head and group member.
template <int D, int W, int kOwn = 2>
__global__ __launch_bounds__(64 * W, 2) void host_attention_group_kernel(const AttnGroupParams gp) {
  const int group = gp.item[0].group, hkv = gp.item[0].hkv;
  const int xcd = blockIdx.x % kXcds;
  int slot = blockIdx.x / kXcds;
  if (gp.arrangements != 0) {
    slot = arranged_slot<D, W, kOwn>(slot, group, hkv, gp.sched.n_entries * hkv, gp.arrangements);
    if (slot < 0) return;
  }
  const int unit = deal(slot / group, xcd, hkv);
  if (unit >= gp.sched.n_entries * hkv) return;
  const int g = slot % group;
  const int entry = unit / hkv, kvh = unit % hkv;
  int m, qt;
  decode_group_entry(gp.sched, entry, m, qt);
  if (m >= gp.n_items || qt < 0 || (int64_t)qt * (16 * kOwn * W) >= gp.item[m].L) return;      // never taken for a schedule the launcher built
  // (a copy, so that the fields live in scalar registers like the single-problem kernel's by-value argument
  // instead of being fetched from the argument block where they are used)
  const AttnParams item = gp.item[m];
  attention_workgroup<D, W, kOwn>(item, qt, 0, kvh, g, 0);
}

}  // namespace

template <int W, int kOwn = 2>
static apbv_status launch_variant(const AttnParams& p, int head_dim, hipStream_t stream) {
  constexpr int kRows = 16 * kOwn * W;
  const int n_qtiles = (int)((p.L + kRows - 1) / kRows);
  const int64_t n_items = (int64_t)n_qtiles * p.batch * p.hkv * p.n_splits;
  const int64_t n_blocks = (n_items + kXcds - 1) / kXcds * kXcds * p.group;
  if (n_blocks > 0x7fffffff) return APBV_ERR_UNSUPPORTED;
  // (blocks of two waves have one or two query tiles, which weigh about the same)
  const int arrangements = W == kWavesNarrow ? 0 : tile_arrangements(workgroups_per_unit(head_dim, W, kOwn), p.group, (int64_t)p.batch * p.hkv * p.n_splits,
                                                                       kRows, p.L, p.n_vis, p.s_kv > p.n_vis);
  dim3 grid((unsigned)n_blocks);
  dim3 block(64 * W);
  Launcher launch(stream);
  if (head_dim == 64) {
    launch(host_attention_kernel<64, W, kOwn>, grid, block, 0, p, n_qtiles, (int)n_items, arrangements);
    return launch.status();
  }
  if constexpr (W != kWavesNarrow)
    if (head_dim == 128) {
      launch(host_attention_kernel<128, W, kOwn>, grid, block, 0, p, n_qtiles, (int)n_items, arrangements);
      return launch.status();
    }
  return APBV_ERR_UNSUPPORTED;
}

// Blocks of at most kAttnNarrowMaxRows rows in more workgroups than leave SIMDs empty (kNarrow64): two waves of two blocks each,
// which read K and V half as often as four of one, with head_dim 64; four with 128, where a wave of two blocks has a SIMD to
// itself either way (64 KB of LDS a workgroup) and moves its O between vector and accumulation registers from round to round.
// 150 launches (1 to 128 rows, up to 8000 workgroups), time of two waves over that of four: head_dim 128 1.24 on average, least
// 1.01 (28 heads x 132 blocks of 64 rows 52.6 / 41.5 us); 64 1.09, but 0.83 where there are few keys (32 heads x 27 blocks of 21
// rows 5.9 / 7.2).
apbv_status launch_host_attention(const AttnParams& p, int head_dim, hipStream_t stream) {
  static_assert(kAttnQueryTile == kBM && kAttnNarrowQueryTile == 32 * kWavesNarrow, "tile sizes the host-side planning assumes");
  switch (attention_kernel(head_dim, p.group, p.batch, p.hq, p.L, p.n_vis, p.s_kv > p.n_vis, p.n_splits)) {
    case AttentionKernel::kShared64: return launch_variant<kWavesShort, 1>(p, head_dim, stream);
    case AttentionKernel::kNarrow64: return head_dim == 64 ? launch_variant<kWavesNarrow>(p, head_dim, stream) : launch_variant<kWavesShort, 1>(p, head_dim, stream);
    case AttentionKernel::k128: return launch_variant<kWavesShort>(p, head_dim, stream);
    case AttentionKernel::k256: break;
  }
  return launch_variant<kWaves>(p, head_dim, stream);
}

template <int W, int kOwn = 2>
static apbv_status launch_group_variant(AttnGroupParams& gp, int head_dim, const int64_t* n_vis, const int64_t* rows, hipStream_t stream) {
  static_assert(sizeof(AttnGroupParams) <= 4096, "kernel arguments are limited to 4 KB");
  if (!build_group_schedule(gp.n_items, n_vis, rows, gp.sched, 16 * kOwn * W)) return APBV_ERR_UNSUPPORTED;
  const AttnParams& p0 = gp.item[0];
  const int64_t n_units = (int64_t)gp.sched.n_entries * p0.hkv;
  const int64_t n_blocks = (n_units + kXcds - 1) / kXcds * kXcds * p0.group;
  if (n_blocks > 0x7fffffff) return APBV_ERR_UNSUPPORTED;
  gp.arrangements = schedule_arrangements(workgroups_per_unit(head_dim, W, kOwn), p0.group, p0.hkv, 16 * kOwn * W, gp.sched, n_vis);
  Launcher launch(stream);
  if (head_dim == 128)
    launch(host_attention_group_kernel<128, W, kOwn>, dim3((unsigned)n_blocks), dim3(64 * W), 0, gp);
  else if (head_dim == 64)
    launch(host_attention_group_kernel<64, W, kOwn>, dim3((unsigned)n_blocks), dim3(64 * W), 0, gp);
  else
    return APBV_ERR_UNSUPPORTED;
  return launch.status();
}

apbv_status launch_host_attention_group(AttnGroupParams& gp, int head_dim, hipStream_t stream) {
  static_assert(kGroupQueryTile == kBM, "the schedule's query tile is the kernel's");
  const int n = gp.n_items;
  if (n < 1 || n > kMaxGroupItems) return APBV_ERR_UNSUPPORTED;
  int64_t n_vis[kMaxGroupItems], rows[kMaxGroupItems];
  for (int m = 0; m < n; ++m) {
    n_vis[m] = gp.item[m].n_vis;
    rows[m] = gp.item[m].L;
  }
  switch (attention_group_kernel(head_dim, gp.item[0].hq, gp.item[0].hkv, n, n_vis, rows)) {
    case AttentionKernel::kShared64: return launch_group_variant<kWavesShort, 1>(gp, head_dim, n_vis, rows, stream);
    case AttentionKernel::k256: return launch_group_variant<kWaves>(gp, head_dim, n_vis, rows, stream);
    default: return launch_group_variant<kWavesShort>(gp, head_dim, n_vis, rows, stream);
  }
}

}  // namespace apbv
