// Merge of partial attention results by their log-sum-exp (Eq. 5: A_qr = Merge({A_qr^(h), lse^(h)})).
//
// Each part h is softmax attention of the same queries over its own set of keys, with
// lse_h = log sum exp of its scaled logits.  Over the union of disjoint key sets the exact result is
//   A = sum_h w_h A_h / sum_h w_h,   w_h = exp(lse_h - max_h lse_h),   lse = max_h lse_h + log sum_h w_h.
// Every partial output is read once (16 bytes per lane per part), fp32 arithmetic.  The work is small and what bounds
// it is the chain of dependent steps and a cold instruction cache, so: the parts' log-sum-exps and outputs are requested
// together, indexes are 32-bit where they fit, and lanes are combined on the DPP path instead of through LDS.
// 16 parts of 64 x 16 rows of 128: 3.8 -> 2.8 us; 100 parts of 16 rows: 5.4 -> 2.6 us; 16 parts of 512 x 28: 19.9 -> 12.8.
#include "apbv_common.h"

namespace apbv {
namespace {

// op over groups of LP consecutive lanes (LP a power of two), the result in every lane of the group.
template <int LP, typename Op>
__device__ __forceinline__ float group_reduce(float x, Op op) {
  auto dpp = [&](auto ctrl, float y) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(y), decltype(ctrl)::value, 0xf, 0xf, false));
  };
  if (LP >= 2) x = op(x, dpp(std::integral_constant<int, 0xB1>{}, x));      // quad_perm [1,0,3,2]
  if (LP >= 4) x = op(x, dpp(std::integral_constant<int, 0x4E>{}, x));      // quad_perm [2,3,0,1]
  if (LP >= 8) x = op(x, dpp(std::integral_constant<int, 0x141>{}, x));     // row_half_mirror: the other quad of eight lanes
  if (LP >= 16) x = op(x, dpp(std::integral_constant<int, 0x140>{}, x));    // row_mirror: the other eight of sixteen
  if (LP >= 32) {
    auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  }
  if (LP >= 64) {
    auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  }
  return x;
}

// LP lanes share one 16-byte output chunk: lane `sub` takes parts sub, sub + LP, ...; up to kPartsPerLane of them are held
// in registers at once; with more the lanes loop over the parts (merge_lanes: how many lanes, and why).
template <int D, int LP, int kPartsPerLane>
__global__ __launch_bounds__(256) void merge_lse_kernel(const MergeParams p) {
  constexpr int KC = D / 8;
  const int64_t thread = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int sub = (int)(thread % LP);
  int64_t item = thread / LP;                                           // over batch * rows * hq * KC
  const int64_t n_items = (int64_t)p.batch * p.rows * p.hq * KC;
  const bool live = item < n_items;
  if (!live) item = n_items - 1;                                        // keep the lane for the exchanges; it writes nothing
  const int c = (int)(item % KC);
  const int64_t rh = item / KC;                                         // (b * rows + row) * hq + head
  int64_t lse_idx;
  if (n_items <= 0x7fffffff) {
    const uint32_t brow = (uint32_t)rh / (uint32_t)p.hq, h = (uint32_t)rh % (uint32_t)p.hq;
    const uint32_t b = p.batch == 1 ? 0 : brow / (uint32_t)p.rows;
    lse_idx = ((int64_t)b * p.hq + h) * p.rows + (brow - b * (uint32_t)p.rows);
  } else {
    const int64_t brow = rh / p.hq, b = brow / p.rows;
    lse_idx = (b * p.hq + rh % p.hq) * p.rows + brow % p.rows;
  }
  const float* lse = p.parts_lse + lse_idx;
  const bf16_t* x = p.parts_out + rh * D + 8 * c;

  auto fmax_ = [](float a, float b) { return fmaxf(a, b); };
  auto add_ = [](float a, float b) { return a + b; };
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  float wsum = 0.f;
  auto add_part = [&](float w, const u32x4 y) {
    wsum += w;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc[2 * e] = __builtin_fmaf(w, __uint_as_float(y[e] << 16), acc[2 * e]);
      acc[2 * e + 1] = __builtin_fmaf(w, __uint_as_float(y[e] & 0xffff0000u), acc[2 * e + 1]);
    }
  };
  float m = -INFINITY;
  if (p.n_parts <= kPartsPerLane * LP) {
    float l[kPartsPerLane];
    u32x4 y[kPartsPerLane];
#pragma unroll
    for (int u = 0; u < kPartsPerLane; ++u) {
      const int s = sub + u * LP;
      l[u] = -INFINITY;
      y[u] = u32x4{0u, 0u, 0u, 0u};
      if (s < p.n_parts) {
        l[u] = lse[s * p.stride_lse];
        y[u] = *reinterpret_cast<const u32x4*>(x + s * p.stride_out);
      }
    }
#pragma unroll
    for (int u = 0; u < kPartsPerLane; ++u) m = fmaxf(m, l[u]);
    m = group_reduce<LP>(m, fmax_);
    if (m > -INFINITY) {                                                // the same in all lanes of an item
#pragma unroll
      for (int u = 0; u < kPartsPerLane; ++u) add_part(__expf(l[u] - m), y[u]);      // exp(-inf) = 0: empty parts drop out
    }
  } else {
#pragma unroll 4
    for (int s = sub; s < p.n_parts; s += LP) m = fmaxf(m, lse[s * p.stride_lse]);
    m = group_reduce<LP>(m, fmax_);
    if (m > -INFINITY) {
#pragma unroll 4
      for (int s = sub; s < p.n_parts; s += LP)
        add_part(__expf(lse[s * p.stride_lse] - m), *reinterpret_cast<const u32x4*>(x + s * p.stride_out));
    }
  }
  wsum = group_reduce<LP>(wsum, add_);
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = group_reduce<LP>(acc[e], add_);
  if (!live || sub != 0) return;
  const float inv = wsum > 0.f ? 1.0f / wsum : 0.f;
  u32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f32x2 xy = {acc[2 * e] * inv, acc[2 * e + 1] * inv};
    bf16x2 bb = __builtin_convertvector(xy, bf16x2);
    o[e] = __builtin_bit_cast(uint32_t, bb);
  }
  *reinterpret_cast<u32x4*>(p.out + rh * D + 8 * c) = o;
  if (p.lse_out != nullptr && c == 0) p.lse_out[lse_idx] = wsum > 0.f ? m + __logf(wsum) : -INFINITY;
}

template <int LP, int kPartsPerLane = kMergePartsPerLane>
apbv_status launch_merge_variant(const MergeParams& p, hipStream_t stream) {
  const int64_t threads = merge_items(p.batch, p.rows, p.hq, p.d) * LP;
  const int64_t blocks = (threads + 255) / 256;
  if (blocks > 0x7fffffff) return APBV_ERR_UNSUPPORTED;
  Launcher launch(stream);
  if (p.d == 128)
    launch(merge_lse_kernel<128, LP, kPartsPerLane>, dim3((unsigned)blocks), dim3(256), 0, p);
  else if (p.d == 64)
    launch(merge_lse_kernel<64, LP, kPartsPerLane>, dim3((unsigned)blocks), dim3(256), 0, p);
  else
    return APBV_ERR_UNSUPPORTED;
  return launch.status();
}

}  // namespace

apbv_status launch_merge_lse(const MergeParams& p, hipStream_t stream) {
  switch (merge_lanes(merge_items(p.batch, p.rows, p.hq, p.d), p.n_parts)) {
    case 1: return p.n_parts <= kMergePartsPerLane ? launch_merge_variant<1>(p, stream) : launch_merge_variant<1, 2 * kMergePartsPerLane>(p, stream);
    case 2: return launch_merge_variant<2>(p, stream);
    case 4: return launch_merge_variant<4>(p, stream);
    case 8: return launch_merge_variant<8>(p, stream);
    case 16: return launch_merge_variant<16>(p, stream);
    case 64: return launch_merge_variant<64>(p, stream);
  }
  return APBV_ERR_UNSUPPORTED;
}

}  // namespace apbv
