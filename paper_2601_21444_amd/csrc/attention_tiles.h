// Key/value tiles of the attention kernels (device code): the layout of a 32-key tile in LDS, the LDS-direct loads
// that fill it and the stream that walks the three KV segments as one virtual key axis.
#pragma once
#include "apbv_common.h"

namespace apbv {
namespace {

constexpr int kBN = 32;                     // keys per tile (one k-step of O^T)
constexpr float kRescaleThreshold = 8.0f;   // log2 units
constexpr float kReferenceBias = 4.0f;      // log2 units between a row's reference and what attention.hip subtracts
constexpr int kXcds = 8;                    // accelerator dies with an L2 of their own; workgroup id modulo 8

#define APBV_LDS(T) __attribute__((address_space(3))) T*

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

// Compile-time loop: f(std::integral_constant<int, 0>{}) ... f(std::integral_constant<int, N-1>{}).
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// kWide: read by the 32x32x16 matrix instruction (32 rows x 16 bytes of K at once, 4 rows x 64 bytes of V) instead of the
// 16x16x32 one; only the swizzle of V differs.
template <int D, int W, bool kWide = false>
struct Tile {
  static constexpr int ROW_BYTES = D * 2;
  static constexpr int KC = D / 8;                        // 16-byte chunks per row
  static constexpr int RPI = 1024 / ROW_BYTES;            // rows covered by one wave-wide LDS-direct load
  static constexpr int LOADS = kBN / RPI;                 // such loads per tile (per tensor)
  static constexpr int IPW = (LOADS + W - 1) / W;         // ... per wave; wave w issues loads w*IPW + u while < LOADS
  static constexpr int KSD = D / 32;                      // MFMA k-steps over the head dimension (S^T)
  static constexpr int DBN = D / 16;                      // 16-row blocks of O^T
  static constexpr int TILE_BYTES = kBN * ROW_BYTES;
  // chunk swizzles (functions of the row within the tile), chosen so that the 16 rows x 16 bytes of a quarter of
  // a K read and the 8 rows x 32 bytes of half a transposing V read cover the 64 LDS banks exactly once
  __device__ static __forceinline__ int fk(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
  __device__ static __forceinline__ int fv(int r) {
    if (kWide) return D == 128 ? ((r & 3) << 2) : (((r >> 1) & 1) << 2);
    return D == 128 ? ((r & 7) << 1) : (((r >> 1) & 3) << 1);
  }
};

struct Segs {
  const char *b0, *b1, *b2;   // byte pointers of the three segments, already offset to (batch, kv head)
  int64_t p0, p1, p2;         // bytes between consecutive tokens
  int64_t e0, e1, e2;         // one past the last virtual key of each segment (starts are 0, e0, e1)
};

// The three segments of K and of V for (batch item b, KV head kvh).
__device__ __forceinline__ void key_segments(const AttnParams& p, int b, int kvh, Segs& ks, Segs& vs) {
  auto base = [&](const View& t) { return reinterpret_cast<const char*>(t.ptr + (int64_t)b * t.sb + (int64_t)kvh * t.sh); };
  ks.b0 = base(p.k_seg[0]); ks.b1 = base(p.k_seg[1]); ks.b2 = base(p.k_seg[2]);
  vs.b0 = base(p.v_seg[0]); vs.b1 = base(p.v_seg[1]); vs.b2 = base(p.v_seg[2]);
  ks.p0 = p.k_seg[0].st * 2; ks.p1 = p.k_seg[1].st * 2; ks.p2 = p.k_seg[2].st * 2;
  vs.p0 = p.v_seg[0].st * 2; vs.p1 = p.v_seg[1].st * 2; vs.p2 = p.v_seg[2].st * 2;
  ks.e0 = vs.e0 = p.l_a; ks.e1 = vs.e1 = p.n_vis; ks.e2 = vs.e2 = p.s_kv;
}

// Pick the fields of the segment that holds virtual key j (selects, no indexed access).
__device__ __forceinline__ void seg_of(const Segs sg, int64_t j, const char*& base, int64_t& pitch, int64_t& start,
                                       int64_t& end) {
  const bool in0 = j < sg.e0, in1 = j < sg.e1;
  base = in0 ? sg.b0 : (in1 ? sg.b1 : sg.b2);
  pitch = in0 ? sg.p0 : (in1 ? sg.p1 : sg.p2);
  start = in0 ? 0 : (in1 ? sg.e0 : sg.e1);
  end = in0 ? sg.e0 : (in1 ? sg.e1 : sg.e2);
}

// LDS-direct 16-byte load: lane l's bytes land at lds_dst + 16*l (lds_dst uniform, in M0).  Issued through
// inline assembly so that the kernel, not the compiler's wait-count insertion, orders these loads against
// the LDS reads (one s_waitcnt vmcnt + barrier per tile).
__device__ __forceinline__ const char* uniform_ptr(const char* p) {      // a wave-uniform pointer, provably so
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const char*)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ void dma16_uniform(const char* base_uniform, uint32_t lane_off, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_dst), "v"(lane_off), "s"(base_uniform)
               : "memory", "m0");
}
__device__ __forceinline__ void dma16_lane(const char* addr, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_dst), "v"(addr) : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_addr(const unsigned char* p) { return (uint32_t)(size_t)(APBV_LDS(const unsigned char))p; }

// Sequential producer of the tiles of ONE tensor (K or V) along the virtual key axis.  While consecutive tiles
// stay inside one segment ("run") a tile costs one 64-bit scalar add and its loads are  uniform tile base + a
// per-lane 32-bit offset computed once per run; the tile that straddles a segment boundary (or the end of the
// keys) takes a per-row lookup.
template <int D, int W, bool kIsV, bool kWide = false>
struct TileStream {
  using T = Tile<D, W, kWide>;
  Segs sg;
  int64_t s_kv;
  int t_next;              // next tile to issue
  int run_end;             // tiles [t_next, run_end) lie inside one segment; base points at tile t_next
  const char* base;
  int64_t step;            // kBN * pitch
  uint32_t off[T::IPW];
  int wave, lane;

  __device__ static __forceinline__ int swz(int r) { return kIsV ? T::fv(r) : T::fk(r); }
  __device__ __forceinline__ int row(int u) const { return (wave * T::IPW + u) * T::RPI + lane / T::KC; }
  __device__ __forceinline__ uint32_t ldst(int u) const { return (uint32_t)((wave * T::IPW + u) * T::RPI * T::ROW_BYTES); }

  __device__ __forceinline__ void init(const Segs& s, int64_t skv, int w, int l, int t_first) {
    sg = s;
    s_kv = skv;
    wave = w;
    lane = l;
    t_next = t_first;
    run_end = t_first;
    base = nullptr;
    step = 0;
#pragma unroll
    for (int u = 0; u < T::IPW; ++u) off[u] = 0;
  }

  // Start a run at tile t_next if that tile lies inside one segment.
  __device__ __forceinline__ void start_run() {
    const int64_t j0 = (int64_t)t_next * kBN;
    const char* b;
    int64_t pitch, start, end;
    seg_of(sg, j0, b, pitch, start, end);
    if (j0 + kBN > end) return;                      // straddling tile: run stays empty
    run_end = (int)(end / kBN);
    base = b + (j0 - start) * pitch;
    step = kBN * pitch;
#pragma unroll
    for (int u = 0; u < T::IPW; ++u) {
      const int r = row(u);
      off[u] = (uint32_t)r * (uint32_t)pitch + 16u * (uint32_t)((lane % T::KC) ^ swz(r));
    }
  }

  // Whether load u of a tile is this wave's to issue (always, when the loads divide evenly among the waves).
  __device__ __forceinline__ bool mine(int u) const { return W * T::IPW == T::LOADS || wave * T::IPW + u < T::LOADS; }

  // Tiles that can still be issued from the current run without a lookup (after trying to start a run if none is open).
  __device__ __forceinline__ int run_left() {
    if (t_next >= run_end) start_run();
    return run_end - t_next;
  }
  // Issue tile t_next, which the caller knows to lie inside the current run: no tests.
  __device__ __forceinline__ void issue_in_run(uint32_t dst) {
    const char* bu = uniform_ptr(base);
#pragma unroll
    for (int u = 0; u < T::IPW; ++u)
      if (mine(u)) dma16_uniform(bu, off[u], dst + ldst(u));
    base += step;
    ++t_next;
  }

  // The u-th of the wave's IPW loads of tile t_next, which the caller knows to lie inside the current run; the last one moves
  // on to the next tile.  From tile t_last on it is t_last that is loaded, again and again.
  __device__ __forceinline__ void issue_in_run(uint32_t dst, int u, int t_last) {
    if (mine(u)) dma16_uniform(uniform_ptr(base), off[u], dst + ldst(u));
    if (u == T::IPW - 1) {
      base += t_next < t_last ? step : 0;
      ++t_next;
    }
  }

  // issue(), staying on tile t_last once there: the callers' last requests repeat it instead of being left out, so that
  // every step of a loop has the same loads outstanding.
  __device__ __forceinline__ void issue_until(uint32_t dst, int t_last) {
    issue(dst);
    if (t_next > t_last) {
      t_next = t_last;
      base -= step;                                    // (unused if t_last is a straddling tile: run_end <= t_last)
    }
  }

  // Issue this wave's share of the loads of tile t_next into the LDS tile at dst.
  __device__ __forceinline__ void issue(uint32_t dst) {
    if (t_next >= run_end) start_run();
    if (t_next < run_end) {
      const char* bu = uniform_ptr(base);
#pragma unroll
      for (int u = 0; u < T::IPW; ++u)
        if (mine(u)) dma16_uniform(bu, off[u], dst + ldst(u));
      base += step;
    } else {
      const int64_t j0 = (int64_t)t_next * kBN;
      // One wave's many loads stay a loop (code size costs launch time); a workgroup's few per wave are unrolled, so that
      // their lookups overlap: 6 queries of 28 heads over 85 keys (64-row
      // workgroups, the last of three tiles such a one) 7.7 -> 7.1 us.
      constexpr int kUnroll = W == 1 ? 1 : T::IPW;
#pragma unroll kUnroll
      for (int u = 0; u < T::IPW; ++u) {
        if (!mine(u)) continue;
        const int r = row(u);
        int64_t j = j0 + r;
        j = j < s_kv ? j : s_kv - 1;                 // rows past the end repeat the last key: always masked
        const char* b;
        int64_t pitch, sj, ej;
        seg_of(sg, j, b, pitch, sj, ej);
        dma16_lane(b + (j - sj) * pitch + 16 * ((lane % T::KC) ^ swz(r)), dst + ldst(u));
      }
    }
    ++t_next;
  }
};

}  // namespace
}  // namespace apbv
