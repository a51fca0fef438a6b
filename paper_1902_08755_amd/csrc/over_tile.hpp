// Workgroup tile body of ordered "over" compositing, shared by the plain
// launch and the persistent batched launch.
//
// Thesis Section 5.2.1: partial images of convex regions are sorted by depth
// and blended in that order. Per pixel, back to front from transparent black:
//     acc <- L + (1 - L.a) * acc        (FP32 fused multiply-add per channel)
// A layer that does not cover the pixel leaves acc unchanged.
//
// Mapping: a wave composites 64 consecutive pixels of one row at a time, so a
// layer's row segment is one coalesced stream of 16-byte (RGBA32F) or 8-byte
// (RGBA16F) loads, and everything that depends on the row and the layer but
// not on the pixel is the same for the whole wave. That part is done for 64
// layers at once, one layer per lane: whether the layer reaches the segment,
// the address of the segment's first pixel in it, and the lanes it covers. A
// ballot lists the layers that reach the segment; each of them then costs
// three lane reads, the cover test and one load (the loop it replaces read
// every placement from LDS and made it uniform once per pixel row and layer,
// about 19 vector instructions each: the 256 jobs of the batch took 2155 us,
// and 1880 with this, before the batch's queues were divided). Loads of up to
// over_batch layers are issued before the first of them is blended; the blend
// chain itself stays strictly in order.
#pragma once

#include "cmp_internal.hpp"

namespace cmp {

struct OverDesc {
  const void* color;   // RGBA32F or RGBA16F
  int64_t pitch;
  int32_t x, y, w, h;  // placement
};

// A stored pixel before widening: FP16 pixels stay packed in two registers
// until they are blended.
template <int FMT>
struct RawPx { typedef f32x4 type; };
template <>
struct RawPx<CMP_RGBA16F> { typedef f16x4 type; };

__device__ __forceinline__ f32x4 widen(f32x4 v) { return v; }
__device__ __forceinline__ f32x4 widen(f16x4 h) {
  return f32x4{(float)h.x, (float)h.y, (float)h.z, (float)h.w};
}

// Most layers whose loads are in flight together: 128 bytes per lane either
// way. What is left of a segment's layers is taken in a half or a quarter of
// that, so that few slots of a batch are padding.
template <int FMT>
constexpr int over_batch() { return FMT == CMP_RGBA32F ? 8 : 16; }
constexpr int kOverBatch = 8;   // the backward pass (FP32 and FP16 alike)

__device__ __forceinline__ f32x4 over_op(f32x4 front, f32x4 back) {
  const float t = 1.0f - front.w;
  return f32x4{__builtin_fmaf(t, back.x, front.x), __builtin_fmaf(t, back.y, front.y),
               __builtin_fmaf(t, back.z, front.z), __builtin_fmaf(t, back.w, front.w)};
}

// Up to 64 layers of a back-to-front list, one per lane.
__device__ __forceinline__ OverDesc lane_layer(const OverDesc* __restrict__ d, int c0, int n) {
  const int j = c0 + (int)(threadIdx.x % kWave);
  return j < n ? d[j] : OverDesc{nullptr, 0, 0, 0, 0, 0};
}

// The address of pixel (X0, Y) of a layer placed at (x, y).
template <int FMT>
__device__ __forceinline__ uint64_t over_address(const void* base, int64_t pitch, int32_t x,
                                                 int32_t y, int X0, int Y) {
  constexpr int bpp = FMT == CMP_RGBA32F ? 16 : 8;
  const int dx = __builtin_elementwise_sub_sat(x, X0);   // exact where the layer reaches the segment
  const uint32_t dy = (uint32_t)Y - (uint32_t)y;
  return (uint64_t)reinterpret_cast<uintptr_t>(base) +
         ((uint64_t)dy * (uint64_t)pitch - (uint64_t)(int64_t)dx) * bpp;
}

// This lane's layer at the row segment [X0, X0 + cols) of row Y (cols <= 64):
// the address of the segment's first pixel in the layer (outside the buffer
// when the layer starts further right; only covered pixels are read), and
// the covered lanes as first | count << 8. `hits` is the ballot of the
// layers that reach the segment. Every lane of the wave must be active.
struct OverSeg {
  uint32_t lo, hi;   // address
  uint32_t span;
};
template <int FMT>
__device__ __forceinline__ OverSeg over_segment(const OverDesc& D, int X0, int cols, int Y,
                                                uint64_t& hits) {
  // saturating, so that placements near the ends of the 32-bit range work
  // too: where a layer reaches the segment nothing saturates
  const int dx = __builtin_elementwise_sub_sat(D.x, X0);
  const uint32_t dy = (uint32_t)Y - (uint32_t)D.y;
  const int first = min(max(dx, 0), kWave), end = min(__builtin_elementwise_add_sat(dx, D.w), cols);
  hits = (uint64_t)__ballot(dy < (uint32_t)D.h && first < end);
  const uint64_t a = over_address<FMT>(D.color, D.pitch, D.x, D.y, X0, Y);
  return OverSeg{(uint32_t)a, (uint32_t)(a >> 32), (uint32_t)first | (uint32_t)(end - first) << 8};
}

// Blends the next (at most N) layers of `hits` onto acc in increasing order,
// taking them out of it; before(i) runs ahead of layer i (lane i's layer).
// The loads are unconditional, so that no branch separates them: a slot past
// the last layer repeats the batch's first layer, and a lane outside a layer
// reads the layer's first covered pixel; both results are discarded.
template <int FMT, int N, typename F>
__device__ __forceinline__ void over_blend(const OverSeg& sg, uint64_t& hits, int lane, f32x4& acc,
                                           F before) {
  constexpr uint32_t bpp = FMT == CMP_RGBA32F ? 16 : 8;
  typedef typename RawPx<FMT>::type Raw;
  typedef const __attribute__((address_space(1))) Raw* GPtr;
  typedef const __attribute__((address_space(1))) char* GBytes;
  Raw L[N];
  bool cov[N], has[N];
  int id[N];
  const int first = (int)__builtin_ctzll(hits);
#pragma unroll
  for (int k = 0; k < N; ++k) {
    has[k] = hits != 0;
    id[k] = has[k] ? (int)__builtin_ctzll(hits) : first;
    hits &= hits - 1;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)sg.lo, id[k]);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)sg.hi, id[k]);
    const uint32_t span = (uint32_t)__builtin_amdgcn_readlane((int)sg.span, id[k]);
    const uint32_t c0 = span & 0xFFu, cn = has[k] ? span >> 8 : 0u;
    cov[k] = (uint32_t)lane - c0 < cn;
    const uint32_t off = (cov[k] ? (uint32_t)lane : c0) * bpp;
    const GBytes base = (GBytes)(((uint64_t)hi << 32) | lo);
    // non-temporal: each layer pixel is read once (measured faster than the
    // default policy for this kernel and the backward pass)
    L[k] = __builtin_nontemporal_load((GPtr)(base + off));
  }
#pragma unroll
  for (int k = 0; k < N; ++k) {
    if (has[k]) before(id[k]);   // uniform
    if (cov[k]) acc = over_op(widen(L[k]), acc);
  }
}

// Blends every layer of `hits` onto acc.
template <int FMT, typename F>
__device__ __forceinline__ void over_hits(const OverSeg& sg, uint64_t hits, int lane, f32x4& acc,
                                          F before) {
  constexpr int B = over_batch<FMT>();
  int left = (int)__builtin_popcountll(hits);
  while (left > B / 2) {   // uniform
    over_blend<FMT, B>(sg, hits, lane, acc, before);
    left -= B;
  }
  if (left > B / 4)
    over_blend<FMT, B / 2>(sg, hits, lane, acc, before);
  else if (left > 0)
    over_blend<FMT, B / 4>(sg, hits, lane, acc, before);
}

// Runs body(Y, X0, cols) for every row segment of a tile that falls to the
// calling wave: the four waves take the segments in turn, row by row.
template <typename F>
__device__ __forceinline__ void over_segments(int x0, int y0, int tw, int th, F body) {
  const int wave = uniform((int)(threadIdx.x / kWave));
  const int per_row = (tw + kWave - 1) / kWave;
  int r = wave / per_row, s = wave - r * per_row;
  const int dr = (kThreads / kWave) / per_row, ds = (kThreads / kWave) - dr * per_row;
  while (r < th) {
    body(y0 + r, x0 + s * kWave, min(kWave, tw - s * kWave));
    r += dr;
    s += ds;
    if (s >= per_row) {
      s -= per_row;
      ++r;
    }
  }
}

// The tile that a requested one is run as: rows are composited 64 pixels at a
// time, so a width is rounded up to a multiple of 64 and the height taken to
// keep the area (16x16 runs as 64x4, which keeps every lane busy).
inline void over_tile_shape(int& tw, int& th) {
  const int w = (tw + kWave - 1) / kWave * kWave;
  th = (int)((int64_t)tw * th / w);
  if (th < 1) th = 1;
  tw = w;
}

// Sequential order (also direct send: same per-pixel chain). `mine`: the
// caller's lane_layer(d, 0, n), which serves every tile when n <= 64.
template <int FMT>
__device__ __forceinline__ void over_tile_seq(const OverDesc* __restrict__ d, const OverDesc& mine,
                                              int n, int x0, int y0, int tw, int th,
                                              float* __restrict__ out, int64_t out_pitch, int vx,
                                              int vy, bool accumulate) {
  const int lane = threadIdx.x % kWave;
  over_segments(x0, y0, tw, th, [&](int Y, int X0, int cols) {
    f32x4* o = reinterpret_cast<f32x4*>(out) + ((int64_t)(Y - vy) * out_pitch + (X0 + lane - vx));
    f32x4 acc{0.f, 0.f, 0.f, 0.f};
    if (accumulate && lane < cols) acc = *o;
    uint64_t hits;
    for (int c0 = 0; c0 < n || c0 == 0; c0 += kWave) {
      const OverSeg sg = n <= kWave ? over_segment<FMT>(mine, X0, cols, Y, hits)
                                    : over_segment<FMT>(lane_layer(d, c0, n), X0, cols, Y, hits);
      over_hits<FMT>(sg, hits, lane, acc, [](int) {});
    }
    if (lane < cols) __builtin_nontemporal_store(acc, o);
  });
}

// Binary-swap merge order (Section 5.2.2): `groups` (a power of two, <= 64)
// contiguous groups of the back-to-front list, group g = positions
// [floor(g n / groups), floor((g + 1) n / groups)), each composited alone,
// then merged pairwise level by level: merge(back, front) = front +
// (1 - front.a) * back. The pending partial of each level is kept in LDS (a
// binary counter over the groups; `lvl` holds one pixel per thread for each
// of log2(groups) levels). n <= 64.
// The layers are taken in the same full batches of loads as without groups,
// and a group is closed between two blends; a batch per group, which this
// replaces, loaded and discarded most of its slots (40 partial FP16 layers in
// 8 groups over 1921x1081: 203 us, bound by 2419 vector instructions per
// wave; with full batches 79 us, 69 since XCDs take runs of tiles).
template <int FMT>
__device__ __forceinline__ void over_tile_tree(const OverDesc* __restrict__ d, int n, int groups,
                                               int x0, int y0, int tw, int th,
                                               float* __restrict__ out, int64_t out_pitch, int vx,
                                               int vy, f32x4* lvl) {
  const int lane = threadIdx.x % kWave;
  const int shift = 31 - __builtin_clz((unsigned)groups);
  const OverDesc mine = lane_layer(d, 0, n);
  over_segments(x0, y0, tw, th, [&](int Y, int X0, int cols) {
    f32x4 acc{0.f, 0.f, 0.f, 0.f};
    int g = 0, next = n >> shift;   // the open group and the position that ends it
    auto close = [&]() {            // uniform
      int l = 0;
      for (; (g >> l) & 1; ++l) acc = over_op(acc, lvl[l * kThreads + threadIdx.x]);
      ++g;
      next = ((g + 1) * n) >> shift;
      if (g == groups) return;      // the last one: acc is the result
      lvl[l * kThreads + threadIdx.x] = acc;
      acc = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    uint64_t hits;
    const OverSeg sg = over_segment<FMT>(mine, X0, cols, Y, hits);
    over_hits<FMT>(sg, hits, lane, acc, [&](int i) {
      while (i >= next) close();
    });
    while (g < groups) close();
    if (lane < cols)
      __builtin_nontemporal_store(acc, reinterpret_cast<f32x4*>(out) +
                                           ((int64_t)(Y - vy) * out_pitch + (X0 + lane - vx)));
  });
}

}  // namespace cmp
