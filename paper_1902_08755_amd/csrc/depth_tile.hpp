// Workgroup tile body of depth-sorted compositing, shared by the plain launch
// and the persistent batched launch.
//
// Thesis Section 5.2.1 (Spatial and Depth-Sorted Sort-Last Compositing): a
// final pixel takes the colour of the source with the front-most depth. Here:
// the smallest (depth, index) pair over the contributors covering the pixel;
// the clear depth never wins.
//
// Mapping: lane = column. A wave covers 64 consecutive pixels of a tile row
// and steps over 4 rows at a time (the four waves of a workgroup take
// interleaved row groups), so every load of a contributor row is one
// coalesced 256-byte access per wave, and a contributor's left or right edge
// is only a per-lane mask. Per contributor only the depth is read; the
// colour is gathered once, from the winner, at the end ("lean" traffic: 4
// bytes per covering contributor plus 4 for the winner). Contributors are
// visited in index order with a strict "<", so ties keep the lower index.
// The loads of four contributors x four rows are issued before any compare.
#pragma once

#include <type_traits>

#include "cmp_internal.hpp"

namespace cmp {

struct DepthDesc {
  const uint32_t* color;
  const uint32_t* depth;
  int64_t pitch;
  int32_t x, y, w, h;   // placement (host rectangle; bounds the buffer)
};

// Composites the tile [x0, x0+tw) x [y0, y0+th) (destination pixels) of a
// viewport whose origin is (vx, vy) into out_color/out_depth. With
// `accumulate`, the outputs already hold the result of earlier contributors
// (a previous pass) and are combined under the same rule.
constexpr int kDepthRows = 4;    // rows per lane per step, but for small views
constexpr int kDepthBatch = 4;   // covering contributors whose loads are in flight together

typedef const __attribute__((address_space(1))) uint32_t* GlobalU32;

// A contributor as the tile reads it: placement and buffers.
struct DepthRec {
  int32_t x, y, w, h;
  const uint32_t* depth;
  const uint32_t* color;
  int64_t pitch;
};

// Stages contributors [0, n) in LDS: their placements (the host rectangle or
// the device ROI, clamped to the host size) and buffers. desc(i) gives
// contributor i's descriptor. `roi_dev` (device int32[][4], row index_base + i
// for contributor i) may override placements (crop == 0) or crop the
// contributors to the rectangles that hold their data (crop == 1: the buffers
// stay where the descriptors place them). All threads of the workgroup; ends
// with a barrier.
template <typename F>
__device__ __forceinline__ void stage_contributors(F desc, int n, const int32_t* roi_dev,
                                                   int index_base, int crop, DepthRec* rec) {
  for (int i = threadIdx.x; i < n; i += kThreads) {
    const DepthDesc D = desc(i);
    DepthRec r{D.x, D.y, D.w, D.h, D.depth, D.color, D.pitch};
    if (roi_dev && crop) {
      // the part of the placed buffer inside the device rectangle
      const int4 q = reinterpret_cast<const int4*>(roi_dev)[index_base + i];
      const int x0 = max(q.x, D.x), y0 = max(q.y, D.y);
      const int x1 = min(q.x + max(q.z, 0), D.x + D.w), y1 = min(q.y + max(q.w, 0), D.y + D.h);
      r.x = x0;
      r.y = y0;
      r.w = max(0, x1 - x0);
      r.h = max(0, y1 - y0);
      if (r.w > 0 && r.h > 0) {
        const int64_t o = (int64_t)(y0 - D.y) * D.pitch + (x0 - D.x);
        r.depth = D.depth + o;
        r.color = D.color + o;
      }
    } else if (roi_dev) {
      const int4 q = reinterpret_cast<const int4*>(roi_dev)[index_base + i];
      r.x = q.x;
      r.y = q.y;
      r.w = max(0, min(q.z, D.w));
      r.h = max(0, min(q.w, D.h));
    }
    if (!D.depth || r.w <= 0 || r.h <= 0) r.w = r.h = 0;
    rec[i] = r;
  }
  __syncthreads();
}

// `rec`: contributors staged by stage_contributors.
// Per step a wave takes 64 contributors at a time, one per lane: whether the
// contributor covers pixels of the wave's rows and columns, the address of the
// step's first pixel in it, its row pitch, and the columns and rows it covers.
// A ballot lists the covering ones; each of them then costs five lane reads
// and scalar arithmetic for its row addresses (it replaces LDS reads made
// uniform and tests of row and column per lane: 40 partial contributors over
// 1920x1080 15.3 -> 14.7 us, 200 over 1281x719 68.7 -> 65.3).
// kDepthBatch covering contributors x kRows rows are loaded at a time, so the
// depth loads of a typical step are one round trip; the winner's colour is
// gathered at the end.
template <int kRows>
__device__ __forceinline__ void depth_tile(const DepthRec* rec, int n, int x0, int y0, int tw,
                                           int th, uint32_t* __restrict__ out_color,
                                           uint32_t* __restrict__ out_depth, int64_t out_pitch,
                                           int vx, int vy, bool accumulate) {
  typedef const __attribute__((address_space(1))) char* Bytes;
  const int lane = threadIdx.x % kWave, wave = uniform((int)(threadIdx.x / kWave));
  constexpr int kStepRows = kRows * (kThreads / kWave);
  for (int cx = 0; cx < tw; cx += kWave) {
    const int cx0 = x0 + cx, cols = min(kWave, tw - cx);   // the wave's columns
    const int X = cx0 + lane;
    const bool col_ok = lane < cols;
    for (int r0 = wave * kRows; r0 < th; r0 += kStepRows) {
      const int Y0 = y0 + r0;                       // rows Y0 .. Y0 + kRows - 1 (uniform)
      const int nrows = min(kRows, th - r0);
      uint32_t bd[kRows], pc[kRows];
      int bi[kRows];
#pragma unroll
      for (int k = 0; k < kRows; ++k) {
        bd[k] = kClearDepth;
        pc[k] = 0;
        bi[k] = -1;
        if (accumulate && col_ok && k < nrows) {
          const int64_t oo = (int64_t)(Y0 + k - vy) * out_pitch + (X - vx);
          bd[k] = out_depth[oo];
          pc[k] = out_color[oo];
        }
      }
      for (int c0 = 0; c0 < n; c0 += kWave) {   // uniform
        // lane i: contributor c0 + i (every lane of the wave is active: the
        // loops are uniform over it). Saturating, so that placements near the
        // ends of the 32-bit range work too: where a contributor covers
        // pixels of the step nothing saturates.
        const DepthRec& R = rec[min(c0 + lane, n - 1)];
        const int dx = __builtin_elementwise_sub_sat(R.x, cx0);
        const int dy = __builtin_elementwise_sub_sat(R.y, Y0);
        const int first = min(max(dx, 0), kWave), end = min(__builtin_elementwise_add_sat(dx, R.w), cols);
        const int k0 = min(max(dy, 0), kRows), k1 = min(__builtin_elementwise_add_sat(dy, R.h), nrows);
        uint64_t cover = (uint64_t)__ballot(c0 + lane < n && first < end && k0 < k1);
        const uint64_t pb = (uint64_t)R.pitch * 4;
        // of row Y0 + k0, the first covered one
        const uint64_t ad = (uint64_t)reinterpret_cast<uintptr_t>(R.depth) +
                            (uint64_t)(uint32_t)(k0 - dy) * pb - (uint64_t)((int64_t)dx * 4);
        const uint32_t span = (uint32_t)first | (uint32_t)(end - first) << 8 | (uint32_t)k0 << 16 |
                              (uint32_t)k1 << 20;
        auto of_lane = [](uint32_t v, int i) {
          return (uint32_t)__builtin_amdgcn_readlane((int)v, i);
        };
        // the next N covering contributors (a slot past the last one repeats
        // the first and is ignored), then every load of the batch, then the
        // compares: no branch between the loads
        auto batch = [&](auto size) {
          constexpr int N = decltype(size)::value;
          int ids[N];
          uint32_t dv[N][kRows];
          bool ok[N][kRows];
          const int i0 = (int)__builtin_ctzll(cover);
#pragma unroll
          for (int j = 0; j < N; ++j) {
            const bool has = cover != 0;
            const int i = has ? (int)__builtin_ctzll(cover) : i0;
            cover &= cover - 1;
            ids[j] = c0 + i;
            const uint32_t s = of_lane(span, i);
            const uint64_t pitch = (uint64_t)of_lane((uint32_t)(pb >> 32), i) << 32 | of_lane((uint32_t)pb, i);
            uint64_t row = (uint64_t)of_lane((uint32_t)(ad >> 32), i) << 32 | of_lane((uint32_t)ad, i);
            const uint32_t f = s & 0xFFu, cnt = has ? (s >> 8) & 0xFFu : 0u;
            const int a0 = (int)(s >> 16) & 15, a1 = (int)(s >> 20);
            // a pixel outside the contributor reads its first covered column
            // or a covered row instead
            const bool in_col = (uint32_t)lane - f < cnt;
            const uint32_t off = (in_col ? (uint32_t)lane : f) * 4u;
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
              dv[j][k] = *(GlobalU32)((Bytes)row + off);
              ok[j][k] = in_col && k >= a0 && k < a1;
              if (k >= a0 && k + 1 < a1) row += pitch;
            }
          }
          // ascending indices and a strict "<": ties keep the lower index
#pragma unroll
          for (int j = 0; j < N; ++j) {
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
              if (ok[j][k] && dv[j][k] < bd[k]) {
                bd[k] = dv[j][k];
                bi[k] = ids[j];
              }
            }
          }
        };
        // (the last two or one in a smaller batch: 40 partial contributors over
        // 1920x1080 13.2 -> 12.6 us, 100 30.6 -> 30.2)
        int left = (int)__builtin_popcountll(cover);   // uniform
        for (; left > 2; left -= kDepthBatch) batch(std::integral_constant<int, kDepthBatch>());
        if (left > 0) batch(std::integral_constant<int, 2>());
      }
      // gather the winners' colours and store (4-byte accesses, coalesced
      // along the row across the wave; non-temporal stores, measured faster
      // here, while non-temporal loads were slower)
      if (col_ok) {
        uint32_t cv[kRows];
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
          cv[k] = pc[k];
          if (k < nrows && bi[k] >= 0) {
            const DepthRec& R = rec[bi[k]];
            cv[k] = ((GlobalU32)R.color)[(int64_t)(Y0 + k - R.y) * R.pitch + (X - R.x)];
          }
        }
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
          if (k >= nrows) continue;
          const int64_t oo = (int64_t)(Y0 + k - vy) * out_pitch + (X - vx);
          __builtin_nontemporal_store(cv[k], &out_color[oo]);
          if (out_depth) __builtin_nontemporal_store(bd[k], &out_depth[oo]);
        }
      }
    }
  }
}

}  // namespace cmp
