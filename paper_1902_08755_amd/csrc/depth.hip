// cmp_composite_depth: plain launch of depth-sorted compositing
// (Section 5.2.1), with the direct-send / binary-swap schedules of
// Section 5.2.2 as tile assignments inside one launch.
#include <string.h>

#include "depth_tile.hpp"

namespace cmp {

// A pass's contributors and regions share the words of the kernel's arguments:
// kDescWords per contributor from the front, kRegionWords per region from the
// back. Up to 111 contributors fit (direct send to 16 owners: 102), so few
// calls need a second pass over the outputs (100 contributors over 1920x1080
// took three passes of 48, 22 + 22 + 11 us; one pass takes 30.7, 200 over
// 1281x719 five passes, 59 us, and now two, 37).
// A pitch is one word; where one does not fit, the upper words of all of them
// follow the contributors.
constexpr int kArgWords = 1004;
constexpr int kDescWords = 9, kRegionWords = sizeof(Region) / 4;
constexpr int kDepthPerPass = (kArgWords - kRegionWords) / kDescWords;
constexpr int kColorOnly = 48;   // most contributors without a depth output (include/cmp.h)

struct DepthArgs {
  const int32_t* roi_dev;
  uint32_t* out_color;
  uint32_t* out_depth;
  int64_t out_pitch;
  int32_t vx, vy;
  int32_t n, nreg;
  int32_t tile_w, tile_h;
  int32_t accumulate;
  int32_t index_base;
  int32_t crop;   // roi_dev crops the placed contributors (else it places them)
  int32_t wide;   // pitches have upper words
  uint32_t words[kArgWords];
};
static_assert(sizeof(DepthArgs) <= 4096, "kernel arguments must fit in 4 KiB");
static_assert(kColorOnly <= (kArgWords - kMaxRegions * kRegionWords) / (kDescWords + 1),
              "one pass takes kColorOnly contributors whatever the regions and pitches");

// Consecutive tiles per XCD: neighbouring tiles share the cache lines of rows
// that are no multiple of 128 bytes, and one L2 then reads them once (40
// partial contributors of 1920x1080: 14.7 us in launch order, 12.7 in runs of
// 16, 14.9 of 64; 30 of 1367x763: 25.9, 21.2, 22.0; 8 of 3841x2161: 61.1,
// 56.0, 56.1; 64 of 3840x2160 for 64 owners: 169, 167, 188).
constexpr int kDepthRun = 16;

__device__ __forceinline__ void tile_of_block(const Region& mine, int nreg, int tile_w, int tile_h,
                                              int& x0, int& y0, int& tw, int& th) {
  const int blk = xcd_tile((int)blockIdx.x, (int)gridDim.x, kDepthRun);
  // lane i holds region i (nreg <= 64, ascending tile_begin from 0)
  const int lane = threadIdx.x % kWave;
  const int r = (int)__builtin_popcountll(__ballot(lane < nreg && mine.tile_begin <= blk)) - 1;
  auto of_lane = [r](int v) { return __builtin_amdgcn_readlane(v, r); };
  const Region R{of_lane(mine.x), of_lane(mine.y), of_lane(mine.w), of_lane(mine.h),
                 of_lane(mine.tile_begin)};
  const int local = blk - R.tile_begin;
  const int tiles_x = (R.w + tile_w - 1) / tile_w;
  const int ty = local / tiles_x, tx = local - ty * tiles_x;
  x0 = R.x + tx * tile_w;
  y0 = R.y + ty * tile_h;
  tw = min(tile_w, R.x + R.w - x0);
  th = min(tile_h, R.y + R.h - y0);
}

template <int kRows>
__device__ __forceinline__ void depth_body(const DepthArgs& a) {
  // in flight while the contributors are staged
  const Region mine = (reinterpret_cast<const Region*>(a.words + kArgWords) -
                       a.nreg)[min((int)(threadIdx.x % kWave), a.nreg - 1)];
  __shared__ DepthRec s_rec[kDepthPerPass];
  stage_contributors(
      [&](int i) {
        const uint32_t* d = a.words + kDescWords * i;
        auto ptr = [&](int k) {
          return reinterpret_cast<const uint32_t*>((uint64_t)d[k + 1] << 32 | d[k]);
        };
        const uint32_t up = a.wide ? a.words[kDescWords * a.n + i] : 0u;
        return DepthDesc{ptr(0), ptr(2), (int64_t)((uint64_t)up << 32 | d[4]), (int32_t)d[5],
                         (int32_t)d[6], (int32_t)d[7], (int32_t)d[8]};
      },
      a.n, a.roi_dev, a.index_base, a.crop, s_rec);   // a.n <= kDepthPerPass
  int x0, y0, tw, th;
  tile_of_block(mine, a.nreg, a.tile_w, a.tile_h, x0, y0, tw, th);
  depth_tile<kRows>(s_rec, a.n, x0, y0, tw, th, a.out_color, a.out_depth, a.out_pitch, a.vx, a.vy,
                    a.accumulate != 0);
}

// Eight waves per SIMD: at the compiler's default the kernel used 106 SGPRs,
// which held it to seven (measured on 16 x 1920x1080 cropped frames:
// 22.85 -> 21.7 us; forcing eight on the over and batch kernels made them
// spill and run slower).
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void depth_kernel(
    const DepthArgs a) {
  depth_body<kDepthRows>(a);
}

// Two rows per lane, for views that have few tiles: a wave's chain of loads
// (arguments, placements, depths, the winners' colours) is what takes the
// time there, and twice the waves of half the rows overlap more of it. Below
// kSmallTiles tiles of 64x16 (six workgroups per CU): 30 contributors over
// 1367x763, 1056 tiles, 20.9 -> 19.3 us, 200 over 1281x719 36 -> 31, the
// cropped frames of 24 x 1279x719 14.2 -> 12.3; above: 40 over 1920x1080, 2040
// tiles, 12.9 -> 14.6, 8 over 3841x2161 57 -> 59.4. One row per lane is slower
// at every size (28.6, 41.6).
constexpr int kSmallRows = 2, kSmallTiles = 1536;
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void
depth_small_kernel(const DepthArgs a) {
  depth_body<kSmallRows>(a);
}

// Host-side validation of one contributor list; shared with the batch planner.
cmp_status validate_depth_inputs(const cmp_image* in, int32_t n) {
  CMP_REQUIRE(n >= 0, "n = %d is negative", n);
  CMP_REQUIRE(n == 0 || in, "in is NULL");
  for (int i = 0; i < n; ++i) {
    const cmp_image& I = in[i];
    CMP_REQUIRE(rect_valid(I.roi), "in[%d].roi has a negative size", i);
    if (rect_empty(I.roi)) continue;
    CMP_REQUIRE(I.color && I.depth, "in[%d]: color and depth are required", i);
    CMP_REQUIRE(I.pitch >= I.roi.w, "in[%d].pitch %lld < roi.w %d", i, (long long)I.pitch,
                I.roi.w);
    CMP_REQUIRE(((uintptr_t)I.color & 3) == 0 && ((uintptr_t)I.depth & 3) == 0,
                "in[%d]: buffers must be 4-byte aligned", i);
  }
  return CMP_OK;
}

}  // namespace cmp

using namespace cmp;

static cmp_status composite_depth_impl(const cmp_image* in, int32_t n, const int32_t* roi_dev,
                                       bool crop, cmp_rect viewport, uint32_t* out_color,
                                       uint32_t* out_depth, int64_t out_pitch,
                                       cmp_schedule sched, cmp_tile tile, void* stream) {
  cmp_status st = validate_depth_inputs(in, n);
  if (st != CMP_OK) return st;
  CMP_REQUIRE(rect_valid(viewport), "viewport has a negative size");
  if (rect_empty(viewport)) return CMP_OK;
  CMP_REQUIRE(out_color, "out_color is NULL");
  CMP_REQUIRE(out_pitch >= viewport.w, "out_pitch %lld < viewport.w %d", (long long)out_pitch,
              viewport.w);
  CMP_REQUIRE(((uintptr_t)out_color & 3) == 0 && ((uintptr_t)out_depth & 3) == 0,
              "outputs must be 4-byte aligned");
  CMP_REQUIRE(n <= kColorOnly || out_depth,
              "out_depth is required when n > %d (it carries the result between passes)",
              kColorOnly);
  CMP_REQUIRE(((uintptr_t)roi_dev & 15) == 0, "roi_dev must be 16-byte aligned");
  const int64_t tiles16 = ((int64_t)viewport.w + 63) / 64 * (((int64_t)viewport.h + 15) / 16);
  const bool small = tile.w == 0 && tile.h == 0 && tiles16 < kSmallTiles;
  const int tw = tile.w ? tile.w : 64;
  const int th = tile.h ? tile.h : small ? kSmallRows * (kThreads / kWave) : 16;
  CMP_REQUIRE(tw > 0 && th > 0 && (int64_t)tw * th <= 65536,
              "tile %dx%d: sizes must be positive, area <= 65536", tw, th);

  DepthArgs a;
  memset(&a, 0, sizeof a);
  int64_t tiles = 0;
  Region reg[kMaxRegions];
  const int nreg = plan_regions(sched, viewport, tw, th, reg, &tiles);
  if (nreg < 0) return nreg;
  memcpy(a.words + kArgWords - nreg * kRegionWords, reg, nreg * sizeof(Region));
  CMP_REQUIRE(tiles < (1ll << 24), "too many tiles (%lld)", (long long)tiles);
  a.roi_dev = roi_dev;
  a.crop = crop ? 1 : 0;
  a.out_color = out_color;
  a.out_depth = out_depth;
  a.out_pitch = out_pitch;
  a.vx = viewport.x;
  a.vy = viewport.y;
  a.nreg = nreg;
  a.tile_w = tw;
  a.tile_h = th;
  hipStream_t s = (hipStream_t)stream;
  bool wide = false;
  for (int i = 0; i < n; ++i)
    if (!rect_empty(in[i].roi) && in[i].pitch > (int64_t)UINT32_MAX) wide = true;
  a.wide = wide ? 1 : 0;
  const int most = (kArgWords - nreg * kRegionWords) / (kDescWords + a.wide);
  int base = 0;
  do {
    const int cnt = n - base < most ? n - base : most;
    for (int i = 0; i < cnt; ++i) {
      const cmp_image& I = in[base + i];
      const bool empty = rect_empty(I.roi);
      const uint64_t v[3] = {empty ? 0 : (uint64_t)(uintptr_t)I.color,
                             empty ? 0 : (uint64_t)(uintptr_t)I.depth,
                             empty ? 0 : (uint64_t)I.pitch};
      uint32_t* d = a.words + kDescWords * i;
      for (int k = 0; k < 2; ++k) {
        d[2 * k] = (uint32_t)v[k];
        d[2 * k + 1] = (uint32_t)(v[k] >> 32);
      }
      d[4] = (uint32_t)v[2];
      d[5] = (uint32_t)I.roi.x;
      d[6] = (uint32_t)I.roi.y;
      d[7] = empty ? 0 : (uint32_t)I.roi.w;
      d[8] = empty ? 0 : (uint32_t)I.roi.h;
      if (wide) a.words[kDescWords * cnt + i] = (uint32_t)(v[2] >> 32);
    }
    a.n = cnt;
    a.accumulate = base > 0;
    a.index_base = base;
    if (small)
      hipLaunchKernelGGL(depth_small_kernel, dim3((unsigned)tiles), dim3(kThreads), 0, s, a);
    else
      hipLaunchKernelGGL(depth_kernel, dim3((unsigned)tiles), dim3(kThreads), 0, s, a);
    CMP_CHECK_HIP(hipGetLastError());
    base += cnt;
  } while (base < n);
  return CMP_OK;
}

extern "C" cmp_status cmp_composite_depth(const cmp_image* in, int32_t n, const int32_t* roi_dev,
                                          cmp_rect viewport, uint32_t* out_color,
                                          uint32_t* out_depth, int64_t out_pitch,
                                          cmp_schedule sched, cmp_tile tile, void* stream) {
  CMP_RANGE("cmp_composite_depth");
  return composite_depth_impl(in, n, roi_dev, false, viewport, out_color, out_depth, out_pitch,
                              sched, tile, stream);
}

extern "C" cmp_status cmp_composite_depth_crop(const cmp_image* in, int32_t n,
                                               const int32_t* roi_dev, cmp_rect viewport,
                                               uint32_t* out_color, uint32_t* out_depth,
                                               int64_t out_pitch, cmp_schedule sched,
                                               cmp_tile tile, void* stream) {
  CMP_RANGE("cmp_composite_depth_crop");
  CMP_REQUIRE(roi_dev, "roi_dev is required");
  return composite_depth_impl(in, n, roi_dev, true, viewport, out_color, out_depth, out_pitch,
                              sched, tile, stream);
}
