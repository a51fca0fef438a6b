// cmp_composite_over / cmp_composite_over_backward: ordered premultiplied
// "over" compositing (Section 5.2.1) and its adjoint.
#include <stdlib.h>
#include <string.h>

#include <algorithm>

#include "over_tile.hpp"

namespace cmp {

constexpr int kOverPerPass = 64;
static_assert(kOverPerPass <= kWave, "a pass's layers are held one per lane");

struct OverArgs {
  OverDesc c[kOverPerPass];      // back to front
  Region reg[kMaxRegions];
  float* out;
  int64_t out_pitch;
  int32_t vx, vy;
  int32_t n, nreg;
  int32_t tile_w, tile_h;
  int32_t accumulate;
  int32_t groups;                // 0: sequential chain
};
static_assert(sizeof(OverArgs) <= 4096, "kernel arguments must fit in 4 KiB");

// Consecutive tiles per XCD: neighbouring tiles share the cache lines of rows
// that are no multiple of 128 bytes, and one L2 then reads them once (20 FP32
// layers of 1919x1079: 127 us in launch order, 120 in runs of 16; 40 FP16 of
// 1921x1081: 143, 130.6; in 8 binary-swap groups 160, 150; 32 FP32 of
// 1024x1024: 100.5, 92; 16 of 3840x2160, whose lines nothing shares: 376
// either way). Runs of 256 spread 1024x1024 better over the memory channels
// (88 us) and lose on the others (122 us, 130.6, 378).
constexpr int kFwdRun = 16;

__device__ __forceinline__ void region_tile(const Region* reg, int nreg, int tile_w, int tile_h,
                                            int& x0, int& y0, int& tw, int& th) {
  const int blk = xcd_tile((int)blockIdx.x, (int)gridDim.x, kFwdRun);
  const int r = segment_of([&](int i) { return reg[i].tile_begin; }, nreg, blk);
  const Region R = reg[r];
  const int local = blk - R.tile_begin;
  const int tiles_x = (R.w + tile_w - 1) / tile_w;
  const int ty = local / tiles_x, tx = local - ty * tiles_x;
  x0 = R.x + tx * tile_w;
  y0 = R.y + ty * tile_h;
  tw = min(tile_w, R.x + R.w - x0);
  th = min(tile_h, R.y + R.h - y0);
}

template <int FMT>
__global__ __launch_bounds__(kThreads) void over_kernel(const OverArgs a) {
  int x0, y0, tw, th;
  region_tile(a.reg, a.nreg, a.tile_w, a.tile_h, x0, y0, tw, th);
  over_tile_seq<FMT>(a.c, lane_layer(a.c, 0, a.n), a.n, x0, y0, tw, th, a.out, a.out_pitch, a.vx,
                     a.vy, a.accumulate != 0);
}

template <int FMT>
__global__ __launch_bounds__(kThreads) void over_tree_kernel(const OverArgs a) {
  int x0, y0, tw, th;
  region_tile(a.reg, a.nreg, a.tile_w, a.tile_h, x0, y0, tw, th);
  extern __shared__ f32x4 lvl[];   // [log2(groups)][kThreads]
  over_tile_tree<FMT>(a.c, a.n, a.groups, x0, y0, tw, th, a.out, a.out_pitch, a.vx, a.vy, lvl);
}

// ------------------------------------------------------------- backward
// For the pixel's covering layers in front-to-back order i, with
// T_0 = 1, T_{i+1} = T_i (1 - a_i) and S_i = L_i + (1 - a_i) S_{i+1}:
//     grad L_i = G T_i,   grad a_i += -T_i <G, S_{i+1}>.
// As in the forward pass a wave takes 64 pixels of a row at a time. It lists
// the layers that reach them, back to front, in LDS (the address of the first
// pixel in the layer and in its gradient, and the covered lanes), and takes
// the list in groups of kGroup. Per group, a back-to-front sweep reads every
// layer once, carries S (FP64) and keeps a_i and D_i = <G, S_{i+1}> in
// registers; a front-to-back sweep then forms T (FP64) from the kept a_i and
// writes the gradients. Nothing per layer goes to memory. The groups run back
// to front, so S carries over; the transmittance in front of each group (a
// checkpoint) comes from a first pass over the alpha of the groups in front
// of the back one, front to back.
// What bounds it: memory. Where every layer covers every pixel, half of the
// bytes are writes (32 FP32 layers of 1024x1024, 1.09 GB: 188 us, 5.8 TB/s,
// where a copy reaches 5.0). Two waves per SIMD, which a_i and D_i in registers
// leave, are enough for it (D_i in LDS and four waves: 191 us). The groups are
// of the layers that a row segment meets, not of list positions: of 80 partial
// FP16 layers it meets about 20, and positions took three groups and two
// readings of most alphas (961x541: 270 us and one zeroing launch per layer
// that reaches out of the view, 430 us in all; now 77).
constexpr int kGroup = 32;
constexpr int kBwdInline = 64;                        // descriptors in the kernel arguments
constexpr int kBwdMaxLayers = 256;                    // with a descriptor workspace
constexpr int kBwdCkpt = kBwdMaxLayers / kGroup - 1;  // checkpoints of the general kernel

struct BwdDesc {
  const void* color;
  void* grad;
  int64_t pitch;
  int64_t gpitch;
  int32_t x, y, w, h;
};

struct BwdArgs {
  BwdDesc c[kBwdInline];   // back to front (n <= kBwdInline)
  const BwdDesc* desc;     // device copy, back to front (n > kBwdInline)
  const float* gout;
  int64_t gout_pitch;
  int32_t vx, vy, vw, vh;
  int32_t n;
  int32_t tile_w, tile_h, tiles_x;
};
static_assert(sizeof(BwdArgs) <= 4096, "kernel arguments must fit in 4 KiB");

// A listed layer: the segment's first pixel in it and in its gradient, and
// its covered lanes (OverSeg).
struct BwdSeg {
  uint32_t lo, hi, span, glo, ghi;
};

typedef const __attribute__((address_space(1))) char* GlobalBytes;
__device__ __forceinline__ uint32_t lane_of(uint32_t v, int i) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, i);
}
__device__ __forceinline__ GlobalBytes lane_address(uint32_t lo, uint32_t hi, int i) {
  return (GlobalBytes)(((uint64_t)lane_of(hi, i) << 32) | lane_of(lo, i));
}

// FP32 to FP16. Without the pragma the FP64 value behind v is rounded to FP16
// at once, which is not the FP32 gradient rounded where that one is a tie.
__device__ __forceinline__ f16x4 narrow(f32x4 v) {
#pragma clang fp contract(off)
  return f16x4{(_Float16)v.x, (_Float16)v.y, (_Float16)v.z, (_Float16)v.w};
}

// T <- T * prod (1 - a_j) over the m layers of a group, front to back.
template <int FMT>
__device__ __forceinline__ double bwd_alpha_product(const BwdSeg& sg, int m, int lane, double T) {
  constexpr uint32_t bpp = FMT == CMP_RGBA32F ? 16 : 8;
  for (int i1 = m; i1 > 0; i1 -= kOverBatch) {   // uniform
    float al[kOverBatch];
    bool cov[kOverBatch];
#pragma unroll
    for (int k = 0; k < kOverBatch; ++k) {
      const int i = max(i1 - 1 - k, 0);
      const uint32_t span = lane_of(sg.span, i), c0 = span & 0xFFu;
      cov[k] = i1 - 1 - k >= 0 && (uint32_t)lane - c0 < (span >> 8);
      const GlobalBytes p =
          lane_address(sg.lo, sg.hi, i) + (cov[k] ? (uint32_t)lane : c0) * bpp + bpp / 4 * 3;
      if constexpr (FMT == CMP_RGBA32F)
        al[k] = *(const __attribute__((address_space(1))) float*)p;
      else
        al[k] = (float)*(const __attribute__((address_space(1))) _Float16*)p;
    }
#pragma unroll
    for (int k = 0; k < kOverBatch; ++k)
      if (cov[k]) T = T * (1.0 - (double)al[k]);
  }
  return T;
}

// One group: the m layers of lanes 0 .. m - 1 of sg, back to front. S (in and
// out) is the composite of everything behind the group; T is the
// transmittance in front of it. GFMT: the format of the gradients, rounded
// once more from FP32 if it is FP16.
template <int FMT, int GFMT>
__device__ __forceinline__ void bwd_group(const BwdSeg& sg, int m, int lane, const f32x4 G,
                                          double (&S)[4], double T) {
  constexpr uint32_t bpp = FMT == CMP_RGBA32F ? 16 : 8, gbpp = GFMT == CMP_RGBA32F ? 16 : 8;
  typedef typename RawPx<FMT>::type Raw;
  typedef const __attribute__((address_space(1))) Raw* GPtr;
  const double g0 = G.x, g1 = G.y, g2 = G.z, g3 = G.w;
  float al[kGroup], dd[kGroup];   // alpha 0 leaves T unchanged
#pragma unroll
  for (int b = 0; b < kGroup; b += kOverBatch) {
    if (b >= m) break;   // uniform
    Raw L[kOverBatch];
    bool cov[kOverBatch];
#pragma unroll
    for (int k = 0; k < kOverBatch; ++k) {
      const int i = b + k < m ? b + k : b;
      const uint32_t span = lane_of(sg.span, i), c0 = span & 0xFFu;
      cov[k] = b + k < m && (uint32_t)lane - c0 < (span >> 8);
      const uint32_t off = (cov[k] ? (uint32_t)lane : c0) * bpp;
      L[k] = __builtin_nontemporal_load((GPtr)(lane_address(sg.lo, sg.hi, i) + off));
    }
#pragma unroll
    for (int k = 0; k < kOverBatch; ++k) {
      al[b + k] = dd[b + k] = 0.f;
      if (cov[k]) {
        const f32x4 v = widen(L[k]);
        dd[b + k] = (float)(g0 * S[0] + g1 * S[1] + g2 * S[2] + g3 * S[3]);
        al[b + k] = v.w;
        const double t = 1.0 - (double)v.w;
        S[0] = (double)v.x + t * S[0];
        S[1] = (double)v.y + t * S[1];
        S[2] = (double)v.z + t * S[2];
        S[3] = (double)v.w + t * S[3];
      }
    }
  }
#pragma unroll
  for (int i = kGroup - 1; i >= 0; --i) {
    if (i >= m) continue;   // uniform: front to back
    const uint32_t span = lane_of(sg.span, i);
    if ((uint32_t)lane - (span & 0xFFu) < (span >> 8)) {
      f32x4 g;
      g.x = (float)(g0 * T);
      g.y = (float)(g1 * T);
      g.z = (float)(g2 * T);
      g.w = (float)(g3 * T - T * (double)dd[i]);
      // a global-address-space store cannot alias the kernel-argument copy
      const GlobalBytes p = lane_address(sg.glo, sg.ghi, i) + (uint32_t)lane * gbpp;
      if constexpr (GFMT == CMP_RGBA32F)
        __builtin_nontemporal_store(g, (__attribute__((address_space(1))) f32x4*)p);
      else
        __builtin_nontemporal_store(narrow(g), (__attribute__((address_space(1))) f16x4*)p);
      T = T * (1.0 - (double)al[i]);
    }
  }
}

// kInline: n <= kBwdInline, descriptors in the arguments, at most two groups
// (the back group's checkpoint stays in a register); otherwise descriptors
// from the workspace and up to kBwdCkpt checkpoints in LDS.
// Tile order: an XCD takes runs of consecutive tiles, so that the cache lines
// which neighbouring tiles share where rows are no multiple of 128 bytes are
// read and written by one L2 (30 layers of 1023x1025: 235 us in launch order,
// 218 in runs of 16, 206 in runs of 256), and the workgroups in flight do not
// all meet in the same memory channels where they are (32 of 1024x1024: 199,
// 198, 188). Below 4096 tiles runs of 256 leave the XCDs unequal shares (80
// partial layers over 961x541, 2176 tiles: 77 us in runs of 16, 89 in runs of
// 256).
template <int FMT, int GFMT, bool kInline>
__global__ __launch_bounds__(kThreads) void over_bwd_kernel(const BwdArgs a) {
  constexpr int kList = kInline ? kBwdInline : kBwdMaxLayers;
  __shared__ uint32_t s_list[kThreads / kWave][5][kList];
  __shared__ double tck[kInline ? 1 : kBwdCkpt][kThreads];
  const BwdDesc* d = kInline ? a.c : a.desc;
  const int blk = xcd_tile((int)blockIdx.x, (int)gridDim.x, gridDim.x >= 4096 ? 256 : 16);
  const int ty = blk / a.tiles_x, tx = blk - ty * a.tiles_x;
  const int x0 = a.vx + tx * a.tile_w, y0 = a.vy + ty * a.tile_h;
  const int tw = min(a.tile_w, a.vx + a.vw - x0), th = min(a.tile_h, a.vy + a.vh - y0);
  const int lane = threadIdx.x % kWave;
  uint32_t(*list)[kList] = s_list[uniform((int)(threadIdx.x / kWave))];
  over_segments(x0, y0, tw, th, [&](int Y, int X0, int cols) {
    f32x4 G{0.f, 0.f, 0.f, 0.f};
    if (lane < cols)
      G = reinterpret_cast<const f32x4*>(
          a.gout)[(int64_t)(Y - a.vy) * a.gout_pitch + (X0 + lane - a.vx)];
    // the layers that reach the segment, back to front
    int cnt = 0;
    for (int c0 = 0; c0 < a.n; c0 += kWave) {
      BwdDesc D{nullptr, nullptr, 0, 0, 0, 0, 0, 0};
      if (c0 + lane < a.n) D = d[c0 + lane];
      uint64_t hits;
      const OverSeg s =
          over_segment<FMT>(OverDesc{D.color, D.pitch, D.x, D.y, D.w, D.h}, X0, cols, Y, hits);
      const uint64_t ga = over_address<GFMT>(D.grad, D.gpitch, D.x, D.y, X0, Y);
      if ((hits >> lane) & 1u) {
        const int at = cnt + (int)__builtin_popcountll(hits & ((1ull << lane) - 1ull));
        list[0][at] = s.lo;
        list[1][at] = s.hi;
        list[2][at] = s.span;
        list[3][at] = (uint32_t)ga;
        list[4][at] = (uint32_t)(ga >> 32);
      }
      cnt += (int)__builtin_popcountll(hits);
    }
    wave_lds_fence();   // a wave reads its own list only
    const int groups = (cnt + kGroup - 1) / kGroup;
    auto group_layers = [&](int g) {
      const int i = g * kGroup + (lane % kGroup), j = i < cnt ? i : 0;
      return BwdSeg{list[0][j], list[1][j], list[2][j], list[3][j], list[4][j]};
    };
    // checkpoints: the transmittance in front of groups `groups` - 2 .. 0
    double T1 = 1.0;
    {
      double T = 1.0;
      for (int g = groups - 1; g >= 1; --g) {
        T = bwd_alpha_product<FMT>(group_layers(g), min(kGroup, cnt - g * kGroup), lane, T);
        if (kInline) T1 = T;
        else tck[g - 1][threadIdx.x] = T;
      }
    }
    double S[4] = {0.0, 0.0, 0.0, 0.0};
    for (int g = 0; g < groups; ++g) {
      const double T = g == groups - 1 ? 1.0 : kInline ? T1 : tck[g][threadIdx.x];
      bwd_group<FMT, GFMT>(group_layers(g), min(kGroup, cnt - g * kGroup), lane, G, S, T);
    }
    wave_lds_fence();   // the list is read
  });
}

// Copies up to kBwdInline descriptors from the arguments to device memory
// (the workspace of a backward pass with more layers): a kernel rather than
// a host copy, so that a captured graph carries the descriptors with it.
struct BwdDescCopy {
  BwdDesc c[kBwdInline];
  BwdDesc* dst;
  int32_t n;
};
static_assert(sizeof(BwdDescCopy) <= 4096, "kernel arguments must fit in 4 KiB");

__global__ __launch_bounds__(kThreads) void bwd_desc_kernel(const BwdDescCopy a) {
  for (int i = threadIdx.x; i < a.n; i += kThreads) a.dst[i] = a.c[i];
}

// Zeroes the parts of layer gradients that the viewport does not reach, of up
// to kBwdInline layers per launch (one launch per layer, over all of it, took
// most of the host's time where many layers reach out of the view).
struct ZeroLayer {
  void* p;
  int64_t pitch;
  int32_t w, h;
  int32_t ix0, iy0, ix1, iy1;   // the part inside the viewport, left alone
};
struct ZeroArgs {
  ZeroLayer l[kBwdInline];
};
static_assert(sizeof(ZeroArgs) <= 4096, "kernel arguments must fit in 4 KiB");

// A wave takes a row at a time; Px: one pixel of the gradient.
template <typename Px>
__global__ __launch_bounds__(kThreads) void zero_outside_kernel(const ZeroArgs a) {
  const ZeroLayer& L = a.l[blockIdx.y];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  for (int y = (int)blockIdx.x * (kThreads / kWave) + wave; y < L.h;
       y += (int)gridDim.x * (kThreads / kWave)) {
    Px* row = reinterpret_cast<Px*>(L.p) + (int64_t)y * L.pitch;
    const bool in = y >= L.iy0 && y < L.iy1;
    const int end0 = in ? L.ix0 : L.w, begin1 = in ? L.ix1 : L.w;
    for (int x = lane; x < end0; x += kWave) row[x] = Px{};
    for (int x = begin1 + lane; x < L.w; x += kWave) row[x] = Px{};
  }
}

cmp_status validate_over_inputs(const cmp_image* in, int32_t n, cmp_format fmt,
                                const int32_t* order) {
  CMP_REQUIRE(n >= 0, "n = %d is negative", n);
  CMP_REQUIRE(n == 0 || (in && order), "in or order_b2f is NULL");
  CMP_REQUIRE(fmt == CMP_RGBA32F || fmt == CMP_RGBA16F, "format %d is not a float format", fmt);
  const uintptr_t align = fmt == CMP_RGBA32F ? 16 : 8;
  for (int i = 0; i < n; ++i) {
    const cmp_image& I = in[i];
    CMP_REQUIRE(rect_valid(I.roi), "in[%d].roi has a negative size", i);
    if (rect_empty(I.roi)) continue;
    CMP_REQUIRE(I.color, "in[%d].color is NULL", i);
    CMP_REQUIRE(I.pitch >= I.roi.w, "in[%d].pitch < roi.w", i);
    CMP_REQUIRE(((uintptr_t)I.color % align) == 0, "in[%d].color must be %d-byte aligned", i,
                (int)align);
  }
  // order must be a permutation
  if (n > 0) {
    uint8_t* seen = (uint8_t*)calloc((size_t)n, 1);
    if (!seen) return CMP_EINVAL;
    bool ok = true;
    for (int j = 0; j < n && ok; ++j) {
      const int v = order[j];
      if (v < 0 || v >= n || seen[v]) ok = false;
      else seen[v] = 1;
    }
    free(seen);
    CMP_REQUIRE(ok, "order_b2f is not a permutation of 0..%d", n - 1);
  }
  return CMP_OK;
}

}  // namespace cmp

using namespace cmp;

extern "C" cmp_status cmp_composite_over(const cmp_image* in, int32_t n, cmp_format fmt,
                                         const int32_t* order_b2f, cmp_rect viewport,
                                         float* out_rgba, int64_t out_pitch, cmp_schedule sched,
                                         cmp_tile tile, void* stream) {
  CMP_RANGE("cmp_composite_over");
  cmp_status st = validate_over_inputs(in, n, fmt, order_b2f);
  if (st != CMP_OK) return st;
  CMP_REQUIRE(rect_valid(viewport), "viewport has a negative size");
  if (rect_empty(viewport)) return CMP_OK;
  CMP_REQUIRE(out_rgba && ((uintptr_t)out_rgba & 15) == 0, "out_rgba must be 16-byte aligned");
  CMP_REQUIRE(out_pitch >= viewport.w, "out_pitch < viewport.w");
  int tw = tile.w ? tile.w : 64, th = tile.h ? tile.h : 4;
  CMP_REQUIRE(tw > 0 && th > 0 && (int64_t)tw * th <= 65536, "bad tile %dx%d", tw, th);
  const bool tree = sched.kind == CMP_SCHED_BINARY_SWAP;
  if (tree && n > kOverPerPass) {
    set_error("binary-swap order supports at most %d layers", kOverPerPass);
    return CMP_EUNSUPPORTED;
  }

  OverArgs a;
  memset(&a, 0, sizeof a);
  int64_t tiles = 0;
  int nreg = plan_regions(sched, viewport, tw, th, a.reg, &tiles);
  if (nreg < 0) return nreg;
  constexpr int64_t kTooMany = 1ll << 24;
  CMP_REQUIRE(tiles < kTooMany, "too many tiles");
  // The requested tile decides what is refused. The one it is run as can be
  // more of them (16x16 over a view 16 pixels wide: four times as many); it is
  // then made as much higher as the limit asks for, at most to the requested
  // height, where it is never more.
  const int rw = tw, rh = th;
  over_tile_shape(tw, th);
  if (tw != rw || th != rh) {
    while ((nreg = plan_regions(sched, viewport, tw, th, a.reg, &tiles)) >= 0 && tiles >= kTooMany)
      th = std::min(2 * th, rh);
    if (nreg < 0) return nreg;
  }
  a.out = out_rgba;
  a.out_pitch = out_pitch;
  a.vx = viewport.x;
  a.vy = viewport.y;
  a.nreg = nreg;
  a.tile_w = tw;
  a.tile_h = th;
  hipStream_t s = (hipStream_t)stream;
  auto launch = [&]() -> cmp_status {
    const dim3 grid((unsigned)tiles), block(kThreads);
    if (a.groups > 0) {
      int levels = 0;
      while ((1 << levels) < a.groups) ++levels;
      const unsigned lds = (unsigned)(levels * kThreads * sizeof(f32x4));
      if (fmt == CMP_RGBA32F)
        hipLaunchKernelGGL(over_tree_kernel<CMP_RGBA32F>, grid, block, lds, s, a);
      else
        hipLaunchKernelGGL(over_tree_kernel<CMP_RGBA16F>, grid, block, lds, s, a);
    } else {
      if (fmt == CMP_RGBA32F)
        hipLaunchKernelGGL(over_kernel<CMP_RGBA32F>, grid, block, 0, s, a);
      else
        hipLaunchKernelGGL(over_kernel<CMP_RGBA16F>, grid, block, 0, s, a);
    }
    CMP_CHECK_HIP(hipGetLastError());
    return CMP_OK;
  };
  if (tree) {
    const int P = sched.owners;
    for (int j = 0; j < n; ++j) {
      const cmp_image& I = in[order_b2f[j]];
      a.c[j] = OverDesc{I.color, I.pitch, I.roi.x, I.roi.y, rect_empty(I.roi) ? 0 : I.roi.w,
                        rect_empty(I.roi) ? 0 : I.roi.h};
    }
    a.n = n;
    a.groups = P;
    return launch();
  }
  int base = 0;
  do {
    const int cnt = n - base < kOverPerPass ? n - base : kOverPerPass;
    for (int j = 0; j < cnt; ++j) {
      const cmp_image& I = in[order_b2f[base + j]];
      a.c[j] = OverDesc{I.color, I.pitch, I.roi.x, I.roi.y, rect_empty(I.roi) ? 0 : I.roi.w,
                        rect_empty(I.roi) ? 0 : I.roi.h};
    }
    a.n = cnt;
    a.accumulate = base > 0;
    st = launch();
    if (st != CMP_OK) return st;
    base += cnt;
  } while (base < n);
  return CMP_OK;
}

extern "C" size_t cmp_over_backward_workspace_size(int32_t n) {
  return n > kBwdInline && n <= kBwdMaxLayers ? (size_t)n * sizeof(BwdDesc) : 0;
}

static cmp_status over_backward_impl(const cmp_image* in, int32_t n, cmp_format fmt,
                                     const int32_t* order_b2f, cmp_rect viewport,
                                     const float* grad_out, int64_t grad_pitch,
                                     void* const* grad_layers, cmp_format grad_fmt,
                                     const int64_t* grad_pitch_layers, void* workspace,
                                     size_t ws_bytes, void* stream) {
  cmp_status st = validate_over_inputs(in, n, fmt, order_b2f);
  if (st != CMP_OK) return st;
  CMP_REQUIRE(grad_fmt == CMP_RGBA32F || grad_fmt == CMP_RGBA16F,
              "gradient format %d is not a float format", grad_fmt);
  const int galign = grad_fmt == CMP_RGBA32F ? 16 : 8;
  if (n > kBwdMaxLayers) {
    set_error("the backward pass supports at most %d layers", kBwdMaxLayers);
    return CMP_EUNSUPPORTED;
  }
  if (n > kBwdInline) {
    CMP_REQUIRE(workspace && ((uintptr_t)workspace & 15) == 0,
                "n = %d > %d layers needs a 16-byte aligned workspace", n, kBwdInline);
    if (ws_bytes < cmp_over_backward_workspace_size(n)) {
      set_error("workspace of %zu bytes is smaller than %zu", ws_bytes,
                cmp_over_backward_workspace_size(n));
      return CMP_ENOSPC;
    }
  }
  CMP_REQUIRE(rect_valid(viewport), "viewport has a negative size");
  CMP_REQUIRE(n == 0 || (grad_layers && grad_pitch_layers), "grad_layers is NULL");
  for (int i = 0; i < n; ++i) {
    if (rect_empty(in[i].roi)) continue;
    CMP_REQUIRE(grad_layers[i] && ((uintptr_t)grad_layers[i] % (uintptr_t)galign) == 0,
                "grad_layers[%d] must be %d-byte aligned", i, galign);
    CMP_REQUIRE(grad_pitch_layers[i] >= in[i].roi.w, "grad_pitch_layers[%d] < roi.w", i);
  }
  const bool work = !rect_empty(viewport) && n > 0;
  if (work) {
    CMP_REQUIRE(grad_out && ((uintptr_t)grad_out & 15) == 0, "grad_out must be 16-byte aligned");
    CMP_REQUIRE(grad_pitch >= viewport.w, "grad_pitch < viewport.w");
  }
  const int tile_w = 64, tile_h = 4;
  const int64_t tiles_x = (viewport.w + tile_w - 1) / tile_w;
  const int64_t tiles = tiles_x * ((viewport.h + tile_h - 1) / tile_h);
  CMP_REQUIRE(!work || tiles < (1ll << 24), "too many tiles");
  hipStream_t s = (hipStream_t)stream;
  // zero the parts of the layer gradients that the viewport does not reach
  ZeroArgs z;
  int nz = 0, rows = 0;
  auto zero = [&]() -> cmp_status {
    const unsigned bx = (unsigned)std::min(64, (rows + kThreads / kWave - 1) / (kThreads / kWave));
    if (grad_fmt == CMP_RGBA32F)
      hipLaunchKernelGGL(zero_outside_kernel<f32x4>, dim3(bx, nz), dim3(kThreads), 0, s, z);
    else
      hipLaunchKernelGGL(zero_outside_kernel<f16x4>, dim3(bx, nz), dim3(kThreads), 0, s, z);
    nz = rows = 0;
    CMP_CHECK_HIP(hipGetLastError());
    return CMP_OK;
  };
  for (int i = 0; i < n; ++i) {
    const cmp_rect r = in[i].roi;
    if (rect_empty(r)) continue;
    auto cut = [](int64_t v, int64_t lo, int64_t hi) { return (int32_t)std::max(lo, std::min(v, hi)); };
    ZeroLayer L{grad_layers[i], grad_pitch_layers[i], r.w, r.h, 0, 0, 0, 0};
    if (!rect_empty(viewport)) {
      L.ix0 = cut((int64_t)viewport.x - r.x, 0, r.w);
      L.iy0 = cut((int64_t)viewport.y - r.y, 0, r.h);
      L.ix1 = cut((int64_t)viewport.x + viewport.w - r.x, 0, r.w);
      L.iy1 = cut((int64_t)viewport.y + viewport.h - r.y, 0, r.h);
    }
    if (L.ix0 == 0 && L.iy0 == 0 && L.ix1 == r.w && L.iy1 == r.h) continue;
    if (L.ix1 <= L.ix0 || L.iy1 <= L.iy0) L.ix0 = L.iy0 = L.ix1 = L.iy1 = 0;
    z.l[nz++] = L;
    rows = std::max(rows, r.h);
    if (nz == kBwdInline && (st = zero()) != CMP_OK) return st;
  }
  if (nz && (st = zero()) != CMP_OK) return st;
  if (!work) return CMP_OK;

  BwdArgs a;
  memset(&a, 0, sizeof a);
  auto desc = [&](int j) {
    const int li = order_b2f[j];
    const cmp_image& I = in[li];
    return BwdDesc{I.color, grad_layers[li], I.pitch, grad_pitch_layers[li], I.roi.x, I.roi.y,
                   rect_empty(I.roi) ? 0 : I.roi.w, rect_empty(I.roi) ? 0 : I.roi.h};
  };
  if (n <= kBwdInline) {
    for (int j = 0; j < n; ++j) a.c[j] = desc(j);
  } else {
    // the descriptors go to the workspace, kBwdInline per copy kernel
    BwdDesc* dst = (BwdDesc*)workspace;
    for (int j0 = 0; j0 < n; j0 += kBwdInline) {
      BwdDescCopy cp;
      memset(&cp, 0, sizeof cp);
      cp.n = n - j0 < kBwdInline ? n - j0 : kBwdInline;
      for (int j = 0; j < cp.n; ++j) cp.c[j] = desc(j0 + j);
      cp.dst = dst + j0;
      hipLaunchKernelGGL(bwd_desc_kernel, dim3(1), dim3(kThreads), 0, s, cp);
      CMP_CHECK_HIP(hipGetLastError());
    }
    a.desc = dst;
  }
  a.gout = grad_out;
  a.gout_pitch = grad_pitch;
  a.vx = viewport.x;
  a.vy = viewport.y;
  a.vw = viewport.w;
  a.vh = viewport.h;
  a.n = n;
  a.tile_w = tile_w;
  a.tile_h = tile_h;
  a.tiles_x = (int32_t)tiles_x;
  const dim3 grid((unsigned)tiles), block(kThreads);
  const bool f32 = fmt == CMP_RGBA32F, g32 = grad_fmt == CMP_RGBA32F;
#define CMP_BWD_LAUNCH(F, GF)                                                             \
  do {                                                                                    \
    if (n <= kBwdInline)                                                                  \
      hipLaunchKernelGGL((over_bwd_kernel<F, GF, true>), grid, block, 0, s, a);           \
    else                                                                                  \
      hipLaunchKernelGGL((over_bwd_kernel<F, GF, false>), grid, block, 0, s, a);          \
  } while (0)
  if (f32 && g32) CMP_BWD_LAUNCH(CMP_RGBA32F, CMP_RGBA32F);
  else if (f32) CMP_BWD_LAUNCH(CMP_RGBA32F, CMP_RGBA16F);
  else if (g32) CMP_BWD_LAUNCH(CMP_RGBA16F, CMP_RGBA32F);
  else CMP_BWD_LAUNCH(CMP_RGBA16F, CMP_RGBA16F);
#undef CMP_BWD_LAUNCH
  CMP_CHECK_HIP(hipGetLastError());
  return CMP_OK;
}

extern "C" cmp_status cmp_composite_over_backward(const cmp_image* in, int32_t n, cmp_format fmt,
                                                  const int32_t* order_b2f, cmp_rect viewport,
                                                  const float* grad_out, int64_t grad_pitch,
                                                  float* const* grad_layers,
                                                  const int64_t* grad_pitch_layers, void* workspace,
                                                  size_t ws_bytes, void* stream) {
  CMP_RANGE("cmp_composite_over_backward");
  return over_backward_impl(in, n, fmt, order_b2f, viewport, grad_out, grad_pitch,
                            (void* const*)grad_layers, CMP_RGBA32F, grad_pitch_layers, workspace,
                            ws_bytes, stream);
}

extern "C" cmp_status cmp_composite_over_backward_as(const cmp_image* in, int32_t n,
                                                     cmp_format fmt, const int32_t* order_b2f,
                                                     cmp_rect viewport, const float* grad_out,
                                                     int64_t grad_pitch, void* const* grad_layers,
                                                     cmp_format grad_fmt,
                                                     const int64_t* grad_pitch_layers,
                                                     void* workspace, size_t ws_bytes,
                                                     void* stream) {
  CMP_RANGE("cmp_composite_over_backward_as");
  return over_backward_impl(in, n, fmt, order_b2f, viewport, grad_out, grad_pitch, grad_layers,
                            grad_fmt, grad_pitch_layers, workspace, ws_bytes, stream);
}
