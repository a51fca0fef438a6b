// Parts shared by the run-length codecs (the per-component RLE1 codec and
// the basic 64-bit RL64 codec of Section 5.5.1, Enhanced RLE Compression):
// block geometry, the slot tickets and decoupled look-back of the
// single-pass compressors, the pixel loads of a block, and wave / workgroup
// scans. Streams of both codecs share one layout (header, block offsets,
// per-block sizes, 16-byte aligned payloads).
#pragma once

#include <atomic>

#include "cmp_internal.hpp"

namespace cmp {

constexpr uint32_t kRleMagic = 0x31454C52u;
constexpr int kBlock = 4096;
constexpr int kSeg = 256;
constexpr int kPxPerLane = 16;
constexpr int kRleMax = 64;
constexpr int kStage = 8 * kBlock + 16;

__host__ __device__ inline int64_t imin64(int64_t a, int64_t b) { return a < b ? a : b; }
__host__ __device__ inline uint64_t align16(uint64_t v) { return (v + 15u) & ~(uint64_t)15u; }
__host__ __device__ inline uint64_t rle_nblocks(int64_t npx) {
  return (uint64_t)((npx + kBlock - 1) / kBlock);
}
__host__ __device__ inline uint64_t rle_p0(uint64_t nb, int np) {
  return align16(32 + 4 * nb * (1 + (uint64_t)np));
}

// ------------------------------------------------------------- helpers
// Bit swizzling (Section 5.5.1): bit 2j+b of component c moves to bit
// 8j + 2c + b, i.e. the 4x4 matrix of 2-bit fields (component, significance
// group) is transposed. Two delta swaps do the transpose: the off-diagonal
// 2x2 blocks, then the off-diagonal fields inside each block. A transpose is
// its own inverse, so the same function undoes it.
__device__ __forceinline__ uint32_t swizzle_bits(uint32_t x) {
  uint32_t t = ((x >> 12) ^ x) & 0x0000F0F0u;
  x ^= t ^ (t << 12);
  t = ((x >> 6) ^ x) & 0x00CC00CCu;
  x ^= t ^ (t << 6);
  return x;
}

// ------------------------------------------------------------ compress
struct RleCImg {
  const uint32_t* color;
  const uint32_t* depth;   // nullptr: 4 planes
  int64_t pitch;
  int32_t W, H;            // image size
  uint8_t* out;
  int32_t flag_base;       // first look-back flag of this image
  int32_t pad;
};

struct RleCArgs {
  RleCImg im[kRleMax];
  const int32_t* roi_dev;
  uint64_t* out_size;
  int32_t* status;
  uint32_t* tickets;       // workspace: a ticket counter per image, kTicketStride words apart
  uint32_t* ctl;           // workspace: the call epoch (word 0), finished workgroups (word
                           // kCtlDone), the most flags any call has used (word kCtlHwm)
  uint64_t* flags;         // workspace: one flag per (image, block)
  int32_t nflags;          // flags of this call
  int32_t n;
  int32_t swizzle;         // CMP_RLE_SWIZZLE
  uint32_t wait_limit;     // look-back polls before a block gives up
};
static_assert(sizeof(RleCArgs) <= 4096, "kernel arguments must fit in 4 KiB");

// Workspace: the ticket counters (one per image, each on its own 128-byte
// line, beside a count of finished workgroups), control words (the call epoch
// on one line; the count of finished workgroups and the most flags any call
// has used on another), then the look-back flags. It is zero-filled once, before its first use; every call
// leaves it ready for the next: the last workgroup to finish zeroes the
// tickets and the count and advances the epoch, and a flag written by an
// earlier call (another epoch) reads as not ready, so the flags are not
// cleared, except when the 30-bit epoch wraps to 0: then the flags that
// calls have used so far are zeroed, since those of the calls 2^30 earlier
// would read as current again.
constexpr int kTicketStride = 32;
constexpr size_t kTicketBytes = (size_t)kRleMax * kTicketStride * 4;
constexpr int kCtlDone = 32;   // word index of the finished-workgroup count
constexpr int kCtlHwm = 33;    // word index of the most flags any call has used
constexpr size_t kCtlBytes = 256;
constexpr uint32_t kDoneGroups = 32;   // counts of finished workgroups at word 1 of ticket lines
static_assert(kDoneGroups <= kRleMax, "one ticket line per group");
constexpr uint32_t kEpochMask = (1u << 30) - 1;

// look-back flag: epoch (30 bits) << 34 | status (2 bits) << 32 | value (32
// bits); status 0, or another call's epoch, = not ready. kPoison marks a
// block whose offset is unknown (a bounded wait gave up): neither it nor
// any later block of the image writes its payload.
constexpr uint64_t kAgg = 1, kIncl = 2, kPoison = 3;
constexpr int kLookback = 4;   // flags per lane per look-back step
__device__ __forceinline__ uint64_t mkflag(uint64_t st, uint32_t v, uint32_t ep) {
  return ((uint64_t)ep << 34) | (st << 32) | v;
}
__device__ __forceinline__ uint64_t flag_state(uint64_t f, uint32_t ep) {
  return (uint32_t)(f >> 34) == ep ? (f >> 32) & 3u : 0u;
}

// The epoch of this call (every workgroup reads it at its start; only the
// previous call's last workgroup wrote it). Loaded into a vector register
// and first used at the block's flag, so that the load's latency passes
// while the pixels arrive (made uniform there, it held up the first ticket
// draw).
__device__ __forceinline__ uint32_t call_epoch(const RleCArgs& a) {
  return __hip_atomic_load(a.ctl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kEpochMask;
}

// Every workgroup ends here, after its last use of the tickets and flags:
// the last one to arrive zeroes the tickets of this call's images and the
// counts, raises the flag high-water mark to this call's flags, and advances
// the epoch, ready for the next call on the workspace; if the epoch wraps to
// 0 it first zeroes the flags below the high-water mark.
// Relaxed atomics suffice: every ticket access is a device-scope atomic, and
// a workgroup's last draw has returned before its count is added; the next
// call reads the epoch after this kernel has ended. (An acquire-release
// count, which writes back the L2 at each workgroup's exit, made a 16 x
// 1920x1080 compression 40% slower.)
// One counter takes 11 ns per workgroup, which is the end of the call where
// the workgroups have at most two slots each (`slots`: of the call) and end
// together: they are then counted in kDoneGroups groups, and each group's last
// one counts for it (24 images of 1279x719, 944 slots for 1024 workgroups:
// 23.1 -> 19.2 us, 6 of 1000x700: 21.0 -> 14.6, RL64 of 3 of 1268x997: 17.8 ->
// 12.1, of 8 of 1920x1080, 1215 slots: 27.3 -> 24.8). With more slots, or few
// workgroups, the second round trip costs more than the queue (RL64 of 16 of
// 2100x1500: 56.0, 56.8 in groups; one image of 400x300: 12.1, 12.5).
__device__ __forceinline__ void finish_call(const RleCArgs& a, uint32_t ep, uint32_t slots) {
  __shared__ int s_last;
  __syncthreads();
  if (threadIdx.x == 0) {
    auto arrive = [](uint32_t* c, uint32_t of) {
      return __hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == of - 1;
    };
    if (slots >= 2 * gridDim.x || gridDim.x <= 2 * kDoneGroups) {
      s_last = arrive(a.ctl + kCtlDone, gridDim.x);
    } else {
      const uint32_t g = blockIdx.x % kDoneGroups;
      s_last = arrive(a.tickets + g * kTicketStride + 1,
                      (gridDim.x - g + kDoneGroups - 1) / kDoneGroups) &&
               arrive(a.ctl + kCtlDone, kDoneGroups);
    }
  }
  __syncthreads();
  if (s_last) {
    for (int i = threadIdx.x; i < kRleMax; i += kThreads) {
      __hip_atomic_store(a.tickets + i * kTicketStride, 0u, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(a.tickets + i * kTicketStride + 1, 0u, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
    const uint32_t hwm =
        max(__hip_atomic_load(a.ctl + kCtlHwm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
            (uint32_t)a.nflags);
    const uint32_t next = (ep + 1) & kEpochMask;
    if (next == 0) {
      for (uint32_t i = threadIdx.x; i < hwm; i += kThreads)
        __hip_atomic_store(a.flags + i, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();   // every thread has read the high-water mark
    if (threadIdx.x == 0) {
      __hip_atomic_store(a.ctl + kCtlHwm, hwm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(a.ctl + kCtlDone, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(a.ctl, next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}


// DPP row shift left by D lanes inside rows of 16 lanes (lane r reads lane
// r + D); lanes whose source lies outside the row keep `fill`.
template <int D>
__device__ __forceinline__ int row_shl_fill(int v, int fill) {
  return __builtin_amdgcn_update_dpp(fill, v, 0x100 + D, 0xF, 0xF, false);
}

// Inclusive scan over the 64 lanes: DPP inside rows of 16, then the row
// totals of the lower rows (read lane by lane).
__device__ __forceinline__ uint32_t wave_incl_scan32(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 15);
  const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)v, 31);
  const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)v, 47);
  const int row = (threadIdx.x % kWave) >> 4;
  return v + (row >= 1 ? r0 : 0u) + (row >= 2 ? r1 : 0u) + (row >= 3 ? r2 : 0u);
}

// Exclusive workgroup scan of kW 32-bit words of packed counters that cannot
// overflow; also returns the totals (uniform). `sh` holds 4 * kW words; one barrier: the
// caller keeps another between these reads of `sh` and its next writes.
template <int kW>
__device__ __forceinline__ void block_scan32_once(const uint32_t (&v)[kW], uint32_t (&ex)[kW],
                                             uint32_t (&tot)[kW], uint32_t* sh) {
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  uint32_t inc[kW];
#pragma unroll
  for (int i = 0; i < kW; ++i) {
    inc[i] = wave_incl_scan32(v[i]);
    if (lane == kWave - 1) sh[4 * i + wave] = inc[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kW; ++i) {
    uint32_t p = 0, t = 0;
#pragma unroll
    for (int w = 0; w < kThreads / kWave; ++w) {
      const uint32_t x = sh[4 * i + w];
      if (w < wave) p += x;
      t += x;
    }
    ex[i] = p + inc[i] - v[i];
    tot[i] = (uint32_t)uniform((int)t);
  }
}

// One compression slot: image s, block b, and the image's clamped ROI.
struct CSlot {
  int s, b, rx, ry, rw, rh;
};

__device__ __forceinline__ CSlot compress_slot(int2 sb, const int4* t_roi) {
  CSlot c;
  c.s = uniform(sb.x);
  c.b = uniform(sb.y);
  const int4 r = t_roi[c.s];
  c.rx = uniform(r.x);
  c.ry = uniform(r.y);
  c.rw = uniform(r.z);
  c.rh = uniform(r.w);
  return c;
}

// How a compression's workgroups share its slots: ticket t of image s is
// block t of s, drawn from the image's counter, so the blocks of an image are
// handed out in order, and only to running workgroups: every block that a
// look-back waits for belongs to a workgroup that runs, and no launch order,
// grid size or other kernel on the device can stall it.
// A workgroup keeps to one image: workgroup i < n to image i, the others in
// proportion to the images' slots (t_first[i]: the first of image i's, counted
// from n), so that the images end together. The holder of ticket t draws again
// if t + g is a ticket, g being the number of workgroups on the image: then
// exactly as many tickets are drawn as there are slots. Reads and read-modify-
// writes of one word pass one after another, about 11 ns each, so nobody looks
// for work in vain: when every workgroup went over the counters of all images
// at the end, draws took 6 us on average and 14 us at the 95th percentile in
// the last third of a compression.
// With fewer workgroups than images, workgroup w takes the images w, w +
// gridDim.x, ... one after another, alone on each.
struct Drawer {
  int img;      // current image; -1: no more slots for this workgroup
  uint32_t g;   // workgroups on it
};

__device__ __forceinline__ Drawer draw_start(const uint32_t* t_first, int n) {
  const int w = (int)blockIdx.x;
  if ((int)gridDim.x <= n) return Drawer{w, 1u};
  // lane i: image i's workgroups are those from t_first[i] to t_first[i + 1]
  const int lane = threadIdx.x % kWave;
  const uint32_t lo = lane < n ? t_first[lane] : ~0u, hi = lane < n ? t_first[lane + 1] : ~0u;
  int img = w;
  if (w >= n) {
    const uint64_t mine = __ballot((uint32_t)(w - n) >= lo && (uint32_t)(w - n) < hi);
    img = mine ? (int)__builtin_ctzll(mine) : -1;
  }
  img = uniform(img);
  return Drawer{img, 1u + (uint32_t)__builtin_amdgcn_readlane((int)(hi - lo), img < 0 ? 0 : img)};
}

// The holder of ticket `last` moves on if its image has no further ticket for
// it. Uniform over the workgroup.
__device__ __forceinline__ void draw_advance(Drawer& d, const uint32_t* t_slots, int n, int last) {
  if ((uint64_t)last + d.g >= (uint64_t)(uint32_t)uniform((int)t_slots[d.img]))
    d = Drawer{d.img + (int)gridDim.x < n ? d.img + (int)gridDim.x : -1, 1u};
}

// Lane 0 draws a ticket of the current image, whose latency can pass while
// the wave works (~0 if there is no image).
__device__ __forceinline__ uint32_t draw_ticket(const Drawer& d, uint32_t* tickets) {
  uint32_t t = ~0u;
  if (d.img >= 0 && threadIdx.x % kWave == 0)
    t = __hip_atomic_fetch_add(&tickets[d.img * kTicketStride], 1u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
  return t;
}

// The slot of a drawn ticket: (image, block), or (-1, 0). Uniform.
__device__ __forceinline__ int2 draw_slot(const Drawer& d, uint32_t t, const uint32_t* t_slots) {
  t = (uint32_t)__builtin_amdgcn_readlane((int)t, 0);
  return d.img >= 0 && t < t_slots[d.img] ? int2{d.img, (int)t} : int2{-1, 0};
}

// A lane's 16 pixels of a slot as they were loaded: four quads of colour and
// of depth, and of the quad that holds a row's end (if one does) the pixels
// that lie in the next row.
struct PxLoad {
  u32x4 c[4], d[4], c2, d2;
  uint32_t left;   // pixels up to the row's end
};

// Issues the loads of this lane's 16 pixels of slot c (zeros past the block);
// compress_join makes the pixels of them. A wave whose pixels all lie in the
// block, of a rectangle at least 16 pixels wide, takes four quads of 16 bytes
// per plane, each from its own row; one quad per lane can hold a row's end:
// it is read a second time at the place where its remaining pixels lie in the
// next row (both reads stay between two pixels of the image). At a width of
// 1000 pixels nearly every wave holds a row's end; taken pixel by pixel by
// that one lane, as it was, it cost the wave 16 rounds of address arithmetic
// behind branches, a third of the compressor's vector instructions.
__device__ __forceinline__ void compress_load(const RleCArgs& a, const CSlot& c, int tid,
                                              PxLoad& px) {
  const RleCImg& I = a.im[c.s];
  const uint32_t* const depth = I.depth;
  const int64_t pitch = I.pitch;
  // a stream is smaller than 4 GiB, so its pixels are counted in 32 bits
  const uint32_t npx = (uint32_t)c.rw * (uint32_t)c.rh, first = (uint32_t)c.b * kBlock;
  const int len = (int)min((uint32_t)kBlock, npx - first);
  const int q0 = tid * kPxPerLane;
  const uint32_t rw = c.rw > 0 ? (uint32_t)c.rw : 1u;
  const uint32_t y = (first + (uint32_t)q0) / rw, x = first + (uint32_t)q0 - y * rw;
  const int64_t off = (int64_t)(uint32_t)(c.ry + (int)y) * pitch + (c.rx + (int)x);
  const int64_t jump = pitch - (int64_t)rw;   // from a row's end to the next row
  const int wave_end = uniform((tid / kWave + 1) * (kWave * kPxPerLane));
  px.c2 = px.d2 = u32x4{0, 0, 0, 0};
  if (rw >= kPxPerLane && wave_end <= len) {   // uniform
    const uint32_t left = px.left = rw - x;
    const bool split = left < kPxPerLane && (left & 3u) != 0;
    const int64_t next = off + (left & ~3u) + jump;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      px.c[v] = ld_u32x4(I.color + (off + 4 * v + ((uint32_t)(4 * v) >= left ? jump : 0)));
    if (split) px.c2 = ld_u32x4(I.color + next);
    if (depth) {   // uniform
#pragma unroll
      for (int v = 0; v < 4; ++v)
        px.d[v] = ld_u32x4(depth + (off + 4 * v + ((uint32_t)(4 * v) >= left ? jump : 0)));
      if (split) px.d2 = ld_u32x4(depth + next);
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v) px.d[v] = u32x4{0, 0, 0, 0};
    }
  } else {
    int64_t o = off;
    uint32_t xx = x;
    px.left = ~0u;
#pragma unroll
    for (int j = 0; j < kPxPerLane; ++j) {
      uint32_t cv = 0, dv = 0;
      if (q0 + j < len) {
        cv = I.color[o];
        if (depth) dv = depth[o];
        ++o;
        if (++xx == rw) {
          xx = 0;
          o += jump;
        }
      }
      px.c[j / 4][j % 4] = cv;
      px.d[j / 4][j % 4] = dv;
    }
  }
}

// The pixels of a load: pixel 4 v + i comes from the second read when the row
// ends inside quad v at or before it.
__device__ __forceinline__ void compress_join(const PxLoad& px, uint32_t (&col)[kPxPerLane],
                                              uint32_t (&dep)[kPxPerLane]) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const uint32_t d = px.left - (uint32_t)(4 * v + 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool next = i > 0 && d < (uint32_t)i;
      col[4 * v + i] = next ? px.c2[i] : px.c[v][i];
      dep[4 * v + i] = next ? px.d2[i] : px.d[v][i];
    }
  }
}

// Arguments of a decompression: the streams and their destinations.
struct RleDImg {
  const uint8_t* in;
  uint64_t in_bytes;
  uint32_t* color;
  uint32_t* depth;
  int64_t pitch;
  int32_t cap_w, cap_h;
};

struct RleDArgs {
  RleDImg im[kRleMax];
  int32_t* roi_out;
  int32_t* status;
  int32_t at_roi;   // blocks go to their ROI's position in a frame (else to its top left)
  int32_t n;
};
static_assert(sizeof(RleDArgs) <= 4096, "kernel arguments must fit in 4 KiB");

// 4 x 4 byte transpose: byte j of o_i is byte i of input j (pixel words to
// plane words and back). v_perm takes bytes 0..3 from its second operand and
// 4..7 from its first: two rounds of four.
__device__ __forceinline__ void transpose4x4(uint32_t a, uint32_t b, uint32_t c, uint32_t d,
                                             uint32_t& o0, uint32_t& o1, uint32_t& o2,
                                             uint32_t& o3) {
  const uint32_t t0 = __builtin_amdgcn_perm(b, a, 0x05010400u);   // a0 b0 a1 b1
  const uint32_t t1 = __builtin_amdgcn_perm(b, a, 0x07030602u);   // a2 b2 a3 b3
  const uint32_t t2 = __builtin_amdgcn_perm(d, c, 0x05010400u);   // c0 d0 c1 d1
  const uint32_t t3 = __builtin_amdgcn_perm(d, c, 0x07030602u);   // c2 d2 c3 d3
  o0 = __builtin_amdgcn_perm(t2, t0, 0x05040100u);                // a0 b0 c0 d0
  o1 = __builtin_amdgcn_perm(t2, t0, 0x07060302u);                // a1 b1 c1 d1
  o2 = __builtin_amdgcn_perm(t3, t1, 0x05040100u);                // a2 b2 c2 d2
  o3 = __builtin_amdgcn_perm(t3, t1, 0x07060302u);                // a3 b3 c3 d3
}

// DPP row shift right by D lanes inside rows of 16 lanes; lanes whose source
// lies outside the row read 0.
template <int D>
__device__ __forceinline__ uint32_t row_shr(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x110 + D, 0xF, 0xF, true);
}

// The slot table of a compression (all threads call it; ends before the
// caller's barrier): wave 0 clamps image i's device ROI in lane i (n <= 64,
// one load) and counts its blocks; an empty ROI still takes one slot, whose
// workgroup writes the header-only stream. t_first: see Drawer; workgroups
// beyond the slots get none.
__device__ __forceinline__ void slot_table(const RleCArgs& a, int4* t_roi, uint32_t* t_slots,
                                           uint32_t* t_first, uint32_t* t_all) {
  const int tid = threadIdx.x, lane = tid % kWave;
  if (tid < kWave) {
    int lx = 0, ly = 0, lw = 0, lh = 0;
    uint32_t lslots = 0;
    if (lane < a.n) {
      const int W = a.im[lane].W, H = a.im[lane].H;
      if (a.roi_dev) {
        const int4 r = reinterpret_cast<const int4*>(a.roi_dev)[lane];
        lx = min(max(r.x, 0), W);
        ly = min(max(r.y, 0), H);
        lw = min(max(r.z, 0), W - lx);
        lh = min(max(r.w, 0), H - ly);
        if (lw == 0 || lh == 0) { lx = 0; ly = 0; lw = 0; lh = 0; }
      } else {
        lw = W; lh = H;
      }
      const uint32_t nb = (uint32_t)rle_nblocks((int64_t)lw * lh);
      lslots = nb ? nb : 1;
    }
    const uint32_t incl = wave_incl_scan32(lslots);   // < 2^24 (checked on the host)
    const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    const uint32_t rest = min(gridDim.x, all) - min(min(gridDim.x, all), (uint32_t)a.n);
    t_roi[lane] = int4{lx, ly, lw, lh};
    t_slots[lane] = lslots;
    // a workgroup per slot if there are enough; else in proportion by a rounded
    // factor (a 64-bit division takes longer than the rest of the table):
    // ascending, and all of them in the end
    const uint32_t share = all <= gridDim.x
                               ? incl - min(incl, (uint32_t)lane + 1u)
                               : (uint32_t)((float)incl * ((float)rest / (float)all));
    t_first[lane + 1] = lane >= a.n - 1 ? rest : min(share, rest);
    if (lane == 0) {
      t_first[0] = 0;
      *t_all = all;
    }
  }
}

// Decoupled look-back (Merrill and Garland 2016) for block b of one image,
// run by all 64 lanes of one wave: the sum of the payload sizes of blocks
// 0..b-1, read from their flags 256 at a time (4 per lane, each load
// instruction contiguous over the lanes), summing aggregates back to the
// nearest inclusive prefix. Split into the issue of a window's loads and its
// examination, so that the wave can encode between the two. A wait that runs
// out of polls, or a poisoned prefix, sets `poisoned`.
struct LookBack {
  uint64_t f[kLookback];   // flag i of lane l: predecessor top - (64 i + l)
  uint32_t excl, spins;
  int b, top;
  bool poisoned;
};

__device__ __forceinline__ void lookback_load(LookBack& lb, const uint64_t* flags) {
  const int lane = threadIdx.x % kWave;
  // unconditional, so that the loads go out together: a lane before block 0
  // reads the block's own flag instead (lookback_step ignores it)
#pragma unroll
  for (int i = 0; i < kLookback; ++i) {
    const int p = lb.top - (kWave * i + lane);
    lb.f[i] = __hip_atomic_load(&flags[p >= 0 ? p : lb.b], __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
  }
}

__device__ __forceinline__ void lookback_begin(LookBack& lb, const uint64_t* flags, int b) {
  lb.excl = lb.spins = 0;
  lb.b = b;
  lb.top = b - 1;
  lb.poisoned = false;
  if (b > 0) lookback_load(lb, flags);
}

// Examines the loaded window. True: the look-back has ended (excl or
// poisoned is set); false: load (a window further back, or the same one
// again) and step again. Uniform.
__device__ __forceinline__ bool lookback_step(LookBack& lb, uint32_t wait_limit, uint32_t ep) {
  if (lb.b == 0) return true;
  const int lane = threadIdx.x % kWave;
  uint64_t f[kLookback];
#pragma unroll
  for (int i = 0; i < kLookback; ++i)   // before block 0: an empty prefix
    f[i] = lb.top - (kWave * i + lane) >= 0 ? lb.f[i] : mkflag(kIncl, 0, ep);
  // the nearest inclusive (or poisoned) prefix, at distance 64 i + lane,
  // and whether every flag up to it is ready
  int first = kWave * kLookback;
  bool waiting = false;
#pragma unroll
  for (int i = kLookback - 1; i >= 0; --i) {
    const uint64_t incl = __ballot(flag_state(f[i], ep) >= kIncl);
    if (incl) first = kWave * i + (int)__builtin_ctzll(incl);
  }
  uint64_t pz = 0;
#pragma unroll
  for (int i = 0; i < kLookback; ++i) {
    const uint64_t st = flag_state(f[i], ep);
    if (__ballot(st == 0 && kWave * i + lane <= first)) waiting = true;
    pz |= __ballot(st == kPoison && kWave * i + lane == first);
  }
  if (waiting) {
    // running out of polls is never expected: see draw_slot
    lb.poisoned = ++lb.spins > wait_limit;
    return lb.poisoned;
  }
  if (pz) {   // the prefix this block needs is unknown
    lb.poisoned = true;
    return true;
  }
  uint32_t v = 0;
#pragma unroll
  for (int i = 0; i < kLookback; ++i)
    if (kWave * i + lane <= first) v += (uint32_t)f[i];
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
  lb.excl += v;
  if (first < kWave * kLookback) return true;
  lb.top -= kWave * kLookback;
  return false;
}

// Polls until the look-back has ended.
__device__ __forceinline__ void lookback_finish(LookBack& lb, const uint64_t* flags,
                                                uint32_t wait_limit, uint32_t ep) {
  while (!lookback_step(lb, wait_limit, ep)) {
    __builtin_amdgcn_s_sleep(1);
    lookback_load(lb, flags);
  }
}

// Block b's inclusive prefix (excl + padded), or its poisoned flag; lane 0
// of the wave that ran the look-back. Block 0 published its inclusive
// prefix with its size.
__device__ __forceinline__ void publish_incl(uint64_t* flags, int b, uint32_t excl,
                                             uint32_t padded, bool poisoned, uint32_t ep) {
  if (b != 0 && threadIdx.x % kWave == 0)
    __hip_atomic_store(&flags[b],
                       poisoned ? mkflag(kPoison, 0, ep) : mkflag(kIncl, excl + padded, ep),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A block that is staged but not written yet: its payload offset is still to
// be found. All uniform; out == nullptr: none.
struct Pending {
  uint8_t* out;
  uint64_t* flags;
  uint64_t P0, nb;
  int s, b;
  uint32_t padded;
};

// Finds the offset of a pending block (wave 0, which has begun the look-back)
// and writes its table entry and its payload. One barrier; the caller keeps
// another between these reads of the stage and its next writes.
__device__ __forceinline__ void write_pending(const RleCArgs& a, const Pending& p, LookBack& lb,
                                              int wave, int lane, int tid, uint32_t ep,
                                              uint32_t* s_excl, int32_t* s_poison,
                                              const uint8_t* stage) {
  if (wave == 0) {
    lookback_finish(lb, p.flags, a.wait_limit, ep);
    publish_incl(p.flags, p.b, lb.excl, p.padded, lb.poisoned, ep);
    if (lane == 0) {
      *s_excl = lb.excl;
      *s_poison = lb.poisoned ? 1 : 0;
      if (lb.poisoned) a.status[p.s] = CMP_ETIMEOUT;
    }
  }
  __syncthreads();   // the offset is written, and the stage complete
  const uint32_t excl = *s_excl;
  const bool poisoned = *s_poison != 0;
  if (tid == 0) {
    // a poisoned block's offset is unknown: its table entry is made invalid
    // (not a multiple of 16, which decompression rejects) and its payload is
    // not written
    if (p.nb != 0) reinterpret_cast<uint32_t*>(p.out + 32)[p.b] = poisoned ? 0xFFFFFFFFu : excl;
    if ((uint64_t)p.b + 1 >= p.nb) a.out_size[p.s] = poisoned ? 0 : p.P0 + excl + p.padded;
  }
  if (!poisoned) {
    u32x4* dst = reinterpret_cast<u32x4*>(p.out + p.P0 + excl);
    const u32x4* src = reinterpret_cast<const u32x4*>(stage);
    for (uint32_t i = tid; i < p.padded / 16; i += kThreads)
      __builtin_nontemporal_store(src[i], &dst[i]);   // streamed out, not re-read
  }
}

// ---------------------------------------------------------------- host
// Workgroups of `kernel` that fit on the device at once, at most `cap` per
// compute unit when cap > 0 (the per-unit occupancy is cached per device).
int resident_groups(const void* kernel, std::atomic<int>* cache, int cap);
// Look-back flags a compression needs: one per block of each image's
// largest possible ROI (one for an empty image).
int64_t rle_flag_count(const cmp_image* imgs, int32_t n);
// Polls before a compressing block gives up (cmp_rle_set_wait_limit).
uint32_t rle_wait_limit();
// Caps on the compressors' workgroups per compute unit (0: as many as fit).
int rle_compress_cap();
// Validates a compression call of n images whose streams need at most
// max_size(w, h, has depth) bytes and fills `a` (all but the codec's flags)
// and `grid` (the number of slots). Enqueues nothing.
cmp_status rle_compress_prepare(const cmp_image* imgs, int32_t n, const int32_t* roi_dev,
                                uint8_t* const* out, const uint64_t* capacity,
                                uint64_t* out_size_dev, int32_t* status_dev, void* workspace,
                                size_t ws_bytes, size_t (*max_size)(int32_t, int32_t, bool),
                                RleCArgs& a, int64_t& grid);

}  // namespace cmp
