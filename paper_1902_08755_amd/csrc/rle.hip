// cmp_rle_compress / cmp_rle_decompress: per-component run-length encoding of
// RGBA8 (+ depth) pixels in the RLE1 format (Section 5.5.1, Enhanced RLE
// Compression: one stream per pixel component; the image is decomposed into
// sub-images compressed in parallel). Format: see cmp.h.
//
// Compression is a single pass over the input. A workgroup owns one block of
// 4096 pixels of one image (16 consecutive pixels per lane) and encodes all
// planes of it from registers:
//   - the pixels become plane words by 4x4 byte transposes;
//   - run starts: byte != previous byte, or a multiple of 256 pixels; the
//     previous lane's last byte comes from the lane's DPP row of 16 (a row
//     starts at a 256-pixel boundary);
//   - token slots: a workgroup-wide exclusive scan of the per-lane run counts
//     (eight 16-bit counters packed in four 32-bit words);
//   - run ends: the next start in the lane, else a suffix minimum of the first
//     starts over the following lanes of the same 256-pixel segment;
//   - the encoded block is staged in LDS, and its payload offset comes from a
//     decoupled look-back over the blocks of the image (Merrill and Garland,
//     "Single-pass Parallel Prefix Scan with Decoupled Look-back", 2016),
//     one wave reading 256 predecessors' flags at a time.
// The grid is at most one resident wave of workgroups, which draw (image,
// block) slots from a ticket counter per image (each on its own cache line),
// so the blocks of an image go out in order and only to running workgroups:
// every block a look-back waits for is held by a workgroup that makes
// progress, whatever else runs on the device. No kernel clears the workspace:
// the last workgroup to finish zeroes the tickets, and the look-back flags
// carry a per-call epoch.
// What bounds it: four blocks per compute unit (LDS and registers), each a
// chain of about 3 to 4 us of pixel loads, 2 us of counting, 2 us of look-back,
// 0.5 us of writes and 2 us of staging. Waits between blocks and contended
// counters used to double that; see the order of work in the kernel, and
// Drawer. 16 x 1920x1080 ROIs (107 MB): 58.3 -> 42.3 us; 8 x 3840x2160 (211
// MB): 112 -> 63 us (3.3 TB/s).
// Every workgroup derives the slot count from the device ROIs, so blocks that
// the ROIs leave out cost nothing.
//
// Decompression: a grid-stride loop over the blocks of all streams (counted
// from the stream headers); per block: table checks (made uniform: scalar
// work), each lane's 16-byte window of every plane straight from the stream
// (its 16 raw bytes, its up to 8 tokens, or the token of its 256-pixel
// segment), one workgroup scan of the run-length sums of the run-coded planes
// with more than a run per segment, the runs of up to four of those planes at
// a time scattered into LDS (value and start bit), and per lane a fill of its
// 16 pixels from the last run start. The value entering a lane comes from a
// scan over its DPP row of 16 lanes: a row covers one 256-pixel segment,
// which no run crosses. Pixels are assembled in registers, restaged through
// the wave's part of LDS and written with 16-byte stores, colour, then depth.
// What bounds it: the memory system (8 x 3840x2160 ROIs, 52 MB read and 160
// MB written: 53 us, 4.0 TB/s, where a copy reaches 5.0) and, where there are
// only about two blocks per workgroup, the two dependent round trips (table,
// windows; 2.3 us each among the stores) that each block starts with. At 62 us
// it had four workgroups per compute unit (40 KB of LDS for eight planes of
// values), 1350 vector instructions per block and wave (now 900) and its row
// ends stored through a division each. Six workgroups (80 registers, one
// spilled): 58 us; the next block's windows prefetched into registers at four:
// 53 us, and slower for one large image (25 against 22 us).
#include <string.h>

#include <atomic>
#include <mutex>

#include "rle_common.hpp"

namespace cmp {

// The tokens (run length - 1, value) of this lane's runs of one plane, to
// `dst` on: m (not 0) marks the runs' first pixels among the lane's 16, byte
// j % 4 of w[j / 4] is pixel j, and the last run ends before pixel `after`
// (counted from the lane's first). 16-bit stores when dst is even.
template <bool kEven>
__device__ __forceinline__ void emit_tokens(uint8_t* dst, uint32_t m, const uint32_t (&w)[4],
                                            uint32_t after) {
  uint32_t j = (uint32_t)__builtin_ctz(m);
  while (true) {
    m &= m - 1u;
    const uint32_t next = m ? (uint32_t)__builtin_ctz(m) : after;
    // byte j of the 16 as byte 1 of the token: from either half by v_perm
    // (selector 0x0c gives a zero byte)
    const uint32_t sel = ((j & 7u) << 8) | 0x0C0C000Cu;
    const uint32_t lo = __builtin_amdgcn_perm(w[1], w[0], sel);
    const uint32_t hi = __builtin_amdgcn_perm(w[3], w[2], sel);
    const uint32_t tok = (j & 8u ? hi : lo) + next + ~j;   // | next - j - 1
    if (kEven) {
      *reinterpret_cast<uint16_t*>(dst) = (uint16_t)tok;
    } else {
      dst[0] = (uint8_t)tok;
      dst[1] = (uint8_t)(tok >> 8);
    }
    if (!m) break;
    dst += 2;
    j = next;
  }
}

// Bit j of the result: byte j % 4 of word j / 4 differs from the byte before
// it (prev: the word whose last byte precedes the first). v_lerp_u8 with
// 0xFF sets a byte's top bit exactly when the byte is not 0, and v_dot4 sums
// the top bits with the weights of their positions.
__device__ __forceinline__ uint32_t change_mask(const uint32_t (&w)[4], uint32_t prev) {
  uint32_t t[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t x = w[i] ^ __builtin_amdgcn_alignbyte(w[i], i ? w[i - 1] : prev, 3);
    t[i] = __builtin_amdgcn_lerp(x, 0xFFFFFFFFu, 0u) & 0x80808080u;
  }
  const uint32_t lo = __builtin_amdgcn_udot4(t[1], 0x80402010u,
                                             __builtin_amdgcn_udot4(t[0], 0x08040201u, 0u, false), false);
  const uint32_t hi = __builtin_amdgcn_udot4(t[3], 0x80402010u,
                                             __builtin_amdgcn_udot4(t[2], 0x08040201u, 0u, false), false);
  return (lo + (hi << 8)) >> 7;
}

// kSwizzle: the colour words are bit-swizzled before their planes are taken
// (a template parameter, so that the plain kernel carries no branch and no
// copies of the pixel registers for it).
template <bool kSwizzle>
__global__ __launch_bounds__(kThreads, 4) void rle_compress_kernel(const RleCArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t stage[kStage];
  __shared__ uint32_t sh[16];
  __shared__ uint32_t s_excl;
  __shared__ int32_t s_poison;

  // Slots: one per block of every image's ROI (an empty ROI still takes one
  // slot, whose workgroup writes the header-only stream). Wave 0 computes the
  // table (lane i: image i, n <= 64; one load) into LDS.
  __shared__ int4 t_roi[kRleMax];
  __shared__ uint32_t t_slots[kRleMax], t_first[kRleMax + 1], t_all;
  __shared__ int2 s_next;   // the slot drawn for the next iteration
  slot_table(a, t_roi, t_slots, t_first, &t_all);
  const uint32_t ep = call_epoch(a);
  __syncthreads();

  // Slots come from per-image tickets, drawn by wave 1: the first here, each
  // further one while the block before it is staged.
  Drawer drawer = draw_start(t_first, a.n);
  if (threadIdx.x / kWave == 1) {
    const uint32_t t = draw_ticket(drawer, a.tickets);
    const int2 sb = draw_slot(drawer, t, t_slots);
    if (threadIdx.x == kWave) s_next = sb;
  }
  __syncthreads();
  int2 cur = s_next;
  Pending pend{nullptr, nullptr, 0, 0, 0, 0, 0};
  // An iteration loads and counts one block, publishes its size, then finds
  // the offset of the block before it (staged in LDS), writes that one, and
  // stages the new one. A block's size is thus published before the workgroup
  // waits for anything: a wait for predecessors never delays a size that
  // others wait for, so waits do not pile up along an image, and by the time
  // a block looks back its predecessors have had a whole block's time to
  // publish. (With the look-back ahead of the next block's loads, waits of 4
  // to 9 us per block made up most of the kernel.) It also means that a wait
  // cannot deadlock: between a slot's draw and its size there is none.
  LookBack lb;
  bool looking = false;   // the pending block's look-back has begun
  while (true) {
    // an opaque copy of the thread index: keeps per-lane values from being
    // hoisted out of the loop and held in registers across iterations
    int tid = threadIdx.x;
    __asm__ volatile("" : "+v"(tid));
    const int lane = tid % kWave, wave = uniform(tid / kWave);
    const bool have = uniform(cur.x) >= 0;
    const int q0 = tid * kPxPerLane;   // block-relative first pixel
    Pending now{nullptr, nullptr, 0, 0, 0, 0, 0};
    uint32_t pl[8][4];   // plane words: byte j of pl[k][i] is plane k of pixel 4 i + j
    uint32_t masks[8], ex[4], poff[8], total = 0, raw = 0;
    int np = 0, len = 0;
    if (have) {
      const CSlot c = compress_slot(cur, t_roi);
      const RleCImg I = a.im[c.s];
      np = I.depth ? 8 : 4;
      const int64_t npx = (int64_t)c.rw * c.rh;
      const uint64_t nb = rle_nblocks(npx);   // 0: an empty ROI, a block without pixels
      const uint64_t P0 = rle_p0(nb, np);
      len = (int)imin64(kBlock, npx - (int64_t)c.b * kBlock);
      {
        PxLoad px;
        compress_load(a, c, tid, px);
        uint32_t col[kPxPerLane], dep[kPxPerLane];
        compress_join(px, col, dep);
        if (kSwizzle) {
#pragma unroll
          for (int j = 0; j < kPxPerLane; ++j) col[j] = swizzle_bits(col[j]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          transpose4x4(col[4 * i], col[4 * i + 1], col[4 * i + 2], col[4 * i + 3], pl[0][i],
                       pl[1][i], pl[2][i], pl[3][i]);
          transpose4x4(dep[4 * i], dep[4 * i + 1], dep[4 * i + 2], dep[4 * i + 3], pl[4][i],
                       pl[5][i], pl[6][i], pl[7][i]);
        }
      }
      // the flags that the pending block waits for are on their way meanwhile
      if (pend.out && wave == 0) lookback_begin(lb, pend.flags, pend.b);

      // ---- run starts (byte != previous byte, or a segment start: the first
      // lane of a DPP row, so the previous lane's last byte comes from the
      // row) as one 16-bit mask per plane, and their counts
      const bool seg_start = (tid % (kSeg / kPxPerLane)) == 0;
      const int nvalid = min(kPxPerLane, max(0, len - q0));
      const uint32_t vmask = (1u << nvalid) - 1u;
      uint32_t cnt[4] = {0, 0, 0, 0}, tot[4];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        masks[k] = 0;
        if (k >= np) continue;
        const uint32_t m = change_mask(pl[k], row_shr<1>(pl[k][3])) | (seg_start ? 1u : 0u);
        masks[k] = m & vmask;
        cnt[k >> 1] |= (uint32_t)__builtin_popcount(masks[k]) << (16 * (k & 1));
      }
      block_scan32_once<4>(cnt, ex, tot, sh);

      // ---- plane sizes and offsets (uniform)
      uint32_t size[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        size[k] = 0;
        poff[k] = total;
        if (k >= np) continue;
        const uint32_t ntok = (tot[k >> 1] >> (16 * (k & 1))) & 0xFFFFu;
        size[k] = (2 * ntok < (uint32_t)len) ? 2 * ntok : (uint32_t)len;
        if (size[k] == (uint32_t)len) raw |= 1u << k;
        total += size[k];
      }
      const uint32_t padded = (uint32_t)align16(total);
      uint64_t* flags = a.flags + I.flag_base;
      // the block's size (block 0: as the inclusive prefix)
      if (tid == 0)
        __hip_atomic_store(&flags[c.b], mkflag(c.b == 0 ? kIncl : kAgg, padded, ep),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      now = Pending{I.out, flags, P0, nb, c.s, c.b, padded};

      // ---- header and the block's plane sizes
      uint32_t* tbl = reinterpret_cast<uint32_t*>(I.out + 32);
      if (nb != 0 && tid < np) {
        uint32_t v = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (k == tid) v = size[k];
        tbl[nb + (uint64_t)c.b * np + tid] = v;
      }
      if (c.b == 0) {
        if (tid < 8) {
          const uint32_t hdr[8] = {kRleMagic, (uint32_t)c.rx, (uint32_t)c.ry, (uint32_t)c.rw,
                                   (uint32_t)c.rh, (uint32_t)np | (kSwizzle ? 0x100u : 0u),
                                   (uint32_t)kBlock, (uint32_t)nb};
          reinterpret_cast<uint32_t*>(I.out)[tid] = hdr[tid];
        }
        const uint64_t tend = 32 + 4 * nb * (1 + (uint64_t)np);
        if ((uint64_t)tid < P0 - tend) I.out[tend + tid] = 0;
      }
    } else if (pend.out && !looking && wave == 0) {
      lookback_begin(lb, pend.flags, pend.b);
    }

    // ---- the pending block: its offset, its table entry, its payload
    if (pend.out) {
      write_pending(a, pend, lb, wave, lane, tid, ep, &s_excl, &s_poison, stage);
      __syncthreads();   // the stage is read
    }
    if (!have) break;
    draw_advance(drawer, t_slots, a.n, now.b);
    uint32_t t_next = ~0u;
    if (wave == 1) t_next = draw_ticket(drawer, a.tickets);
    // the workgroup's last block looks back while it is staged
    looking = drawer.img < 0;
    if (looking && wave == 0) lookback_begin(lb, now.flags, now.b);

    // ---- stage the encoded block in LDS
    const uint32_t seg_end = (uint32_t)min(len, ((q0 / kSeg) + 1) * kSeg);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (k >= np) continue;
      const uint32_t m = masks[k];
      const uint32_t off = poff[k];
      if (!((raw >> k) & 1u)) {
        // a run ends at the next start: in this lane, else the first start
        // of the following lanes of the segment (a suffix minimum over the
        // lane's DPP row), else the segment end
        uint32_t fs = m ? (uint32_t)(q0 + __builtin_ctz(m)) : ~0u;
        fs = min(fs, (uint32_t)row_shl_fill<1>((int)fs, -1));
        fs = min(fs, (uint32_t)row_shl_fill<2>((int)fs, -1));
        fs = min(fs, (uint32_t)row_shl_fill<4>((int)fs, -1));
        fs = min(fs, (uint32_t)row_shl_fill<8>((int)fs, -1));
        const uint32_t after = min((uint32_t)row_shl_fill<1>((int)fs, -1), seg_end) - (uint32_t)q0;
        const uint32_t tok0 = (ex[k >> 1] >> (16 * (k & 1))) & 0xFFFFu;
        if (m) {
          if ((off & 1u) == 0)
            emit_tokens<true>(stage + off + 2 * tok0, m, pl[k], after);
          else
            emit_tokens<false>(stage + off + 2 * tok0, m, pl[k], after);
        }
      } else if ((off & 1u) == 0 && q0 + kPxPerLane <= len) {
        // raw plane at an even offset: 32-bit stores, shifted by a half word
        // when the offset is 2 modulo 4 (the size of a run-coded plane before
        // it is even)
        uint8_t* dst = stage + off + q0;
        if ((off & 2u) == 0) {
#pragma unroll
          for (int i = 0; i < 4; ++i) reinterpret_cast<uint32_t*>(dst)[i] = pl[k][i];
        } else {
          *reinterpret_cast<uint16_t*>(dst) = (uint16_t)pl[k][0];
#pragma unroll
          for (int i = 0; i < 3; ++i)
            reinterpret_cast<uint32_t*>(dst + 2)[i] =
                __builtin_amdgcn_alignbyte(pl[k][i + 1], pl[k][i], 2);
          *reinterpret_cast<uint16_t*>(dst + 14) = (uint16_t)(pl[k][3] >> 16);
        }
      } else {
#pragma unroll
        for (int j = 0; j < kPxPerLane; ++j)
          if (q0 + j < len) stage[off + q0 + j] = (uint8_t)(pl[k][j >> 2] >> (8 * (j & 3)));
      }
    }
    if ((uint32_t)tid < now.padded - total) stage[total + tid] = 0;
    pend = now;
    cur = int2{-1, 0};
    if (!looking) {   // (after the last block, write_pending's barrier is the next one)
      if (wave == 1) {
        const int2 sb = draw_slot(drawer, t_next, t_slots);
        if (lane == 0) s_next = sb;
      }
      __syncthreads();   // s_next is written
      cur = s_next;
    }
  }
  finish_call(a, ep, t_all);
}

// ---------------------------------------------------------- decompress
// 16 bytes at any byte offset `off` of a buffer whose first `end` bytes
// (end >= 16) may be read: load16_from reads them with one 16-byte load from
// src = min(off, end - 16); when the bytes run past `end`, load16_fix shifts
// the 16 bytes that end there into place (bytes past `end` read 0). Split in
// two so that a lane's loads are all issued before any of them is waited for.
// Offsets are 32-bit: a stream is smaller than 4 GiB.
__device__ __forceinline__ u32x4 load16_from(const uint8_t* base, uint32_t src) {
  u32x4 v;
  __builtin_memcpy(&v, base + src, 16);
  return v;
}
__device__ __forceinline__ u32x4 load16_fix(u32x4 v, uint32_t src, uint32_t off) {
  if (src != off) {   // rare: the last bytes of an exactly sized buffer
    uint32_t d = (uint32_t)(off - src);   // 1..15
    uint64_t lo = (uint64_t)v.x | ((uint64_t)v.y << 32), hi = (uint64_t)v.z | ((uint64_t)v.w << 32);
    if (d >= 8) { lo = hi; hi = 0; d -= 8; }
    if (d) { lo = (lo >> (8 * d)) | (hi << (64 - 8 * d)); hi >>= 8 * d; }
    v = u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
  }
  return v;
}

// A block to decode: what its table entries say. All uniform.
struct DBlock {
  int np, len;
  uint32_t pay, btotal;
  uint32_t tokmask;   // planes stored as runs
  uint32_t segmask;   // ... of one run per 256-pixel segment
  uint32_t size[8], poff[8];
  // Tokens per lane of a run-coded plane: T tokens are taken ceil(T / 256) to
  // a lane (at most 8), so that all four waves share the scatter.
  __device__ __forceinline__ int tpl(int k) const {
    return max(1, ((int)(size[k] / 2) + kThreads - 1) / kThreads);
  }
  // This lane's tokens.
  __device__ __forceinline__ int tokens(int k, int tid) const {
    return min(tpl(k), max(0, (int)(size[k] / 2) - tid * tpl(k)));
  }
  // This lane's first byte in plane k.
  __device__ __forceinline__ uint32_t step(int k, int tid) const {
    if ((segmask >> k) & 1u) return 2u * (uint32_t)(tid / (kSeg / kPxPerLane));
    return ((tokmask >> k) & 1u ? 2u * (uint32_t)tpl(k) : (uint32_t)kPxPerLane) * (uint32_t)tid;
  }
};

// Waves per SIMD, so workgroups per compute unit: what 89 registers allow.
constexpr int kDecompressWaves = 5;
// Planes whose runs are placed in LDS at a time. Rendered frames seldom have
// more that are neither raw nor one run per segment; a block that does takes
// two rounds.
constexpr int kValPlanes = 4;

__global__ __launch_bounds__(kThreads, kDecompressWaves) void rle_decompress_kernel(const RleDArgs a) {
  // the bytes of each run-coded plane's runs at their start positions
  __shared__ __attribute__((aligned(16))) uint8_t vals[kValPlanes * kBlock];
  __shared__ __attribute__((aligned(16))) uint32_t starts[kValPlanes][kBlock / 32];   // run-start bits
  __shared__ uint32_t sh[16];
  __shared__ int32_t s_bad[3];   // a malformed block, in rotation over consecutive slots
  // byte selectors that fill a word from its run starts: for start nibble n,
  // byte j takes the word's byte at the last start <= j, else byte 3 of the
  // previous word (v_perm numbering: 0..3 this word, 4..7 the previous one)
  __shared__ uint32_t fill_sel[16];
  const int tid = threadIdx.x;
  if (tid < 16) {
    uint32_t sel = 0;
    int last = 7;
    for (int j = 0; j < 4; ++j) {
      if ((tid >> j) & 1) last = j;
      sel |= (uint32_t)last << (8 * j);
    }
    fill_sel[tid] = sel;
  }
  if (tid < kValPlanes * kBlock / 32 / 4)
    reinterpret_cast<u32x4*>(&starts[0][0])[tid] = u32x4{0, 0, 0, 0};
  if (tid < 3) s_bad[tid] = 0;
  const int lane = tid % kWave;

  // Wave 0 reads and checks the header of stream i in lane i (n <= 64) into
  // LDS; a stream takes one slot per block, or one slot if it has no blocks
  // or a bad header (that slot reports the status or writes the ROI).
  __shared__ uint32_t t_hdr[kRleMax][8];
  __shared__ int32_t t_err[kRleMax];
  __shared__ uint32_t t_slots[kRleMax], t_incl[kRleMax], t_total;
  if (tid < kWave) {
    uint32_t lh[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int lerr = 0;
    uint32_t lslots = 0;
    if (lane < a.n) {
      const RleDImg& I = a.im[lane];
      if (I.in_bytes < 32) {
        lerr = CMP_ECORRUPT;
      } else {
        const u32x4 h0 = reinterpret_cast<const u32x4*>(I.in)[0];
        const u32x4 h1 = reinterpret_cast<const u32x4*>(I.in)[1];
        lh[0] = h0.x; lh[1] = h0.y; lh[2] = h0.z; lh[3] = h0.w;
        lh[4] = h1.x; lh[5] = h1.y; lh[6] = h1.z; lh[7] = h1.w;
        const int32_t w = (int32_t)lh[3], hh = (int32_t)lh[4];
        const uint32_t np = lh[5] & 0xFFu;
        if (lh[0] != kRleMagic || w < 0 || hh < 0 || (np != 4 && np != 8) ||
            lh[6] != (uint32_t)kBlock || (lh[5] & ~0x1FFu))
          lerr = CMP_ECORRUPT;
        else if ((uint64_t)lh[7] != rle_nblocks((int64_t)w * hh))
          lerr = CMP_ECORRUPT;
        else if (I.in_bytes < rle_p0(lh[7], (int)np))
          lerr = CMP_ECORRUPT;
        else if ((np == 8 && !I.depth) ||
                 (a.at_roi ? (int32_t)lh[1] < 0 || (int32_t)lh[2] < 0 ||
                                 (int64_t)(int32_t)lh[1] + w > I.cap_w ||
                                 (int64_t)(int32_t)lh[2] + hh > I.cap_h
                           : w > I.cap_w || hh > I.cap_h))
          lerr = CMP_ENOSPC;
      }
      lslots = (lerr || lh[7] == 0) ? 1u : lh[7];
    }
    uint32_t lincl = lslots;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const uint32_t o = __shfl_up(lincl, d);
      if (lane >= d) lincl += o;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) t_hdr[lane][k] = lh[k];
    t_err[lane] = lerr;
    t_slots[lane] = lslots;
    t_incl[lane] = lincl;
    if (lane == kWave - 1) t_total = lincl;
  }
  __syncthreads();
  const uint32_t total = t_total;

  uint32_t tslot = 0;   // slots with run-coded planes so far (uniform): picks the s_bad entry
  for (uint32_t g = blockIdx.x; g < total; g += gridDim.x) {
    int tid = threadIdx.x;   // opaque per iteration (see the compressor)
    __asm__ volatile("" : "+v"(tid));
    const int lane = tid % kWave, wave = uniform(tid / kWave);
    const int q0 = tid * kPxPerLane;
    // slot g: stream s, block b
    const uint64_t hit = __ballot(lane < a.n && g < t_incl[lane]);
    const int s = uniform(__builtin_ctzll(hit));
    const int b = uniform((int)(g - (t_incl[s] - t_slots[s])));
    const RleDImg I = a.im[s];
    uint32_t h[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) h[k] = (uint32_t)uniform((int)t_hdr[s][k]);
    const int err = uniform(t_err[s]);
    if (err) {
      if (tid == 0) a.status[s] = err;
      continue;   // uniform; no LDS was touched in this slot
    }
    if (b == 0 && a.roi_out && tid == 0)
      reinterpret_cast<int4*>(a.roi_out)[s] = int4{(int)h[1], (int)h[2], (int)h[3], (int)h[4]};
    const uint32_t nb = h[7];
    if ((uint32_t)b >= nb) continue;   // uniform: a stream without blocks
    const int32_t rw = (int32_t)h[3], rh = (int32_t)h[4];
    const int64_t npx = (int64_t)rw * rh;
    DBlock c;
    c.np = (int)(h[5] & 0xFFu);
    c.len = (int)imin64(kBlock, npx - (int64_t)b * kBlock);
    const uint32_t len = (uint32_t)c.len, in_end = (uint32_t)imin64((int64_t)I.in_bytes, 0xFFFFFFFFll);
    {
      // block table: uniform addresses (three loads issued together; all
      // inside the table the header check found readable, since np is 4 or 8
      // and entry nb is the first size), made uniform, so that the checks and
      // plane offsets are scalar work
      const uint32_t* tbl = reinterpret_cast<const uint32_t*>(I.in + 32);
      const uint32_t* srow = tbl + nb + (uint64_t)b * c.np;
      const u32x4 v03 = ld_u32x4(srow);
      const u32x4 v47 = ld_u32x4(srow + (c.np == 8 ? 4 : 0));
      uint2 bo;   // boff[b], boff[b + 1]: a 4-byte aligned pair
      __builtin_memcpy(&bo, __builtin_assume_aligned(tbl + b, 4), 8);
      const uint32_t boff = (uint32_t)uniform((int)bo.x);
      const uint32_t bnext = (uint32_t)uniform((int)bo.y);   // the first size entry when b is the last block
      c.pay = (uint32_t)(rle_p0(nb, c.np) + boff);
      c.btotal = c.tokmask = c.segmask = 0;
      int e = 0;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const uint32_t sz = (uint32_t)uniform((int)(k < 4 ? v03[k] : v47[k - 4]));
        c.size[k] = k < c.np ? sz : 0u;
        c.poff[k] = c.btotal;
        if (k >= c.np) continue;
        if (sz > len || (sz < len && (sz == 0 || (sz & 1u)))) e = CMP_ECORRUPT;
        if (sz != len) {
          c.tokmask |= 1u << k;
          if (sz / 2 == (len + kSeg - 1) / kSeg) c.segmask |= 1u << k;
        }
        c.btotal += sz;
      }
      if ((boff & 15u) || (b == 0 && boff != 0)) e = CMP_ECORRUPT;
      if ((uint32_t)b + 1 < nb && (uint64_t)bnext != boff + align16(c.btotal)) e = CMP_ECORRUPT;
      // (a stream smaller than 4 GiB: all its offsets are 32-bit)
      if (rle_p0(nb, c.np) + boff + align16(c.btotal) > in_end) e = CMP_ECORRUPT;
      if (e) {   // uniform; no LDS was touched in this slot
        if (tid == 0) a.status[s] = e;
        continue;
      }
    }

    // Every plane's 16-byte window of this lane, straight from the stream: the
    // raw bytes of its 16 pixels, its tokens (run length - 1, value), or its
    // segment's token. A lane without bytes in a plane reads other bytes of
    // the stream, which are not used; a window past the end of the buffer is
    // read from its last 16 bytes and shifted into place.
    u32x4 win[8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      win[k] = load16_from(I.in, min(c.pay + c.poff[k] + c.step(k, tid), in_end - 16u));
    if (c.pay + c.btotal + 16u > in_end || c.pay + c.btotal + 16u < c.pay) {
      // the end of the buffer (uniform)
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const uint32_t lo = c.step(k, tid), off = c.pay + c.poff[k] + lo;
        if (lo < c.size[k]) win[k] = load16_fix(win[k], min(off, in_end - 16u), off);
      }
    }
    if (c.np == 4) {   // uniform
#pragma unroll
      for (int k = 4; k < 8; ++k) win[k] = u32x4{0, 0, 0, 0};
    }
    if (c.tokmask) {   // uniform
      bool bad = false;
      // this slot's flag; the next one's is cleared now: its last readers (two
      // such slots ago) have all passed the previous slot's barrier
      int32_t* bad_flag = &s_bad[tslot % 3];
      if (tid == 0) s_bad[(tslot + 1) % 3] = 0;
      ++tslot;
      // planes with one run per 256-pixel segment: the lane's segment is its
      // token's value throughout, no position is needed
      const uint32_t seg_len = min((uint32_t)kSeg, len - min(len, (uint32_t)(q0 & ~(kSeg - 1))));
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if ((c.segmask >> k) & 1u) {
          const uint32_t tok = win[k].x;
          if ((uint32_t)q0 < len && (tok & 0xFFu) + 1u != seg_len) bad = true;
          const uint32_t v = __builtin_amdgcn_perm(tok, tok, 0x01010101u);
          win[k] = u32x4{v, v, v, v};
        }
      }
      uint32_t runmask = c.tokmask & ~c.segmask;   // the other run-coded planes
      // Start position of this lane's first token in every such plane: sums of
      // run lengths, two 16-bit fields per word. A valid plane's fit (at most
      // 4096); in a malformed one a field may run over into the next, but then
      // some run of its own ends past the block, which every run is checked
      // for below.
      uint32_t ex4[4] = {0, 0, 0, 0};
      if (runmask) {   // uniform
        uint32_t v4[4] = {0, 0, 0, 0}, tot4[4];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if ((runmask >> k) & 1u) {
            const int tpl = c.tpl(k), nv = c.tokens(k, tid);
            uint32_t sum = (uint32_t)nv;   // + the (length - 1) bytes of its tokens
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              if (2 * i < tpl) {   // uniform
                const uint32_t keep = nv > 2 * i + 1 ? 0x00FF00FFu : nv > 2 * i ? 0xFFu : 0u;
                sum = __builtin_amdgcn_sad_u8(win[k][i] & keep, 0u, sum);
              }
            }
            v4[k >> 1] |= sum << (16 * (k & 1));
          }
        }
        block_scan32_once<4>(v4, ex4, tot4, sh);
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (((runmask >> k) & 1u) && ((tot4[k >> 1] >> (16 * (k & 1))) & 0xFFFFu) != len)
            bad = true;   // uniform
      }
      // The runs of up to kValPlanes planes at a time: each run's value at its
      // start position, and its start bit; a run must not cross a multiple of
      // 256 pixels nor end past the block (positions are taken modulo the
      // block, so that a malformed one stays in it too).
      bool block_bad = false;
#pragma unroll 1
      do {
        uint32_t later = runmask;   // the planes of the next round
#pragma unroll
        for (int i = 0; i < kValPlanes; ++i) later &= later - 1u;
        const uint32_t grp = runmask & ~later;
        uint32_t cross = 0, far = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if ((grp >> k) & 1u) {   // uniform
            const int at = __builtin_popcount(grp & ((1u << k) - 1u));
            const int tpl = c.tpl(k), nv = c.tokens(k, tid);
            uint32_t pos = (ex4[k >> 1] >> (16 * (k & 1))) & 0xFFFFu;
            uint8_t* vk = vals + at * kBlock;
            uint32_t* bits = starts[at];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              if (j < tpl) {   // uniform
                if (j < nv) {
                  const uint32_t w = win[k][j >> 1] >> (16 * (j & 1));
                  const uint32_t lastp = pos + (w & 0xFFu);   // the run's last pixel
                  cross = max(cross, pos ^ lastp);
                  far = max(far, lastp);
                  const uint32_t p = pos & (uint32_t)(kBlock - 1);
                  vk[p] = (uint8_t)(w >> 8);
                  __hip_atomic_fetch_or(&bits[p >> 5], 1u << (p & 31u), __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_WORKGROUP);
                  pos = lastp + 1u;
                }
              }
            }
          }
        }
        bad = bad || cross >= (uint32_t)kSeg || far >= len;
        // one vote per wave into this slot's flag, then the barrier that also
        // publishes the runs
        if (__ballot(bad) && lane == 0)
          __hip_atomic_fetch_or(bad_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __syncthreads();
        // Expand: a pixel takes the value of the last run start at or before
        // it. A 256-pixel segment (the 16 lanes of one DPP row) starts with a
        // run, so the value entering a lane comes from a scan over its row.
        const uint32_t lane_key = ((uint32_t)lane + 1u) << 8;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if ((grp >> k) & 1u) {
            const int at = __builtin_popcount(grp & ((1u << k) - 1u));
            const u32x4 d = *reinterpret_cast<const u32x4*>(vals + at * kBlock + q0);
            const uint32_t m = (starts[at][q0 >> 5] >> (q0 & 31)) & 0xFFFFu;
            const uint32_t dv[4] = {d.x, d.y, d.z, d.w};
            // the lane's last start: its byte of the 16 by v_perm (selector
            // 0x0c gives a zero byte)
            const uint32_t hb = 31u - (uint32_t)__builtin_clz(m | 1u);
            const uint32_t sel = (hb & 7u) | 0x0C0C0C00u;
            const uint32_t lo = __builtin_amdgcn_perm(d.y, d.x, sel);
            const uint32_t hi = __builtin_amdgcn_perm(d.w, d.z, sel);
            // the nearest lane of the row with a start, as the maximum over
            // the lanes up to this one of (lane, value)
            uint32_t x = m ? lane_key | (hb & 8u ? hi : lo) : 0u;
            x = max(x, row_shr<1>(x));
            x = max(x, row_shr<2>(x));
            x = max(x, row_shr<4>(x));
            x = max(x, row_shr<8>(x));
            // word by word: each byte from the last start in the word, else the
            // previous word's last byte (the value entering the lane for word 0)
            uint32_t prev = row_shr<1>(x) << 24;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              prev = __builtin_amdgcn_perm(prev, dv[i], fill_sel[(m >> (4 * i)) & 0xFu]);
              win[k][i] = prev;
            }
          }
        }
        // clear this round's start bits: word q0 / 32 is read only by this
        // lane and its neighbour in the same wave, which have both read it
        if ((tid & 1) == 0) {
#pragma unroll
          for (int i = 0; i < kValPlanes; ++i) starts[i][q0 >> 5] = 0;
        }
        block_bad = uniform(*bad_flag) != 0;
        runmask = later;
        if (runmask) __syncthreads();   // the values are read
      } while (runmask);
      if (block_bad) {   // uniform
        if (tid == 0) a.status[s] = CMP_ECORRUPT;
        continue;
      }
    }

    // ---- write the pixels (row-major over the ROI), colour, then depth: byte
    // k of pixel 4 i + j is byte j of plane k's word i (a 4 x 4 byte transpose
    // per word). A lane holds 16 consecutive pixels, but stores are issued so
    // that consecutive lanes write consecutive 16-byte quads: the wave's 1024
    // pixels are restaged through LDS (the wave's quarter of every plane's run
    // values, which only this wave reads), and in store v lane i writes pixels
    // 256 v + 4 i .. + 3 of the wave's range (16-byte stores at a 64-byte lane
    // stride cost four times the memory requests).
    const int qw = (kBlock / 4) * wave + 4 * lane;   // block pixel of store 0
    // the block's origin: the frame's top left, or its ROI's position there
    const int64_t org = a.at_roi ? (int64_t)(int32_t)h[2] * I.pitch + (int32_t)h[1] : 0;
    // the quad's row and column, by a 32-bit division (of the pixel's place in
    // the block's first row where the ROI has 2^32 pixels or more)
    const uint32_t urw = (uint32_t)rw;
    uint32_t y0 = 0, px = (uint32_t)b * kBlock;
    if (npx >> 32) {   // uniform
      y0 = (uint32_t)uniform((int)((int64_t)b * kBlock / rw));
      px = (uint32_t)((int64_t)b * kBlock - (int64_t)y0 * rw);
    }
    px += (uint32_t)qw;
    const uint32_t y = px / urw;
    const uint32_t x0 = px - y * urw;
    const int64_t jump = I.pitch - (int64_t)rw;   // from a row's end to the next row
    const int64_t o0 = org + (int64_t)(y0 + y) * I.pitch + x0;
    const bool swizzled = (h[5] >> 8) & 1u;
    uint8_t* wbase = vals + (kBlock / 4) * wave;
    // quad q of the wave (pixels 4 q ..) sits in piece q / 64 at slot
    // swz(q % 64): within each group of 8 slots (128 bytes, all banks) the
    // slots rotate by the group index, so that the 8 lanes served together
    // hit 8 different 16-byte bank groups both when lane L writes its quads
    // 4 L + c and when lane i reads quad 64 v + i
    auto swz = [](int x) { return (x & ~7) | ((x + (x >> 3)) & 7); };
    auto write_words = [&](const u32x4& w0, const u32x4& w1, const u32x4& w2, const u32x4& w3,
                           uint32_t* __restrict__ dst, bool unswizzle) {
      uint8_t* wl = wbase + (lane / 16) * kBlock;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t p0, p1, p2, p3;
        transpose4x4(w0[i], w1[i], w2[i], w3[i], p0, p1, p2, p3);
        if (unswizzle) {   // uniform
          p0 = swizzle_bits(p0);
          p1 = swizzle_bits(p1);
          p2 = swizzle_bits(p2);
          p3 = swizzle_bits(p3);
        }
        *reinterpret_cast<u32x4*>(wl + 16 * swz((4 * lane + i) % 64)) = u32x4{p0, p1, p2, p3};
      }
      __builtin_amdgcn_wave_barrier();
      u32x4 q[4];
#pragma unroll
      for (int v = 0; v < 4; ++v)
        q[v] = *reinterpret_cast<const u32x4*>(wbase + v * kBlock + 16 * swz(lane));
      __builtin_amdgcn_wave_barrier();
      int64_t o = o0;
      uint32_t xx = x0;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int qq = qw + (kBlock / 16) * v;
        const uint32_t left = urw - xx;   // pixels up to the row's end
        if (qq + 4 <= c.len && left >= 4u) {
          st_u32x4_nt(dst + o, q[v]);
        } else if (qq < c.len) {   // a quad at the end of a row or of the block
          if (urw >= 4u) {         // uniform: at most one row's end in it
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (qq + j < c.len) dst[o + j + ((uint32_t)j >= left ? jump : 0)] = q[v][j];
          } else {
            int64_t oj = o;
            uint32_t xj = xx;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              if (qq + j < c.len) {
                dst[oj] = q[v][j];
                ++oj;
                if (++xj == urw) {
                  xj = 0;
                  oj += jump;
                }
              }
            }
          }
        }
        // advance 256 pixels
        xx += kBlock / 16;
        o += kBlock / 16;
        if (urw >= (uint32_t)(kBlock / 16)) {   // uniform: at most one row's end
          if (xx >= urw) {
            xx -= urw;
            o += jump;
          }
        } else {
          const uint32_t rows = xx / urw;
          xx -= rows * urw;
          o += (int64_t)rows * jump;
        }
      }
    };
    write_words(win[0], win[1], win[2], win[3], I.color, swizzled);
    if (c.np == 8) write_words(win[4], win[5], win[6], win[7], I.depth, false);
  }
}

// Workgroups of `kernel` that fit on the device at once, at most `cap` per
// compute unit when cap > 0 (the per-unit occupancy is cached per device).
int resident_groups(const void* kernel, std::atomic<int>* cache, int cap) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 1024;
  int packed = cache[dev].load(std::memory_order_relaxed);
  if (packed <= 0) {
    int cus = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kThreads, 0) != hipSuccess ||
        cus <= 0 || per_cu <= 0)
      return 1024;
    packed = cus * 256 + per_cu;   // both fit: cus < 2^23, per_cu < 256
    cache[dev].store(packed, std::memory_order_relaxed);
  }
  const int cus = packed / 256, per_cu = packed % 256;
  return cus * (cap > 0 && cap < per_cu ? cap : per_cu);
}
static std::atomic<int> g_compress_groups[64], g_decompress_groups[64];
// Caps on the workgroups per compute unit (0: as many as fit).
static std::atomic<int> g_compress_cap{0}, g_decompress_cap{0};
// Look-back polls before a compressing block gives up (negative: the default).
constexpr uint32_t kDefaultWaitLimit = 1u << 20;
static std::atomic<int32_t> g_wait_limit{-1};
uint32_t rle_wait_limit() {
  const int32_t wl = g_wait_limit.load(std::memory_order_relaxed);
  return wl < 0 ? kDefaultWaitLimit : (uint32_t)wl;
}
int rle_compress_cap() { return g_compress_cap.load(std::memory_order_relaxed); }

// Look-back flags: one per block of each image's largest possible ROI.
int64_t rle_flag_count(const cmp_image* imgs, int32_t n) {
  int64_t f = 0;
  for (int i = 0; i < n; ++i) {
    const int64_t npx = (int64_t)(imgs[i].roi.w > 0 ? imgs[i].roi.w : 0) *
                        (imgs[i].roi.h > 0 ? imgs[i].roi.h : 0);
    const int64_t nb = (int64_t)rle_nblocks(npx);
    f += nb ? nb : 1;
  }
  return f;
}

// Scratch memory of cmp_rle_compress_noalloc: the tickets and look-back
// flags that cmp_rle_compress keeps in the caller's workspace. Each device
// holds its own copy until the process ends. Host code never passes this
// name to a kernel (on the host it is only a stand-in for the symbol): it
// passes the device address that hipGetSymbolAddress returns for the
// current device, looked up once per device and kept in g_scratch_ptr.
static_assert(CMP_RLE_SCRATCH_BYTES == kTicketBytes + kCtlBytes + 8 * 131072,
              "the scratch holds the tickets, the control words and 131072 look-back flags");
static __device__ __align__(256) uint8_t scratch[CMP_RLE_SCRATCH_BYTES];
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[64];

// The current device's address of `scratch` (nullptr, with the error set,
// if it cannot be found).
static void* scratch_address() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    set_error("no current HIP device (or more than 64 devices)");
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      set_error("hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
      return nullptr;
    }
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

}  // namespace cmp

using namespace cmp;

extern "C" size_t cmp_rle_max_size(int32_t w, int32_t h, int32_t nplanes) {
  if (w < 0 || h < 0 || nplanes <= 0) return 0;
  const int64_t npx = (int64_t)w * h;
  const uint64_t nb = rle_nblocks(npx);
  uint64_t total = rle_p0(nb, nplanes);
  if (nb) total += (nb - 1) * align16((uint64_t)kBlock * nplanes) +
                   align16((uint64_t)(npx - (int64_t)(nb - 1) * kBlock) * nplanes);
  return (size_t)total;
}

extern "C" size_t cmp_rle_workspace_size(const cmp_image* imgs, int32_t n) {
  if (n < 0 || (n > 0 && !imgs)) return 0;
  return kTicketBytes + kCtlBytes + (size_t)(8 * rle_flag_count(imgs, n));
}

namespace cmp {

cmp_status rle_compress_prepare(const cmp_image* imgs, int32_t n, const int32_t* roi_dev,
                                uint8_t* const* out, const uint64_t* capacity,
                                uint64_t* out_size_dev, int32_t* status_dev, void* workspace,
                                size_t ws_bytes, size_t (*max_size)(int32_t, int32_t, bool),
                                RleCArgs& a, int64_t& grid) {
  CMP_REQUIRE(imgs && out && capacity && out_size_dev && status_dev && workspace, "NULL argument");
  CMP_REQUIRE(((uintptr_t)roi_dev & 15) == 0 && ((uintptr_t)workspace & 15) == 0 &&
                  ((uintptr_t)out_size_dev & 7) == 0 && ((uintptr_t)status_dev & 3) == 0,
              "roi_dev/workspace must be 16-byte, out_size_dev 8-byte and status_dev "
              "4-byte aligned");
  memset(&a, 0, sizeof a);
  int64_t nflags = 0;
  grid = 0;
  for (int i = 0; i < n; ++i) {
    const cmp_image& I = imgs[i];
    CMP_REQUIRE(rect_valid(I.roi), "imgs[%d] has a negative size", i);
    const int W = rect_empty(I.roi) ? 0 : I.roi.w, H = rect_empty(I.roi) ? 0 : I.roi.h;
    if (W > 0) {
      CMP_REQUIRE(I.color, "imgs[%d].color is NULL", i);
      CMP_REQUIRE(I.pitch >= W, "imgs[%d].pitch < width", i);
      CMP_REQUIRE(((uintptr_t)I.color & 3) == 0 && ((uintptr_t)I.depth & 3) == 0,
                  "imgs[%d]: buffers must be 4-byte aligned", i);
    }
    CMP_REQUIRE(out[i] && ((uintptr_t)out[i] & 15) == 0, "out[%d] must be 16-byte aligned", i);
    const size_t need = max_size(W, H, I.depth != nullptr);
    CMP_REQUIRE(need < (1ull << 32), "image %d too large for 32-bit stream offsets", i);
    if (capacity[i] < need) {
      set_error("capacity[%d] = %llu < %zu", i, (unsigned long long)capacity[i], need);
      return CMP_ENOSPC;
    }
    const int64_t nb = (int64_t)rle_nblocks((int64_t)W * H);
    a.im[i] = RleCImg{(const uint32_t*)I.color, I.depth, I.pitch, W, H, out[i], (int32_t)nflags, 0};
    nflags += nb ? nb : 1;
    grid += nb ? nb : 1;
  }
  CMP_REQUIRE(grid < (1ll << 24), "too many blocks");
  const size_t need = kTicketBytes + kCtlBytes + (size_t)(8 * nflags);
  if (ws_bytes < need) {
    set_error("workspace of %zu bytes is smaller than %zu", ws_bytes, need);
    return CMP_ENOSPC;
  }
  a.roi_dev = roi_dev;
  a.out_size = out_size_dev;
  a.status = status_dev;
  a.tickets = (uint32_t*)workspace;
  a.ctl = (uint32_t*)((uint8_t*)workspace + kTicketBytes);
  a.flags = (uint64_t*)((uint8_t*)workspace + kTicketBytes + kCtlBytes);
  a.nflags = (int32_t)nflags;
  a.n = n;
  a.wait_limit = rle_wait_limit();
  return CMP_OK;
}

}  // namespace cmp

static size_t rle1_max_size(int32_t w, int32_t h, bool depth) {
  return cmp_rle_max_size(w, h, depth ? 8 : 4);
}

extern "C" cmp_status cmp_rle_compress(const cmp_image* imgs, int32_t n, cmp_format fmt,
                                       uint32_t flags, const int32_t* roi_dev, uint8_t* const* out,
                                       const uint64_t* capacity, uint64_t* out_size_dev,
                                       int32_t* status_dev, void* workspace, size_t ws_bytes,
                                       void* stream) {
  CMP_RANGE("cmp_rle_compress");
  CMP_REQUIRE(n >= 0 && n <= kRleMax, "n = %d must be 0..%d", n, kRleMax);
  if (n == 0) return CMP_OK;
  if (fmt != CMP_RGBA8) {
    set_error("RLE compression handles RGBA8 (+ depth) pixels");
    return CMP_EUNSUPPORTED;
  }
  CMP_REQUIRE((flags & ~CMP_RLE_SWIZZLE) == 0, "unknown flags 0x%x", flags);
  RleCArgs a;
  int64_t grid = 0;
  hipStream_t s = (hipStream_t)stream;
  const cmp_status st = rle_compress_prepare(imgs, n, roi_dev, out, capacity, out_size_dev,
                                             status_dev, workspace, ws_bytes, rle1_max_size, a,
                                             grid);
  if (st != CMP_OK) return st;
  a.swizzle = (flags & CMP_RLE_SWIZZLE) ? 1 : 0;
  // one wave of workgroups at most: more would find the tickets drawn
  // (both instances have the same resources, so one occupancy serves both)
  const int64_t cap = resident_groups((const void*)rle_compress_kernel<false>, g_compress_groups,
                                      rle_compress_cap());
  const dim3 grid_dim((unsigned)(grid < cap ? grid : cap));
  log_plan("rle compress: %d images, %lld block slots, %u resident workgroups%s", n,
           (long long)grid, grid_dim.x, a.swizzle ? ", swizzled" : "");
  if (a.swizzle)
    hipLaunchKernelGGL(rle_compress_kernel<true>, grid_dim, dim3(kThreads), 0, s, a);
  else
    hipLaunchKernelGGL(rle_compress_kernel<false>, grid_dim, dim3(kThreads), 0, s, a);
  CMP_CHECK_HIP(hipGetLastError());
  return CMP_OK;
}

extern "C" cmp_status cmp_rle_compress_noalloc(const cmp_image* imgs, int32_t n, cmp_format fmt,
                                               uint32_t flags, const int32_t* roi_dev,
                                               uint8_t* const* out, const uint64_t* capacity,
                                               uint64_t* out_size_dev, int32_t* status_dev,
                                               void* stream) {
  CMP_RANGE("cmp_rle_compress_noalloc");
  CMP_REQUIRE(n >= 0 && n <= kRleMax, "n = %d must be 0..%d", n, kRleMax);
  if (n == 0) return CMP_OK;
  CMP_REQUIRE(imgs, "imgs is NULL");
  for (int i = 0; i < n; ++i)
    CMP_REQUIRE(rect_valid(imgs[i].roi), "imgs[%d] has a negative size", i);
  const size_t need = cmp_rle_workspace_size(imgs, n);
  if (need > CMP_RLE_SCRATCH_BYTES) {
    set_error("these images need %zu bytes of scratch; the static maximum is %zu "
              "(131072 blocks of 4096 pixels): use cmp_rle_compress with a workspace",
              need, (size_t)CMP_RLE_SCRATCH_BYTES);
    return CMP_ENOSPC;
  }
  void* ws = scratch_address();
  if (!ws) return CMP_EHIP;
  return cmp_rle_compress(imgs, n, fmt, flags, roi_dev, out, capacity, out_size_dev, status_dev,
                          ws, CMP_RLE_SCRATCH_BYTES, stream);
}

extern "C" cmp_status cmp_rle_set_wait_limit(int32_t polls) {
  g_wait_limit.store(polls < 0 ? -1 : polls, std::memory_order_relaxed);
  return CMP_OK;
}

extern "C" cmp_status cmp_rle_set_groups_per_cu(int32_t compress, int32_t decompress) {
  CMP_REQUIRE(compress >= 0 && decompress >= 0, "caps must be >= 0 (0: as many as fit)");
  g_compress_cap.store(compress, std::memory_order_relaxed);
  g_decompress_cap.store(decompress, std::memory_order_relaxed);
  return CMP_OK;
}

static cmp_status rle_decompress_impl(const uint8_t* const* in, const uint64_t* in_bytes,
                                      int32_t n, const cmp_image* out, int32_t* roi_out_dev,
                                      int32_t* status_dev, bool at_roi, void* stream) {
  CMP_REQUIRE(n >= 0 && n <= kRleMax, "n = %d must be 0..%d", n, kRleMax);
  if (n == 0) return CMP_OK;
  CMP_REQUIRE(in && in_bytes && out && status_dev, "NULL argument");
  CMP_REQUIRE(((uintptr_t)roi_out_dev & 15) == 0 && ((uintptr_t)status_dev & 3) == 0,
              "roi_out_dev must be 16-byte aligned");
  RleDArgs a;
  memset(&a, 0, sizeof a);
  int64_t grid = 0;
  for (int i = 0; i < n; ++i) {
    const cmp_image& O = out[i];
    CMP_REQUIRE(in[i] && ((uintptr_t)in[i] & 15) == 0, "in[%d] must be 16-byte aligned", i);
    CMP_REQUIRE(rect_valid(O.roi), "out[%d] has a negative size", i);
    const int W = rect_empty(O.roi) ? 0 : O.roi.w, H = rect_empty(O.roi) ? 0 : O.roi.h;
    if (W > 0) {
      CMP_REQUIRE(O.color && O.pitch >= W, "out[%d]: NULL colour or pitch < width", i);
      CMP_REQUIRE(((uintptr_t)O.color & 3) == 0 && ((uintptr_t)O.depth & 3) == 0,
                  "out[%d]: buffers must be 4-byte aligned", i);
    }
    const int64_t nb = (int64_t)rle_nblocks((int64_t)W * H);
    a.im[i] = RleDImg{in[i], in_bytes[i], (uint32_t*)O.color, (uint32_t*)O.depth, O.pitch, W, H};
    grid += nb ? nb : 1;
  }
  CMP_REQUIRE(grid < (1ll << 24), "too many blocks");
  a.roi_out = roi_out_dev;
  a.status = status_dev;
  a.n = n;
  a.at_roi = at_roi ? 1 : 0;
  const int64_t cap = resident_groups((const void*)rle_decompress_kernel, g_decompress_groups,
                                      g_decompress_cap.load(std::memory_order_relaxed));
  log_plan("rle decompress: %d streams, at most %lld blocks, %lld resident workgroups%s", n,
           (long long)grid, (long long)(grid < cap ? grid : cap), at_roi ? ", at the ROIs" : "");
  hipLaunchKernelGGL(rle_decompress_kernel, dim3((unsigned)(grid < cap ? grid : cap)),
                     dim3(kThreads), 0, (hipStream_t)stream, a);
  CMP_CHECK_HIP(hipGetLastError());
  return CMP_OK;
}

extern "C" cmp_status cmp_rle_decompress(const uint8_t* const* in, const uint64_t* in_bytes,
                                         int32_t n, const cmp_image* out, int32_t* roi_out_dev,
                                         int32_t* status_dev, void* stream) {
  CMP_RANGE("cmp_rle_decompress");
  return rle_decompress_impl(in, in_bytes, n, out, roi_out_dev, status_dev, false, stream);
}

extern "C" cmp_status cmp_rle_decompress_at_roi(const uint8_t* const* in,
                                                const uint64_t* in_bytes, int32_t n,
                                                const cmp_image* out, int32_t* roi_out_dev,
                                                int32_t* status_dev, void* stream) {
  CMP_RANGE("cmp_rle_decompress_at_roi");
  return rle_decompress_impl(in, in_bytes, n, out, roi_out_dev, status_dev, true, stream);
}
