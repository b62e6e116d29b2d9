// Filter_s (Eq. 4) of Key channel vectors, from lists of candidates collected while the tensor streams by.
//
// A block takes 8 or 16 neighbouring channels of one slab.  Reading such a column costs a whole 128-byte line per 16 or 32
// bytes between the CU's first-level cache and the L2, so the column should be read once, and a vector of thousands of
// tokens is best not kept: of its entries only a few per cent can belong to S.  So
//   1. the segment is cut into up to 2048 stretches of L rows (4096 with 8 channels per block, and up to 4096 tokens); one row of each
//      gives every channel a rough threshold per end: the j-th most extreme of the extremes of groups of eight or sixteen sampled
//      entries (gear_select_ext.h), with j far enough above the number of wanted entries that are expected in the sample (stream_plan).
//      With L = 1 the sample is the whole segment, and the threshold holds for certain;
//   2. the sample, which is still in registers, and then the other rows of the stretches are looked at once; what passes a rough
//      threshold goes onto its channel's list in LDS;
//   3. one wave per channel ranks its list exactly, index and all, and leaves the selected entries as bits in LDS, whence the
//      mask is stored.
// A channel whose list overflows (many entries at a threshold), or holds fewer entries than are wanted, is selected by stream_way_out.
//
// 64 x 8 slabs x 8192 tokens at 2 %, one wave per vector in registers before: 609 -> 440 us.  Of those the sample and the thresholds
// take 80, the rest of the read 230 (four 32-byte pieces per line: the first-level cache takes in 32 bytes per cycle and CU, which is
// 220 us), the appending 60, the ranking 60, the mask 20.  32 slabs x 32768 (8 channels per block) 268 -> 146, in blocks of 16
// channels and 1024 threads, one per CU, 35 less (32 channels in such a block, half the bytes through the first-level cache again: 512 slabs x
// 8192 25 us more, 512 x 4096 67 more, one block's phases lie bare), 280 x 1777 92 -> 62,
// 512 x 4096 261 -> 203.  As three kernels (sample; candidates from whole rows into the workspace; ranking) 72 + 255 + 108: no gain.
#pragma once
#include "gear_internal.h"
#include "gear_select.h"
#include "gear_select_ext.h"

namespace gear {

constexpr int STREAM_BITS = 11;                      // resolution of the rough thresholds (1/32 of an octave)
// T: threads of a block, 512 or 1024; PC: 16-byte pieces of a row it takes
__host__ __device__ constexpr int stream_rows(int pc, int t) { return t / pc; }   // rows a block reads side by side
__host__ __device__ constexpr int stream_wave_channels(int pc, int t) { return 8 * pc / (t / 64); }   // channels that a wave ranks
constexpr int STREAM_BATCH = 4;                      // rows of a thread in flight, in the passes of the way out
constexpr int STREAM_WALK = 16;                      // its ordered walk takes 64 times as many rows at a time
struct StreamState {   // per channel, in LDS; [2]: of the top, of the bottom
  // The way out, with the bottom's keys as their complements: the need-th largest key is one of base .. base + width - 1; width 0: found, or
  // not in work.  shift: from a key's offset to its counter.  range: (base | shift << 16, width) of either end; before that x and z are
  // estimates of the threshold, and channel 0's w says whether some channel has usable rough thresholds
  uint4 range;
  uint32_t cnt;               // entries on the list
  uint32_t fail;              // 1: the channel takes the way out
  uint32_t kmx, kmn;          // the extremes of what is not selected (kmn: complement)
  union {
    uint32_t rough[2];        // the rough thresholds (0x10000: none)
    uint32_t need[2];         // the way out
  };
  uint32_t equal[2];          // the way out: the entries at the threshold; which of them are taken (EQUAL_..) << 16
};
static_assert(sizeof(StreamState) == 48, "part of the LDS that stream_plan counts");
// Decodes a 1-D grid of ncb * nslab blocks, one per slab and block of channels.  Consecutive block ids go round-robin to
// the chip's 8 XCDs (each with its own L2), so the id is decoded with the column block fastest INSIDE one XCD: the blocks
// that share the 128-byte lines of one slab (of its rows, of its mask) then meet in one L2 instead of eight.  The up to
// seven slabs past a multiple of eight go to all XCDs.  231 slabs x 3000 tokens, which went to all XCDs as a whole before:
// 245 -> 106 us.
__device__ __forceinline__ void slab_and_column_block(int i, int nslab, int ncb, int& slab, int& cb) {
  const int even = (nslab & ~7) * ncb;
  if (i < even) {
    const int xcd = i & 7, j = i >> 3;
    cb = j % ncb;
    slab = (j / ncb) * 8 + xcd;
  } else {
    cb = i % ncb;
    slab = i / ncb;
  }
}

// The column of a block: its rows' pieces of 16 bytes, one per thread and row.
struct StreamColumn {
  GEAR_BUF_T buf;   // ends with the last row's piece of the block: rows past n read as 0
  int n, pc, slot;  // the thread's piece of a row, its row among those read side by side
  __device__ __forceinline__ uint4 load(int row) const { return GEAR_BUF_LOAD16(buf, row * (D * 2) + pc * 16); }
};
// f(pieces, row of the first, rows from one to the next) for the rows of the thread, a batch at a time (rows past n are 0)
template <int PC, int T, class F>
__device__ __forceinline__ void for_each_batch(const StreamColumn& col, F&& f) {
  constexpr int RS = stream_rows(PC, T);
#pragma unroll 1
  for (int base = col.slot; base < col.n; base += RS * STREAM_BATCH) {
    uint4 v[STREAM_BATCH];
#pragma unroll
    for (int i = 0; i < STREAM_BATCH; ++i) v[i] = col.load(base + i * RS);
    f(v, base, RS);
  }
}
template <int PC>
__device__ __forceinline__ void mark_bit(uint32_t* bits, uint32_t row, uint32_t ch) {   // byte PC row + ch / 8, bit ch % 8
  const uint32_t byte = row * PC + (ch >> 3);
  atomicOr(&bits[byte >> 2], 1u << ((byte & 3u) * 8u + (ch & 7u)));
}

// Ranks a channel's list (total entries, row | fp16 value << 16).  Returns false where it does not hold enough entries (one more
// than are wanted where the extremes of the rest are asked for), and where it holds only the first of more candidates: k_top and k_bot are
// then their shares, and kmx, kmn come back as estimates of the threshold keys (of the bottom: the complement).  Called by a whole wave.
template <int R, int PC>
__device__ __forceinline__ bool stream_rank(uint32_t* list, uint32_t total, int k_top, int k_bot, uint32_t tt, uint32_t tb, uint32_t ch,
                                            uint32_t* bits, int rows, bool rest, bool part, uint32_t& kmx, uint32_t& kmn) {
  const int lane = lane_id();
  uint32_t c[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const uint32_t p = (uint32_t)(lane + 64 * i);
    c[i] = 0u;
    if (p < total) {
      const uint32_t e = list[p];
      c[i] = key16(e >> 16) << 16 | (0xFFFFu - (e & 0xFFFFu));
    }
  }
  auto enough = [&](uint32_t rough, int k) {
    uint32_t n = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) n += (uint32_t)__popcll(__ballot(c[i] >= rough << 16));
    return n >= (uint32_t)(k + (rest ? 1 : 0));
  };
  auto flip = [&]() {   // to the composites that grow towards the bottom, and back
#pragma unroll
    for (int i = 0; i < R; ++i) c[i] = c[i] != 0u ? c[i] ^ 0xFFFF0000u : 0u;
  };
  kmx = kmn = 0u;
  if (k_top > 0 && !enough(tt, k_top)) return false;
  const uint32_t xt = k_top > 0 ? wave_kth_by_bins<R>(c, (uint32_t)k_top, tt, list, rows, part) : 0xFFFFFFFFu;
  flip();
  if (k_bot > 0 && !enough(tb, k_bot)) return false;
  const uint32_t xb = k_bot > 0 ? wave_kth_by_bins<R>(c, (uint32_t)k_bot, tb, list, rows, part) : 0xFFFFFFFFu;
  if (__builtin_expect(part, 0)) {
    kmx = xt >> 16;
    kmn = xb >> 16;
    return false;
  }
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const uint32_t t = c[i] ^ 0xFFFF0000u;
    if (c[i] != 0u) {
      if (t >= xt || c[i] >= xb) mark_bit<PC>(bits, 0xFFFFu - (c[i] & 0xFFFFu), ch);
      else {
        kmx = max(kmx, t >> 16);
        kmn = max(kmn, c[i] >> 16);
      }
    }
  }
  return true;
}

// The selection of the channels marked in st[].fail, for inputs whose thresholds are shared by many entries and for the rare channel
// whose list came out too long or too short.  Passes over the column:
//   1  an estimate of each threshold (of the full list's entries, or the sample's; rather too near than too far out) is counted: the
//      entries beyond it and those not as far out, and the nearest value beyond it, which is taken next.  Where many entries share the
//      threshold it is mostly the estimate itself.  90 instructions per row piece, where a histogram takes 360;
//   2  for what is not found in STREAM_PROBES passes, and for the few channels of a block that are not tied, histograms of the keys:
//      32 keys per counter (256 where the rough threshold was no bound), then single keys.  A counter holds the top's count in its lower half
//      and the bottom's in the upper one (at most 32768 rows); a channel that is not searched costs nothing;
//   3  the bits of the entries beyond the thresholds.  Where only some of the entries at a threshold are wanted, those of the lowest
//      rows are: up to STREAM_FEW of them are listed in this pass and ranked;
//   4  where they are more, one wave per channel walks the rows in order until it has as many as it needs.
// Until there were estimates it took a histogram over a byte of the composite (key, row) per pass and end, up to nine passes.  A call at rank
// 0 and 2 %, one wave per vector in registers -> nine passes -> now: 16 x 8 slabs x 8192 tokens, all Keys equal 1184 -> 1281 -> 632 us,
// clamped to 1.2 standard deviations 522 -> 939 -> 537, clamped at 0 from below 783 -> 1003 -> 858; clamped to 1.2, 256 x 3000 363 -> 747 ->
// 428, 1280 x 1100 662 -> 1508 -> 934, 8 x 32768 (from a channel-major copy) 247 -> 619 -> 254, 2 x 9001 70 -> 295 -> 114; multiples of
// 1/4, 8 x 32768 231 -> 598 -> 348.  What is left of a call of few blocks is the chain of a block's passes, 7 to 15 us each.
constexpr uint32_t STREAM_FEW = 64;
constexpr int STREAM_PROBES = 3;
constexpr uint32_t STREAM_ALONE = 2;   // so many channels of a block go by histograms at once
enum : uint32_t { EQUAL_NONE = 0, EQUAL_ALL, EQUAL_LISTED, EQUAL_WALK };   // which of the entries at a threshold are taken
template <int PC, int T>
__device__ __forceinline__ void stream_way_out(const StreamColumn& usual, StreamState* st, uint32_t* hist /* [8 PC][256] */, uint32_t* bits,
                                               int k_top, int k_bot, bool rest) {
  constexpr int CW = stream_wave_channels(PC, T);
  int tid = threadIdx.x;
  GEAR_PIN_VGPR(tid);   // (nothing made from it is kept over the usual way)
  const int wave = GEAR_WAVE_UNIFORM(tid >> 6), lane = tid & 63, ch0 = tid % PC * 8;
  const StreamColumn col{usual.buf, usual.n, tid % PC, tid / PC};
  uint32_t* count = hist;               // [4 PC][2][2]: entries beyond the estimate, entries not as far out; two channels per word
  uint32_t* near = hist + 16 * PC;      // [8 PC][2]: the nearest value beyond it (complement)
  uint32_t failed = 0u;
  for (int i = 0; i < 8 * PC; ++i) failed += st[i].fail;
  if (tid < 8 * PC) {
    StreamState& s = st[tid];
    uint32_t* range = reinterpret_cast<uint32_t*>(&s.range);
    const uint32_t rough[2] = {s.rough[0], s.rough[1]}, k[2] = {(uint32_t)k_top, (uint32_t)k_bot};
    s.cnt = 0u;                         // the ends whose estimate is to be counted
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      s.need[d] = s.fail ? k[d] : 0u;
      if (s.need[d] == 0u) range[2 * d] = range[2 * d + 1] = 0u;
      else if (failed > STREAM_ALONE) {
        s.cnt |= 1u << d;
        range[2 * d + 1] = 0u;
      } else {
        range[2 * d] = rough[d] < 0x10000u ? rough[d] | 5u << 16 : 8u << 16;
        range[2 * d + 1] = rough[d] < 0x10000u ? 0x10000u - rough[d] : 0x10000u;
      }
    }
    if (s.fail) s.kmx = s.kmn = 0u;
  }
#pragma unroll 1
  for (int pass = 0; pass < STREAM_PROBES; ++pass) {
    block_lds_sync();
    uint32_t probed = 0u;
    for (int i = 0; i < 8 * PC; ++i) probed |= st[i].cnt;
    for (int i = tid; i < 32 * PC; i += T) hist[i] = 0u;
    uint32_t at[2][4], above[2][4], below[2][4], next[2][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const StreamState &a = st[ch0 + 2 * j], &b = st[ch0 + 2 * j + 1];
      at[0][j] = (a.range.x & 0xFFFFu) | b.range.x << 16;
      at[1][j] = (a.range.z & 0xFFFFu) | b.range.z << 16;
#pragma unroll
      for (int d = 0; d < 2; ++d) above[d][j] = below[d][j] = next[d][j] = 0u;
    }
    block_lds_sync();
    if (GEAR_WAVE_UNIFORM((int)probed) == 0) break;   // the same in every thread of the block
    for_each_batch<PC, T>(col, [&](const uint4 (&v)[STREAM_BATCH], int row, int step) {
#pragma unroll
      for (int i = 0; i < STREAM_BATCH; ++i) {
        if (row + i * step >= col.n) continue;
        const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t k = key16x2(w[j]);
#pragma unroll
          for (int d = 0; d < 2; ++d) {
            const uint32_t x = d == 0 ? k : ~k, over = nonzero_u16x2(sub_sat_u16x2(x, at[d][j])), under = nonzero_u16x2(sub_sat_u16x2(at[d][j], x));
            above[d][j] += over;   // (no carry: at most 32768)
            below[d][j] += under;
            next[d][j] = max_u16x2(next[d][j], ~x & neg_u16x2(over));
          }
        }
      }
    });
    // over the lanes of a row of 16 that hold the same piece, then in LDS
    auto row_sum = [](uint32_t x) {
      if constexpr (PC == 1) x += dpp_u<DPP_XOR1>(x);
      x += dpp_u<DPP_XOR2>(x);
      x += dpp_u<DPP_ROR4>(x);
      return x + dpp_u<DPP_ROR8>(x);
    };
    auto row_max = [](uint32_t x) {
      if constexpr (PC == 1) x = max_u16x2(x, dpp_u<DPP_XOR1>(x));
      x = max_u16x2(x, dpp_u<DPP_XOR2>(x));
      x = max_u16x2(x, dpp_u<DPP_ROR4>(x));
      return max_u16x2(x, dpp_u<DPP_ROR8>(x));
    };
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        const uint32_t a = row_sum(above[d][j]), b = row_sum(below[d][j]), x = row_max(next[d][j]);
        if ((lane & 15) < PC) {
          uint32_t* c = count + 4 * (4 * col.pc + j) + 2 * d;
          uint32_t* y = near + 2 * (ch0 + 2 * j) + d;
          atomicAdd(&c[0], a);
          atomicAdd(&c[1], b);
          atomicMax(&y[0], x & 0xFFFFu);
          atomicMax(&y[2], x >> 16);
        }
      }
    block_lds_sync();
    if (tid < 8 * PC) {
      StreamState& s = st[tid];
      uint32_t* range = reinterpret_cast<uint32_t*>(&s.range);
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        if ((s.cnt >> d & 1u) == 0u) continue;
        const uint32_t* c = count + 4 * (tid >> 1) + 2 * d;
        const uint32_t beyond = (c[0] >> (16 * (tid & 1))) & 0xFFFFu, from = (uint32_t)col.n - ((c[1] >> (16 * (tid & 1))) & 0xFFFFu);
        if (beyond < s.need[d] && from >= s.need[d]) {   // it is the threshold
          s.cnt &= ~(1u << d);
          s.need[d] -= beyond;
          s.equal[d] = from - beyond;
        } else if (from >= s.need[d] && pass < STREAM_PROBES - 1) {
          range[2 * d] = 0xFFFFu - near[2 * tid + d];
        } else {
          s.cnt &= ~(1u << d);
          range[2 * d + 1] = from >= s.need[d] ? 0xFFFFu - range[2 * d] : 0x10000u;
          range[2 * d] = from >= s.need[d] ? (range[2 * d] + 1u) | 5u << 16 : 8u << 16;
        }
      }
    }
  }
  // (an end takes at most three passes: by 32 keys, by 256 if these were not it or did not reach, and by single ones)
#pragma unroll 1
  for (int pass = 0; pass < 4; ++pass) {
    block_lds_sync();
    uint32_t searched = 0u;
    for (int i = 0; i < 8 * PC; ++i) searched |= st[i].range.y | st[i].range.w;
    for (int i = tid; i < 8 * PC * 256; i += T) hist[i] = 0u;
    block_lds_sync();
    if (GEAR_WAVE_UNIFORM((int)searched) == 0) break;   // the same in every thread of the block
    for_each_batch<PC, T>(col, [&](const uint4 (&v)[STREAM_BATCH], int row, int step) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint4 rg = st[ch0 + e].range;
        if ((rg.y | rg.w) == 0u) continue;   // (mostly the same in all lanes)
        uint32_t key[STREAM_BATCH];
#pragma unroll
        for (int i = 0; i < STREAM_BATCH; ++i) key[i] = key16(half_of(v[i].x, v[i].y, v[i].z, v[i].w, e));
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          uint32_t* h = hist + (ch0 + e) * 256;
          const uint32_t from = d == 0 ? rg.x : rg.z, width = d == 0 ? rg.y : rg.w;
          uint32_t run = 0u, len = 0u;
          if (width == 0u) continue;
#pragma unroll
          for (int i = 0; i < STREAM_BATCH; ++i) {
            const uint32_t off = (d == 0 ? key[i] : 0xFFFFu - key[i]) - (from & 0xFFFFu);
            if (off < width && row + i * step < col.n) {
              const uint32_t bin = min(off >> (from >> 16), 255u);
              if (bin != run && len != 0u) {
                atomicAdd(&h[run], len);
                len = 0u;
              }
              run = bin;
              len += d == 0 ? 1u : 0x10000u;
            }
          }
          if (len != 0u) atomicAdd(&h[run], len);
        }
      }
    });
    block_lds_sync();
#pragma unroll 1
    for (int i = 0; i < 2 * CW; ++i) {
      const int ch = wave * CW + (i >> 1), d = i & 1;
      StreamState& s = st[ch];
      uint32_t* range = reinterpret_cast<uint32_t*>(&s.range) + 2 * d;
      const uint32_t from = (uint32_t)GEAR_WAVE_UNIFORM((int)range[0]), base = from & 0xFFFFu, shift = from >> 16,
                     need = (uint32_t)GEAR_WAVE_UNIFORM((int)s.need[d]);
      if (GEAR_WAVE_UNIFORM((int)range[1]) == 0) continue;
      uint32_t hh[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) hh[b] = (hist[ch * 256 + 4 * lane + b] >> (16 * d)) & 0xFFFFu;
      const uint32_t total = lane_bcast_u(wave_incl_scan(hh[0] + hh[1] + hh[2] + hh[3]), 63);
      int bin;
      uint32_t above;
      scan_bins_from_top(hh, need, bin, above);
      const uint32_t equal = (hist[ch * 256 + bin] >> (16 * d)) & 0xFFFFu;
      wave_lds_sync();
      if (lane == 0) {
        if (total < need) {   // the rough threshold was no bound of this end
          range[0] = 8u << 16;
          range[1] = 0x10000u;
        } else {
          const bool last = shift == 5u && bin == 255;   // all that lies beyond 255 x 32 keys
          const uint32_t at = base + ((uint32_t)bin << shift);
          range[0] = at | (last ? 8u : 0u) << 16;
          range[1] = shift == 0u ? 0u : last ? 0x10000u - at : 1u << shift;
          s.need[d] = need - above;
          s.equal[d] = equal;
        }
      }
    }
  }
  block_lds_sync();
  uint32_t* equal_keys = hist + 8 * PC * 2 * STREAM_FEW;   // behind the lists: [4 PC] pairs of words, keys of two channels each
  if (tid < 8 * PC) {
    StreamState& s = st[tid];
    uint32_t need[2] = {s.need[0], s.need[1]}, take[2];
    const uint32_t at[2] = {s.range.x & 0xFFFFu, 0xFFFFu - (s.range.z & 0xFFFFu)};
    if (need[0] != 0u && need[1] != 0u && at[0] == at[1]) {   // one threshold: the bottom goes on where the top stops
      need[0] += need[1];
      need[1] = 0u;
    }
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      take[d] = need[d] == 0u ? EQUAL_NONE : need[d] == s.equal[d] ? EQUAL_ALL : s.equal[d] <= STREAM_FEW ? EQUAL_LISTED : EQUAL_WALK;
      s.equal[d] = (need[d] == 0u ? 0u : s.equal[d]) | take[d] << 16;
      reinterpret_cast<uint16_t*>(equal_keys)[4 * (tid >> 1) + 2 * d + (tid & 1)] = (uint16_t)(take[d] == EQUAL_LISTED ? at[d] : 0xFFFFu);
    }
    // taken in any case: keys above x, keys below y (z, w: at the thresholds themselves)
    s.range = make_uint4(s.need[0] == 0u ? 0xFFFFu : take[0] == EQUAL_ALL ? at[0] - 1u : at[0],
                         s.need[1] == 0u ? 0u : take[1] == EQUAL_ALL ? at[1] + 1u : at[1], at[0], at[1]);
    s.need[0] = need[0];
    s.need[1] = need[1];
    s.cnt = 0u;   // entries listed: of the top, of the bottom << 16
  }
  block_lds_sync();
  {
    uint32_t gt[4], lt[4], kmx[4], kmn[4], listed = 0u;   // two channels per word
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint4 a = st[ch0 + 2 * j].range, b = st[ch0 + 2 * j + 1].range;
      gt[j] = a.x | b.x << 16;
      lt[j] = a.y | b.y << 16;
      kmx[j] = kmn[j] = 0u;
    }
    for (int i = 0; i < 8 * PC; ++i) listed |= st[i].equal[0] >> 16 == EQUAL_LISTED || st[i].equal[1] >> 16 == EQUAL_LISTED ? 1u : 0u;
    listed = (uint32_t)GEAR_WAVE_UNIFORM((int)listed);
    for_each_batch<PC, T>(col, [&](const uint4 (&v)[STREAM_BATCH], int row0, int step) {
#pragma unroll
      for (int i = 0; i < STREAM_BATCH; ++i) {
        const int row = row0 + i * step;
        if (row >= col.n) continue;
        const uint32_t k[4] = {key16x2(v[i].x), key16x2(v[i].y), key16x2(v[i].z), key16x2(v[i].w)};
        uint32_t f = 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t z = nonzero_u16x2(sub_sat_u16x2(k[j], gt[j]) | sub_sat_u16x2(lt[j], k[j]));
          f |= z << j;
          if (rest) {   // (of entries at a threshold of which only some are taken, one stays)
            const uint32_t keep = ~neg_u16x2(z);
            kmx[j] = max_u16x2(kmx[j], k[j] & keep);
            kmn[j] = max_u16x2(kmn[j], ~k[j] & keep);
          }
        }
        while (f != 0u) {   // bit j + 16 h: channel 2 j + h of the piece
          const uint32_t b = (uint32_t)__ffs((int)f) - 1u;
          f &= f - 1u;
          mark_bit<PC>(bits, (uint32_t)row, ch0 + 2u * (b & 3u) + (b >> 4));
        }
        if (listed) {   // bit j + 4 d + 16 h
          uint32_t q = 0u;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const uint2 eq = reinterpret_cast<const uint2*>(equal_keys)[4 * col.pc + j];
            q |= (nonzero_u16x2(k[j] ^ eq.x) ^ 0x00010001u) << j;
            q |= (nonzero_u16x2(k[j] ^ eq.y) ^ 0x00010001u) << (j + 4);
          }
          while (q != 0u) {
            const uint32_t b = (uint32_t)__ffs((int)q) - 1u, d = (b >> 2) & 1u, ch = ch0 + 2u * (b & 3u) + (b >> 4);
            q &= q - 1u;
            const uint32_t at = (atomicAdd(&st[ch].cnt, d == 0u ? 1u : 0x10000u) >> (16u * d)) & 0xFFFFu;
            if (at < STREAM_FEW) hist[(2u * ch + d) * STREAM_FEW + at] = (uint32_t)row;
          }
        }
      }
    });
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (rest && st[ch0 + e].fail) {
        atomicMax(&st[ch0 + e].kmx, slot_key(kmx, e));
        atomicMax(&st[ch0 + e].kmn, slot_key(kmn, e));
      }
  }
  block_lds_sync();
#pragma unroll 1
  for (int cc = 0; cc < CW; ++cc) {
    const int ch = wave * CW + cc;
    StreamState& s = st[ch];
    uint32_t left[2], key[2];   // of a walk
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const uint32_t word = (uint32_t)GEAR_WAVE_UNIFORM((int)s.equal[d]), how = word >> 16, equal = word & 0xFFFFu,
                     need = (uint32_t)GEAR_WAVE_UNIFORM((int)s.need[d]);
      key[d] = (uint32_t)GEAR_WAVE_UNIFORM((int)(d == 0 ? s.range.z : s.range.w));
      left[d] = how == EQUAL_WALK ? need : 0u;
      if (how == EQUAL_LISTED) {
        const bool mine = lane < (int)equal;
        const uint32_t row = mine ? hist[(2 * ch + d) * STREAM_FEW + lane] : 0xFFFFFFFFu;
        uint32_t before = 0u;
        for (uint32_t j = 0; j < equal; ++j) before += lane_bcast_u(row, GEAR_WAVE_UNIFORM((int)j)) < row ? 1u : 0u;   // wave-uniform
        if (mine && before < need) mark_bit<PC>(bits, row, (uint32_t)ch);
      }
    }
#pragma unroll 1
    for (int base = 0; base < col.n && (left[0] | left[1]) != 0u; base += 64 * STREAM_WALK) {   // wave-uniform
      uint32_t x[STREAM_WALK];
#pragma unroll
      for (int i = 0; i < STREAM_WALK; ++i) x[i] = GEAR_BUF_LOAD2(col.buf, (base + 64 * i + lane) * (D * 2) + ch * 2);
#pragma unroll
      for (int i = 0; i < STREAM_WALK; ++i) {
        const int row = base + 64 * i + lane;
        const uint32_t k = key16(x[i]);
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          const bool hit = row < col.n && left[d] != 0u && k == key[d];
          const unsigned long long m = __ballot(hit);
          const uint32_t before = (uint32_t)__popcll(m & ((1ull << lane) - 1ull)), found = (uint32_t)__popcll(m);
          if (hit && before < left[d]) mark_bit<PC>(bits, (uint32_t)row, (uint32_t)ch);
          left[d] -= found < left[d] ? found : left[d];
        }
      }
    }
  }
  block_lds_sync();
}

// grid: slab_and_column_block over 128 / (8 PC) blocks per slab; block T; dynamic LDS: StreamPlan.  Thread (slot = tid / PC,
// pc = tid % PC) takes channels 8 pc .. 8 pc + 7 of the stretches slot + i T / PC, i < NB, of L rows each.  ONCE: L is 1.
// k_top, k_bot: entries wanted per channel; j_top, j_bot: the group extremes that make the rough thresholds; cap: entries of a
// channel's list.
template <int PC, int NB, bool ONCE, int T>
__global__ __launch_bounds__(T, ONCE && NB == 8 && T == 512 ? 6 : 4) void k_select_stream_kernel(const uint16_t* __restrict__ K, int n, int L, int nslab, int k_top,
                                                                            int k_bot, int j_top, int j_bot, int cap,
                                                                            uint4* __restrict__ mask, uint32_t* __restrict__ zero,
                                                                            int zero_count, uint32_t* __restrict__ ksz, int ng_cap, float qmax) {
  static_assert(PC == 1 || PC == 2, "the mask is stored a byte or two at a time");
  static_assert(stream_wave_channels(PC, T) >= 1, "every wave ranks channels");
  constexpr int CB = 8 * PC, RS = stream_rows(PC, T), NG = RS / 64, CW = stream_wave_channels(PC, T);
  GEAR_DYN_LDS(smem_raw);
  StreamState* st = reinterpret_cast<StreamState*>(smem_raw);
  uint32_t* list = reinterpret_cast<uint32_t*>(smem_raw + CB * sizeof(StreamState));   // also the sample's extremes, and histograms
  uint32_t* bits = list + (size_t)CB * cap;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < zero_count; i += gridDim.x * blockDim.x) zero[i] = 0u;
  int slab, cb;
  slab_and_column_block(blockIdx.x, nslab, D / CB, slab, cb);
  const int tid = threadIdx.x, wave = GEAR_WAVE_UNIFORM(tid >> 6), lane = tid & 63;
  const int pc = tid % PC, slot = tid / PC;
  const StreamColumn col{GEAR_BUF_MAKE(K + (size_t)slab * n * D + cb * CB, (n - 1) * (D * 2) + CB * 2), n, pc, slot};
  if (ONCE) L = 1;

  // ---- the sample: one row of each stretch, at a place that follows no pattern in the slots (rows past n read as 0); the
  // next rows are requested along with it
  const int step = RS * L;   // from one stretch of the thread to the next
  int o = ONCE ? 0 : (int)((((uint32_t)slot * 2654435761u ^ (uint32_t)slab * 2246822519u) * 3266489917u >> 16) * (uint32_t)L >> 16);
  uint4 p[NB];
  const int row0 = slot * L + o;
#pragma unroll
  for (int i = 0; i < NB; ++i) p[i] = col.load(row0 + i * step);
  // the other rows, stretch by stretch, so that the rows in flight lie close together
  uint4 cur[ONCE ? 1 : NB];
  int rows[ONCE ? 1 : NB], at = slot * L, ob = o, left = L - 1;   // stretch, offset of the last row taken in it, rows it has left
  auto request = [&](uint4 (&v)[ONCE ? 1 : NB], int (&r)[ONCE ? 1 : NB]) {
#pragma unroll
    for (int i = 0; i < (ONCE ? 1 : NB); ++i) {
      if (left == 0) {   // block-uniform
        left = L - 1;
        at += step;
        ob = o;
      }
      --left;
      ob = ob + 1 < L ? ob + 1 : 0;
      r[i] = at + ob;
      v[i] = col.load(r[i]);
    }
  };
  if constexpr (!ONCE) {
    if (L > 1) request(cur, rows);
  }
  if (tid == 0) st[0].range.w = 0u;
  for (int i = tid; i < (n * PC + 3) / 4; i += T) bits[i] = 0u;
  {
    uint32_t mx[4], mn[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      mx[j] = 0xFC00FC00u;
      mn[j] = 0x7C007C00u;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (row0 + i * step >= n) continue;
      const uint32_t w[4] = {p[i].x, p[i].y, p[i].z, p[i].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        mx[j] = pk_max_f16(mx[j], w[j]);
        mn[j] = pk_min_f16(mn[j], w[j]);
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {   // a word per channel: key of the maximum, complement of the key of the minimum
      const uint32_t kx = key16x2(mx[j]), kn = ~key16x2(mn[j]);
      list[(pc * 8 + 2 * j) * RS + slot] = GEAR_BYTE_PERM(kn, kx, 0x05040100u);
      list[(pc * 8 + 2 * j + 1) * RS + slot] = GEAR_BYTE_PERM(kn, kx, 0x07060302u);
    }
  }
  block_lds_sync();
#pragma unroll 1
  for (int cc = 0; cc < CW; ++cc) {
    const int ch = wave * CW + cc;
    uint32_t gx[NG], gn[NG];
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const uint32_t g = list[ch * RS + lane + 64 * i];
      gx[i] = g & 0xFFFFu;
      gn[i] = g >> 16;
    }
    uint32_t tt = 0u, tb = 0u;
    const auto search = [&](int from, int to) {   // these bits of the thresholds
#pragma unroll 1
      for (int b = from; b >= to; --b) {
        uint32_t nt = 0, nb = 0;
        const uint32_t qt = tt | 1u << b, qb = tb | 1u << b;
#pragma unroll
        for (int i = 0; i < NG; ++i) {
          nt += (uint32_t)__popcll(__ballot(gx[i] >= qt));
          nb += (uint32_t)__popcll(__ballot(gn[i] >= qb));
        }
        if (nt >= (uint32_t)j_top) tt = qt;
        if (nb >= (uint32_t)j_bot) tb = qb;
      }
    };
    search(15, 16 - STREAM_BITS);
    if (k_top == 0) tt = 0x10000u;
    if (k_bot == 0) tb = 0x10000u;
    const bool ok = rough_usable(tt, tb);
    if (__builtin_expect(!ok, 0)) {
      search(15 - STREAM_BITS, 0);
      if (lane == 0) {   // estimates for the way out
        st[ch].range.x = tt;
        st[ch].range.z = tb;
      }
    }
    if (lane == 0) {
      st[ch].cnt = 0u;
      st[ch].rough[0] = ok ? tt : 0x10000u;
      st[ch].rough[1] = ok ? tb : 0x10000u;
      st[ch].fail = ok ? 0u : 1u;
      if (ok) st[0].range.w = 1u;
    }
  }
  block_lds_sync();

  // ---- the candidates
  RoughBounds rb[4];   // of the channels 2 j (low halves) and 2 j + 1
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const StreamState &a = st[pc * 8 + 2 * j], &b = st[pc * 8 + 2 * j + 1];
    const RoughBounds ra = rough_bounds(a.rough[0], a.rough[1]), rc = rough_bounds(b.rough[0], b.rough[1]);
    rb[j].lo = (ra.lo & 0xFFFFu) | (rc.lo & 0xFFFF0000u);
    rb[j].hi = (ra.hi & 0xFFFFu) | (rc.hi & 0xFFFF0000u);
  }
  auto look = [&](const uint4& v, int row) {
    uint32_t f = outside_bits(v.x, rb[0], 0) | outside_bits(v.y, rb[1], 1) | outside_bits(v.z, rb[2], 2) | outside_bits(v.w, rb[3], 3);
    while (f != 0u) {   // bit j + 16 h: channel 2 j + h of the piece
      const uint32_t b = (uint32_t)__ffs((int)f) - 1u, e = 2u * (b & 3u) + (b >> 4), ch = pc * 8 + e;
      f &= f - 1u;
      const uint32_t at = atomicAdd(&st[ch].cnt, 1u);
      if (at < (uint32_t)cap) list[ch * cap + at] = (uint32_t)row | half_of(v.x, v.y, v.z, v.w, (int)e) << 16;
    }
  };
  const bool usable = GEAR_WAVE_UNIFORM((int)st[0].range.w) != 0;   // the same in every thread of the block
  if (usable) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (row0 + i * step < n) look(p[i], row0 + i * step);
  }
  if constexpr (!ONCE) {
    // (a stretch past the last one has no rows below n)
#pragma unroll 1
    for (int q = 0; usable && q < L - 1; ++q) {   // NB (L - 1) rows per thread, NB at a time
      uint4 nxt[NB];
      int nrows[NB];
      request(nxt, nrows);   // (the last time round: rows past the end, nothing is fetched)
#pragma unroll
      for (int i = 0; i < NB; ++i)
        if (rows[i] < n) look(cur[i], rows[i]);
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        cur[i] = nxt[i];
        rows[i] = nrows[i];
      }
    }
  }
  block_lds_sync();

  // ---- the exact sets
#pragma unroll 1
  for (int cc = 0; cc < CW; ++cc) {
    const int ch = wave * CW + cc;
    const uint32_t total = (uint32_t)GEAR_WAVE_UNIFORM((int)st[ch].cnt), tt = (uint32_t)GEAR_WAVE_UNIFORM((int)st[ch].rough[0]), tb = (uint32_t)GEAR_WAVE_UNIFORM((int)st[ch].rough[1]);
    bool ok = GEAR_WAVE_UNIFORM((int)st[ch].fail) == 0;
    uint32_t* l = list + ch * cap;   // (its place serves the ranking once the entries are in registers)
    uint32_t kmx = 0u, kmn = 0u;
    if (ok) {
      const bool part = total > (uint32_t)cap, rest = ksz != nullptr && !part;
      uint32_t held = total;
      int kt = k_top, kb = k_bot;
      if (__builtin_expect(part, 0)) {
        held = (uint32_t)cap;
        const float f = 1.25f * (float)held / (float)total;
        kt = (int)(f * (float)k_top) + 1;
        if (k_bot > 0) kb = (int)(f * (float)k_bot) + 1;
      }
      if (held <= 128u) ok = stream_rank<2, PC>(l, held, kt, kb, tt, tb, ch, bits, n, rest, part, kmx, kmn);
      else if (held <= 256u) ok = stream_rank<4, PC>(l, held, kt, kb, tt, tb, ch, bits, n, rest, part, kmx, kmn);
      else if (held <= 512u) ok = stream_rank<8, PC>(l, held, kt, kb, tt, tb, ch, bits, n, rest, part, kmx, kmn);
      else if (ONCE || held <= 1024u) ok = stream_rank<16, PC>(l, held, kt, kb, tt, tb, ch, bits, n, rest, part, kmx, kmn);
      else if constexpr (!ONCE) ok = stream_rank<32, PC>(l, held, kt, kb, tt, tb, ch, bits, n, rest, part, kmx, kmn);
      if (__builtin_expect(!ok, 0) && lane == 0) {
        st[ch].range.x = kmx != 0u ? kmx : tt;
        st[ch].range.z = kmx != 0u ? kmn : tb;
      }
    }
    if (ksz) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        kmx = max(kmx, (uint32_t)__shfl_xor(kmx, o, 64));
        kmn = max(kmn, (uint32_t)__shfl_xor(kmn, o, 64));
      }
    }
    wave_lds_sync();
    if (lane == 0) {
      st[ch].fail = ok ? 0u : 1u;
      st[ch].kmx = kmx;
      st[ch].kmn = kmn;
    }
  }
  block_lds_sync();
  uint32_t failed = 0;
  for (int i = 0; i < CB; ++i) failed |= st[i].fail;
  if (__builtin_expect(GEAR_WAVE_UNIFORM((int)failed) != 0, 0)) {   // the same in every thread of the block
    // (a failed channel has no bits yet: stream_rank sets them only where it returns true)
    stream_way_out<PC, T>(col, st, list, bits, k_top, k_bot, ksz != nullptr);
  }
  // per-vector grouping: the channel's (scale, zero), outliers counted as 0
  if (ksz && tid < CB) {
    const uint32_t hi = max(st[tid].kmx, 0x8000u), lo = min(0xFFFFu - st[tid].kmn, 0x8000u);
    ksz[(size_t)slab * ng_cap * D + cb * CB + tid] = group_bits(make_group(h2f(unkey16(lo)), h2f(unkey16(hi)), qmax));
  }
  uint8_t* mrow = reinterpret_cast<uint8_t*>(mask + (size_t)slab * n) + cb * PC;
  for (int t = tid; t < n; t += T) {
    if constexpr (PC == 1) mrow[(size_t)t * 16] = reinterpret_cast<const uint8_t*>(bits)[t];
    else *reinterpret_cast<uint16_t*>(mrow + (size_t)t * 16) = reinterpret_cast<const uint16_t*>(bits)[t];
  }
}

// Everything the host decides: false where the lists would not fit, the ratio is near one entry in two, or nothing is wanted.
struct StreamPlan {
  int L, j_top, j_bot, cap;
  size_t lds;
};
// A sample of m of the n entries holds mu = k m / n of the k wanted ones on average, with a spread of sqrt(mu (1 - m / n)); five and
// a half of those above it, and a little for the skew of small counts, leave too short a list once in some millions of channels, and the
// room on the list one too long once in some ten thousand (of 43000 normal channels of 24000 tokens at 1 %, one).  That holds for rows in no order:
// a thread's stretches share one offset, so a channel sorted by position, or periodic in the stretches, may go the long way (not the
// wrong one).  j of G groups of s sampled entries reach the threshold when a share of 1 - (1 - j / G)^(1/s) of all entries does.
inline bool stream_plan(int pc, int nb, bool once, int t, int n, int k_top, int k_bot, bool rest, size_t lds_max, StreamPlan& p) {
  const int slots = stream_rows(pc, t);
  p.L = (n + slots * nb - 1) / (slots * nb);
  const int m = n / p.L, groups = m < slots ? m : slots;   // rows of the sample, groups that hold some
  double expect = 0.0, spread = 0.0;
  const auto side = [&](int k) {
    if (k == 0) return 0;
    const double mu = (double)k * m / n;
    const int j = p.L == 1 ? k + (rest ? 1 : 0) : (int)ceil(mu + 5.5 * sqrt(mu * (1.0 - (double)m / n)) + 3.0);
    if (j >= groups) { expect = 1e9; return j; }
    const double e = 1.04 * n * (1.0 - pow(1.0 - (double)j / groups, (double)groups / m));
    expect += e;
    spread += e * e / j;
    return j;
  };
  p.j_top = side(k_top);
  p.j_bot = side(k_bot);
  if (k_top == 0 || (rest && k_bot == 0) || expect > 4096.0) return false;   // (the extremes of the rest need a list at both ends)
  p.cap = ((int)(expect + 4.5 * sqrt(spread) + 64.0) + 63) & ~63;
  if (p.cap > (once ? 1024 : 2048)) return false;   // (what a wave ranks in registers)
  if (p.cap < 256) p.cap = 256;                // a histogram
  if (p.cap < slots) p.cap = slots;            // the sample's extremes lie in the lists' place
  p.lds = 8 * pc * sizeof(StreamState) + (size_t)8 * pc * p.cap * 4 + ((size_t)n * pc + 3) / 4 * 4;
  return p.lds <= lds_max;
}

}  // namespace gear
