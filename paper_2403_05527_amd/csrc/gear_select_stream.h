// Filter_s (Eq. 4) of Key channel vectors, from lists of candidates collected while the tensor streams by.
//
// A block takes 8 or 16 neighbouring channels of one slab.  Reading such a column costs a whole 128-byte line per 16 or 32
// bytes between the CU's first-level cache and the L2, so the column should be read once, and a vector of thousands of
// tokens is best not kept: of its entries only a few per cent can belong to S.  So
//   1. the segment is cut into some 2048 stretches of L rows; one row of each gives every channel a rough threshold per end: the
//      j-th most extreme of the extremes of groups of eight sampled entries (gear_select_ext.h), with j far enough above the
//      number of wanted entries that are expected in the sample (stream_plan).  With L = 1 the sample is the whole segment, and
//      the threshold holds for certain;
//   2. the sample, which is still in registers, and then the other rows of the stretches are looked at once; what passes a rough
//      threshold goes onto its channel's list in LDS;
//   3. one wave per channel ranks its list exactly, index and all, and leaves the selected entries as bits in LDS, whence the
//      mask is stored.
// A channel whose list overflows (ties), or holds fewer entries than are wanted, is selected by stream_way_out: radix levels over
// histograms in LDS, reading the column again for each.  It is slow, and for inputs of a few distinct values (all channels of 128
// slabs x 8192 tokens constant: a call of 1752 us takes 1878; one constant channel: some 50 us of one block).
//
// 64 x 8 slabs x 8192 tokens at 2 %, one wave per vector in registers before: 621 -> 450 us.  Of those the sample and the thresholds
// take 80, the rest of the read 230 (four 32-byte pieces per line: the first-level cache takes in 32 bytes per cycle and CU, which is
// 220 us), the appending 60, the ranking 60, the mask 20.  32 slabs x 32768 (8 channels per block) 274 -> 147, 280 x 1777 92 -> 67,
// 512 x 4096 270 -> 215.  As three kernels (sample; candidates from whole rows into the workspace; ranking) 72 + 255 + 108: no gain.
#pragma once
#include "gear_internal.h"
#include "gear_select.h"
#include "gear_select_ext.h"

namespace gear {

constexpr int STREAM_BITS = 11;                      // resolution of the rough thresholds (1/32 of an octave)
constexpr int STREAM_THREADS = 512;
__host__ __device__ constexpr int stream_rows(int pc) { return STREAM_THREADS / pc; }   // rows a block reads side by side
struct StreamState {   // per channel, in LDS
  uint32_t cnt, tt, tb, fail;
  uint32_t xt, xb;            // way_out: the two exact thresholds (composites)
  uint32_t prefix, need;      // way_out: what is known of the threshold in work, entries still to be found
  uint32_t kmx, kmn;          // way_out: the extremes of what is not selected (kmn: complement)
  uint32_t pad[2];
};

// Decodes a 1-D grid of ncb * nslab blocks, one per slab and block of channels.  Consecutive block ids go round-robin to
// the chip's 8 XCDs (each with its own L2), so the id is decoded with the column block fastest INSIDE one XCD: the blocks
// that share the 128-byte lines of one slab (of its rows, of its mask) then meet in one L2 instead of eight.  The up to
// seven slabs past a multiple of eight go to all XCDs.  231 slabs x 3000 tokens, which went to all XCDs as a whole before:
// 245 -> 106 us.
__device__ __forceinline__ void slab_and_column_block(int nslab, int ncb, int& slab, int& cb) {
  const int i = blockIdx.x, even = (nslab & ~7) * ncb;
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
// f(piece, row) for every row of the thread
template <int PC, class F>
__device__ __forceinline__ void for_each_row(const StreamColumn& col, F&& f) {
  constexpr int RS = stream_rows(PC), NB = 4;
#pragma unroll 1
  for (int base = col.slot; base < col.n; base += RS * NB) {
    uint4 v[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) v[i] = col.load(base + i * RS);
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (base + i * RS < col.n) f(v[i], base + i * RS);
  }
}
template <int PC>
__device__ __forceinline__ void mark_bit(uint32_t* bits, uint32_t row, uint32_t ch) {   // byte PC row + ch / 8, bit ch % 8
  const uint32_t byte = row * PC + (ch >> 3);
  atomicOr(&bits[byte >> 2], 1u << ((byte & 3u) * 8u + (ch & 7u)));
}

// Ranks a channel's list (total entries, row | fp16 value << 16).  Returns false where it does not hold enough entries (one more
// than are wanted where the extremes of the rest are asked for).  Called by a whole wave.
template <int R, int PC>
__device__ __forceinline__ bool stream_rank(uint32_t* list, uint32_t total, int k_top, int k_bot, uint32_t tt, uint32_t tb, uint32_t ch,
                                            uint32_t* bits, bool rest, uint32_t& kmx, uint32_t& kmn) {
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
  if (k_top > 0 && !enough(tt, k_top)) return false;
  const uint32_t xt = k_top > 0 ? wave_kth_by_bins<R>(c, (uint32_t)k_top, tt, list) : 0xFFFFFFFFu;
  flip();
  if (k_bot > 0 && !enough(tb, k_bot)) return false;
  const uint32_t xb = k_bot > 0 ? wave_kth_by_bins<R>(c, (uint32_t)k_bot, tb, list) : 0xFFFFFFFFu;
  kmx = kmn = 0u;
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

// The exact thresholds of the channels marked in st[].fail, one byte of the composite (key, index) per pass over the column: first
// those of the top, then those of the bottom among the rest; their entries' bits and, if asked for, the extremes of the rest.
template <int PC>
__device__ __forceinline__ void stream_way_out(const StreamColumn& col, StreamState* st, uint32_t* hist /* [8 PC][256] */, uint32_t* bits,
                                            int k_top, int k_bot) {
  const int tid = threadIdx.x, wave = GEAR_WAVE_UNIFORM(tid >> 6), lane = tid & 63, ch0 = col.pc * 8;
  if (tid < 8 * PC) {
    st[tid].xt = st[tid].xb = 0xFFFFFFFFu;
    if (st[tid].fail) st[tid].kmx = st[tid].kmn = 0u;
  }
  block_lds_sync();
#pragma unroll 1
  for (int side = 0; side < 2; ++side) {
    const uint32_t k = (uint32_t)(side == 0 ? k_top : k_bot), flip = side == 0 ? 0u : 0xFFFF0000u;
    if (k == 0u) continue;
    if (tid < 8 * PC) {
      st[tid].prefix = 0u;
      st[tid].need = st[tid].fail ? k : 0u;   // 0: found, or not in work
    }
#pragma unroll 1
    for (int shift = 24; shift >= 0; shift -= 8) {
      block_lds_sync();
      for (int i = tid; i < 8 * PC * 256; i += STREAM_THREADS) hist[i] = 0u;
      block_lds_sync();
      // (runs of one counter are added up in the thread: where most of a channel is one value, adds to one address would be
      // applied one after another)
      uint32_t prefix[8], xt[8], run[8], len[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const StreamState& s = st[ch0 + e];
        prefix[e] = s.need != 0u ? s.prefix : 0xFFFFFFFFu;   // (found, or not in work: no entry has this prefix)
        xt[e] = side == 1 ? s.xt : 0xFFFFFFFFu;
        run[e] = len[e] = 0u;
      }
      for_each_row<PC>(col, [&](const uint4& v, int row) {
        const uint32_t kw[4] = {key16x2(v.x), key16x2(v.y), key16x2(v.z), key16x2(v.w)};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint32_t t = slot_key(kw, e) << 16 | (0xFFFFu - (uint32_t)row), c = t ^ flip;
          const uint32_t above = shift == 24 ? 0u : c >> ((shift + 8) & 31), bin = (c >> shift) & 255u;
          if (above != prefix[e] || t >= xt[e]) continue;
          if (bin != run[e]) {
            if (len[e] != 0u) atomicAdd(&hist[(ch0 + e) * 256 + run[e]], len[e]);
            run[e] = bin;
            len[e] = 0u;
          }
          ++len[e];
        }
      });
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (len[e] != 0u) atomicAdd(&hist[(ch0 + e) * 256 + run[e]], len[e]);
      block_lds_sync();
#pragma unroll 1
      for (int cc = 0; cc < PC; ++cc) {
        StreamState& s = st[wave * PC + cc];
        const uint32_t need = s.need;
        if (need == 0u) continue;   // wave-uniform
        const uint32_t* h = hist + (wave * PC + cc) * 256;
        int bin;
        uint32_t above;
        scan_from_top(h, need, bin, above);
        const uint32_t prefix = s.prefix << 8 | (uint32_t)bin;
        const bool found = need - above == h[bin] || shift == 0;   // the whole bin is wanted
        wave_lds_sync();
        if (lane == 0) {
          s.prefix = prefix;
          s.need = found ? 0u : need - above;
          if (found) (side == 0 ? s.xt : s.xb) = prefix << shift;
        }
      }
    }
    block_lds_sync();
  }
  {
    uint32_t xt[8], xb[8], kmx[8], kmn[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const StreamState& s = st[ch0 + e];
      xt[e] = s.fail ? s.xt : 0xFFFFFFFFu;
      xb[e] = s.fail ? s.xb : 0xFFFFFFFFu;
      kmx[e] = kmn[e] = 0u;
    }
    for_each_row<PC>(col, [&](const uint4& v, int row) {
      const uint32_t kw[4] = {key16x2(v.x), key16x2(v.y), key16x2(v.z), key16x2(v.w)};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t key = slot_key(kw, e), t = key << 16 | (0xFFFFu - (uint32_t)row);
        if (t >= xt[e] || (t ^ 0xFFFF0000u) >= xb[e]) mark_bit<PC>(bits, (uint32_t)row, (uint32_t)(ch0 + e));
        else {
          kmx[e] = max(kmx[e], key);
          kmn[e] = max(kmn[e], 0xFFFFu - key);
        }
      }
    });
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (st[ch0 + e].fail) {
        atomicMax(&st[ch0 + e].kmx, kmx[e]);
        atomicMax(&st[ch0 + e].kmn, kmn[e]);
      }
  }
  block_lds_sync();
}

// grid: slab_and_column_block over 128 / (8 PC) blocks per slab; block 512; dynamic LDS: StreamPlan.  Thread (slot = tid / PC,
// pc = tid % PC) takes channels 8 pc .. 8 pc + 7 of the stretches slot + i 512 / PC, i < NB, of L rows each.  ONCE: L is 1.
// k_top, k_bot: entries wanted per channel; j_top, j_bot: the group extremes that make the rough thresholds; cap: entries of a
// channel's list.
template <int PC, int NB, bool ONCE>
__global__ __launch_bounds__(STREAM_THREADS, 4) void k_select_stream_kernel(const uint16_t* __restrict__ K, int n, int L, int nslab, int k_top,
                                                                            int k_bot, int j_top, int j_bot, int cap,
                                                                            uint4* __restrict__ mask, uint32_t* __restrict__ zero,
                                                                            int zero_count, uint32_t* __restrict__ ksz, int ng_cap, float qmax) {
  constexpr int CB = 8 * PC, RS = stream_rows(PC), NG = RS / 64;
  GEAR_DYN_LDS(smem_raw);
  StreamState* st = reinterpret_cast<StreamState*>(smem_raw);
  uint32_t* list = reinterpret_cast<uint32_t*>(smem_raw + CB * sizeof(StreamState));   // also the sample's extremes, and histograms
  uint32_t* bits = list + (size_t)CB * cap;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < zero_count; i += gridDim.x * blockDim.x) zero[i] = 0u;
  int slab, cb;
  slab_and_column_block(nslab, D / CB, slab, cb);
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
  for (int i = tid; i < (n * PC + 3) / 4; i += STREAM_THREADS) bits[i] = 0u;
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
  for (int cc = 0; cc < PC; ++cc) {
    const int ch = wave * PC + cc;
    uint32_t gx[NG], gn[NG];
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const uint32_t g = list[ch * RS + lane + 64 * i];
      gx[i] = g & 0xFFFFu;
      gn[i] = g >> 16;
    }
    uint32_t tt = 0u, tb = 0u;
#pragma unroll 1
    for (int b = 15; b >= 16 - STREAM_BITS; --b) {
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
    if (k_top == 0) tt = 0x10000u;
    if (k_bot == 0) tb = 0x10000u;
    const bool ok = rough_usable(tt, tb);
    if (lane == 0) {
      st[ch].cnt = 0u;
      st[ch].tt = ok ? tt : 0x10000u;
      st[ch].tb = ok ? tb : 0x10000u;
      st[ch].fail = ok ? 0u : 1u;
    }
  }
  block_lds_sync();

  // ---- the candidates
  RoughBounds rb[4];   // of the channels 2 j (low halves) and 2 j + 1
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const StreamState &a = st[pc * 8 + 2 * j], &b = st[pc * 8 + 2 * j + 1];
    const RoughBounds ra = rough_bounds(a.tt, a.tb), rc = rough_bounds(b.tt, b.tb);
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
#pragma unroll
  for (int i = 0; i < NB; ++i)
    if (row0 + i * step < n) look(p[i], row0 + i * step);
  if constexpr (!ONCE) {
    // (a stretch past the last one has no rows below n)
#pragma unroll 1
    for (int q = 0; q < L - 1; ++q) {   // NB (L - 1) rows per thread, NB at a time
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
  for (int cc = 0; cc < PC; ++cc) {
    const int ch = wave * PC + cc;
    const uint32_t total = (uint32_t)GEAR_WAVE_UNIFORM((int)st[ch].cnt), tt = (uint32_t)GEAR_WAVE_UNIFORM((int)st[ch].tt), tb = (uint32_t)GEAR_WAVE_UNIFORM((int)st[ch].tb);
    bool ok = GEAR_WAVE_UNIFORM((int)st[ch].fail) == 0 && total <= (uint32_t)cap;
    uint32_t* l = list + ch * cap;   // (its place serves the ranking once the entries are in registers)
    uint32_t kmx = 0u, kmn = 0u;
    if (ok) {
      const bool rest = ksz != nullptr;
      if (total <= 128u) ok = stream_rank<2, PC>(l, total, k_top, k_bot, tt, tb, ch, bits, rest, kmx, kmn);
      else if (total <= 256u) ok = stream_rank<4, PC>(l, total, k_top, k_bot, tt, tb, ch, bits, rest, kmx, kmn);
      else if (total <= 512u) ok = stream_rank<8, PC>(l, total, k_top, k_bot, tt, tb, ch, bits, rest, kmx, kmn);
      else if (ONCE || total <= 1024u) ok = stream_rank<16, PC>(l, total, k_top, k_bot, tt, tb, ch, bits, rest, kmx, kmn);
      else if constexpr (!ONCE) ok = stream_rank<32, PC>(l, total, k_top, k_bot, tt, tb, ch, bits, rest, kmx, kmn);
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
  if (GEAR_WAVE_UNIFORM((int)failed) != 0) {   // the same in every thread of the block
    // (a failed channel has no bits yet: stream_rank sets them only where it returns true)
    stream_way_out<PC>(col, st, list, bits, k_top, k_bot);
  }
  // per-vector grouping: the channel's (scale, zero), outliers counted as 0
  if (ksz && tid < CB) {
    const uint32_t hi = max(st[tid].kmx, 0x8000u), lo = min(0xFFFFu - st[tid].kmn, 0x8000u);
    ksz[(size_t)slab * ng_cap * D + cb * CB + tid] = group_bits(make_group(h2f(unkey16(lo)), h2f(unkey16(hi)), qmax));
  }
  uint8_t* mrow = reinterpret_cast<uint8_t*>(mask + (size_t)slab * n) + cb * PC;
  for (int t = tid; t < n; t += STREAM_THREADS) {
    if constexpr (PC == 1) mrow[(size_t)t * 16] = reinterpret_cast<const uint8_t*>(bits)[t];
    else if constexpr (PC == 2) *reinterpret_cast<uint16_t*>(mrow + (size_t)t * 16) = reinterpret_cast<const uint16_t*>(bits)[t];
    else *reinterpret_cast<uint32_t*>(mrow + (size_t)t * 16) = bits[t];
  }
}

// Everything the host decides: false where the lists would not fit, the ratio is near one entry in two, or nothing is wanted.
struct StreamPlan {
  int L, j_top, j_bot, cap;
  size_t lds;
};
// A sample of m of the n entries holds mu = k m / n of the k wanted ones on average, with a spread of sqrt(mu (1 - m / n)); five and
// a half of those above it, and a little for the skew of small counts, fail once in some millions of channels.  j of G groups of
// s sampled entries reach the threshold when a share of 1 - (1 - j / G)^(1/s) of all entries does.
inline bool stream_plan(int pc, int nb, bool once, int n, int k_top, int k_bot, bool rest, size_t lds_max, StreamPlan& p) {
  const int slots = stream_rows(pc);
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
