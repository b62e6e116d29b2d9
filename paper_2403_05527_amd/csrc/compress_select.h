// The selections of short segments, a block or a wave at a time: Filter_s (Eq. 4) of Key channel vectors of up to 8192 entries held in
// registers, of those of a flushed buffer, and of one Value token.
#pragma once
#include "gear_internal.h"
#include "gear_select.h"
#include "gear_select_ext.h"
#include "gear_select_stream.h"

namespace gear {

// ------------------------------------------------------------------ sources
template <int NC>
struct RegSource {  // the vector lives in the wave's registers
  static constexpr int kMaxChunks = NC;
  const uint4* x;
  __device__ __forceinline__ uint4 operator()(int ch) const { return x[ch]; }
};

// A block's eight channels' outlier bits go through LDS as an 8 x 8 bit matrix per eight consecutive tokens, 8 bytes at
// 8 (t / 8).  Every wave leaves its channel's byte (bit e: token 8 (t / 8) + e), one byte store per chunk and lane; the block
// then transposes the matrices in place (byte e: the eight channels of that token) and stores them into the mask rows, byte
// cb of row t.  Bits past n are not masked out: they end up in rows that are not stored.  Whole bytes, because hardly a chunk of
// 512 keys holds no outlier: one atomic per set bit ran its divergent loop for every chunk.  Keys of 512 slabs x 8192 tokens
// 645 -> 620 us, 32 slabs x 32768 (rank-8 call) 201 -> 187, 8 slabs x 32768 109 -> 96.
__device__ __forceinline__ void mark_chunk(const uint4& v, int ch, uint32_t* bits, const ThreshPair& tp, const ThreshKeys& tk) {
  const uint32_t first = (uint32_t)(ch * 512 + lane_id() * 8);
  reinterpret_cast<uint8_t*>(bits)[first + (threadIdx.x >> 6)] = (uint8_t)(tk.cut ? piece_bits(v, first, tp) : key_bits(v, tk));
}
__device__ __forceinline__ void store_mask_bytes(uint32_t* bits, uint4* mask_slab, int n, int cb) {
  for (int q = threadIdx.x; q < (n + 7) / 8; q += blockDim.x) {
    uint2* m = reinterpret_cast<uint2*>(bits) + q;
    *m = transpose_bits8(*m);
  }
  block_lds_sync();
  for (int t = threadIdx.x; t < n; t += blockDim.x)
    reinterpret_cast<uint8_t*>(mask_slab + t)[cb] = reinterpret_cast<const uint8_t*>(bits)[t];
}

// ------------------------------------------------------------------ K select, segments of at most 64 tokens
// A flushed buffer: 128 vectors of n_b entries per slab, of which Filter_s keeps one or two.  One block per
// slab, one thread per channel; the slab's rows sit in LDS as keys, row-major as they come, and a thread
// walks down its column.  The selected sets are found by taking the column's largest composite
// (key, index) below the previous one k_top times, then the smallest above the previous one among the
// entries outside the top set k_bot times: (k_top + k_bot) n steps per vector instead of a ranking of
// every entry against every other.
constexpr int KSEL_TINY_ROWS = 64;
struct KTinySmem {
  __attribute__((aligned(16))) uint16_t tile[KSEL_TINY_ROWS * D];
  uint4 rowmask[KSEL_TINY_ROWS];
};
// A block of 128 threads, number `slab` of nslab.
__device__ __forceinline__ void k_select_tiny_block(KTinySmem& sm, const uint16_t* __restrict__ K, int slab, int nslab, int n, int k_top, int k_bot,
                                                    uint4* __restrict__ mask, uint32_t* __restrict__ zero, int zero_count,
                                                    uint32_t* __restrict__ ksz, int ng_cap, float qmax) {
  uint16_t* tile = sm.tile;
  uint4* rowmask = sm.rowmask;
  // the first kernel of a compress call also clears the call's list counters
  for (int i = slab * 128 + threadIdx.x; i < zero_count; i += nslab * 128) zero[i] = 0u;
  const int c = threadIdx.x;
  if (c < KSEL_TINY_ROWS) rowmask[c] = make_uint4(0, 0, 0, 0);
  {
    const GEAR_BUF_T xb = GEAR_BUF_MAKE(K + (size_t)slab * n * D, n * (D * 2));
    const int npieces = n * (D / 8);   // 16-byte pieces of the slab's rows
    for (int p0 = 0; p0 < npieces; p0 += 4 * 128) {
      uint4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = GEAR_BUF_LOAD16(xb, (p0 + u * 128 + c) * 16);   // pieces past the end read as 0
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int p = p0 + u * 128 + c;
        if (p < npieces)
          *reinterpret_cast<uint4*>(tile + p * 8) = make_uint4(key16x2(v[u].x), key16x2(v[u].y), key16x2(v[u].z), key16x2(v[u].w));
      }
    }
  }
  block_lds_sync();
  Thresh th = thresh_none();
  // composites: (key << 16) | (0xFFFF - index) orders (value desc, index asc) from the top,
  // (key << 16) | index orders (value asc, index asc) from the bottom; all distinct, and the first kind > 0
  uint32_t T = 0u;   // composite of the last top entry
  for (int it = 0; it < k_top; ++it) {
    uint32_t best = 0u;
    for (int j = 0; j < n; ++j) {
      const uint32_t cT = ((uint32_t)tile[j * D + c] << 16) | (0xFFFFu - (uint32_t)j);
      if ((it == 0 || cT < T) && cT > best) best = cT;
    }
    T = best;
  }
  if (k_top > 0 && T != 0u) {
    th.tau_top = T >> 16;
    th.i_top = (int)(0xFFFFu - (T & 0xFFFFu));
  }
  if (k_bot > 0) {
    uint32_t Bc = 0u;
    bool found = true;
    for (int it = 0; it < k_bot && found; ++it) {
      uint32_t best = 0xFFFFFFFFu;
      for (int j = 0; j < n; ++j) {
        const uint32_t key = tile[j * D + c];
        const bool in_top = k_top > 0 && ((key << 16) | (0xFFFFu - (uint32_t)j)) >= T;
        const uint32_t cB = (key << 16) | (uint32_t)j;
        if (!in_top && (it == 0 || cB > Bc) && cB < best) best = cB;
      }
      found = best != 0xFFFFFFFFu;
      Bc = best;
    }
    if (found) {
      th.tau_bot = Bc >> 16;
      th.i_bot = (int)(Bc & 0xFFFFu);
      th.l_bot = (k_top > 0 && th.tau_bot == th.tau_top) ? th.i_top : -1;
    }
  }
  const ThreshPair tp = pack_thresh(th);
  uint32_t kmn = 0xFFFFu, kmx = 0u;
  for (int j = 0; j < n; ++j) {
    const uint32_t k = tile[j * D + c];
    const bool out = outlier(k, (uint32_t)j, tp);
    if (out) atomicOr(&reinterpret_cast<uint32_t*>(&rowmask[j])[c >> 5], 1u << (c & 31));
    const uint32_t y = out ? 0x8000u : k;
    kmn = min(kmn, y);
    kmx = max(kmx, y);
  }
  // per-vector grouping: the channel's one group of this call spans the whole vector: min and max of
  // X - S, i.e. with the outliers counted as 0
  if (ksz) ksz[(size_t)slab * ng_cap * D + c] = group_bits(make_group(h2f(unkey16(kmn)), h2f(unkey16(kmx)), qmax));
  block_lds_sync();
  if (mask && c < n) mask[(size_t)slab * n + c] = rowmask[c];
}

// ------------------------------------------------------------------ K select, vectors in registers
// For segments of 65 .. 8192 tokens: a block of eight waves takes eight neighbouring channels, one per
// wave, and every wave ends up with its whole channel vector in registers (NC chunks of 512 keys, the
// layout wave_select reads), so LDS only holds the histograms and a staging buffer and the occupancy no
// longer falls with the segment length.  The vector arrives 1024 tokens at a time: thread tid loads the
// 16-byte row pieces (8 channels) of rows 2 tid and 2 tid + 1, pairs the two rows' keys of each channel
// in one word and writes it to stage[channel][tid]; wave w then reads channel w's 1024 keys back as two
// 16-byte pieces per lane.  All of a thread's loads are requested at the start.
template <int NC>
struct KRegSmem {
  uint32_t hist[8 * SELECT_LDS_WORDS];
  __attribute__((aligned(16))) uint32_t bits[NC * 512 / 4];
  __attribute__((aligned(16))) uint32_t stage[8][512];
};
// A block of 512 threads, number `block` of 16 * nslab (slab_and_column_block).
template <int NC>
__device__ __forceinline__ void k_select_reg_block(KRegSmem<NC>& sm, const uint16_t* __restrict__ K, int block, int n, int nslab, int k_top, int k_bot,
                                                   uint4* __restrict__ mask, uint32_t* __restrict__ zero, int zero_count,
                                                   uint32_t* __restrict__ ksz, int ng_cap, float qmax) {
  uint32_t* hist = sm.hist;
  uint32_t* bits = sm.bits;
  uint32_t (&stage)[8][512] = sm.stage;
  for (int i = block * 512 + (int)threadIdx.x; i < zero_count; i += nslab * (D / 8) * 512) zero[i] = 0u;
  int slab, cb;
  slab_and_column_block(block, nslab, D / 8, slab, cb);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  // a view of the column block that ends with its last row: rows past n read as 0
  const GEAR_BUF_T xb = GEAR_BUF_MAKE(K + (size_t)slab * n * D + cb * 8, (n - 1) * (D * 2) + 16);
  // every row piece of the thread is requested before the first one is used (rows past n read as 0): the
  // pieces wait in the registers that the finished chunks take over one after another
  uint4 x[NC], raw[NC];
#pragma unroll
  for (int it = 0; it < NC / 2; ++it) {
    raw[2 * it] = GEAR_BUF_LOAD16(xb, (it * 1024 + 2 * tid) * (D * 2));
    raw[2 * it + 1] = GEAR_BUF_LOAD16(xb, (it * 1024 + 2 * tid + 1) * (D * 2));
  }
#pragma unroll
  for (int it = 0; it < NC / 2; ++it) {
    const uint4 ra = raw[2 * it], rb = raw[2 * it + 1];
    const uint32_t ka[4] = {key16x2(ra.x), key16x2(ra.y), key16x2(ra.z), key16x2(ra.w)};
    const uint32_t kb[4] = {key16x2(rb.x), key16x2(rb.y), key16x2(rb.z), key16x2(rb.w)};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      stage[2 * j][tid] = GEAR_BYTE_PERM(kb[j], ka[j], 0x05040100u);       // channel 2j of rows 2 tid, 2 tid + 1
      stage[2 * j + 1][tid] = GEAR_BYTE_PERM(kb[j], ka[j], 0x07060302u);   // channel 2j + 1
    }
    block_lds_sync();
    x[2 * it] = *reinterpret_cast<const uint4*>(&stage[wave][lane * 4]);
    x[2 * it + 1] = *reinterpret_cast<const uint4*>(&stage[wave][256 + lane * 4]);
    block_lds_sync();
  }
  RegSource<NC> src{x};
  const Thresh th = wave_select(src, n, k_top, k_bot, hist + wave * SELECT_LDS_WORDS, true);
  const int ch = cb * 8 + wave;
  const ThreshPair tp = pack_thresh(th);
  if (ksz) {   // per-vector grouping: the channel's (scale, zero), outliers counted as 0
    uint32_t kmn = 0xFFFFu, kmx = 0u;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const uint32_t kw[4] = {x[c].x, x[c].y, x[c].z, x[c].w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t k = slot_key(kw, e), idx = (uint32_t)(c * 512 + lane * 8 + e);
        if ((int)idx < n) {
          const uint32_t y = outlier(k, idx, tp) ? 0x8000u : k;
          kmn = min(kmn, y);
          kmx = max(kmx, y);
        }
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      kmn = min(kmn, (uint32_t)__shfl_xor(kmn, o, 64));
      kmx = max(kmx, (uint32_t)__shfl_xor(kmx, o, 64));
    }
    if (lane == 0) ksz[(size_t)slab * ng_cap * D + ch] = group_bits(make_group(h2f(unkey16(kmn)), h2f(unkey16(kmx)), qmax));
  }
  if (!mask) return;
  const ThreshKeys tk = key_thresh(tp);
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (c * 512 < n) mark_chunk(x[c], c, bits, tp, tk);
  block_lds_sync();
  store_mask_bytes(bits, mask + (size_t)slab * n, n, cb);
}

// ------------------------------------------------------------------ V select
// The mask of a token from the bits of its vector, which the selection leaves in LDS: lane h stores head h's 16 bytes.
__device__ __forceinline__ void store_token_mask(const uint32_t* smask, uint4* mask, int b, int H, int n, int t) {
  const int h = lane_id();
  if (h < H) mask[((size_t)b * H + h) * n + t] = *reinterpret_cast<const uint4*>(smask + 4 * h);
}

// A token of a batch element, by one wave.  raw: NC * 64 pieces, list: EXT_LIST words of LDS of its own.
// lane l, chunk ch  <->  head 4*ch + l/16, channels 8*(l%16)..+7, i.e. in-vector index
// ch*512 + l*8 + e.
// Under the per-vector grouping (vsz != nullptr) the kernel also leaves the token's (scale, zero):
// its one Value group spans the whole vector, outliers counted as 0.  per_head: the Filter ranks
// each head's 128 channels (the 16 lanes of a row) on their own; the mask is then not stored (the quantization kernel
// finds the entries again, they cost less than their round trip).
template <int NC>
__device__ __forceinline__ void v_select_token(uint4* raw, uint32_t* list, const uint16_t* __restrict__ V, int b, int t, int H, int n, int k_top,
                                               int k_bot, uint4* __restrict__ mask, uint32_t* __restrict__ vsz, float qmax, int per_head) {
  static_assert(EXT_LIST >= SELECT_LDS_WORDS, "the histograms of the way out take the list's place");
  const int N = H * D;
  // (a view of the batch element's H * n rows: heads past H read as 0)
  const GEAR_BUF_T vb = GEAR_BUF_MAKE(V + (size_t)b * H * n * D, (uint32_t)H * n * (D * 2));
  const int lane = lane_id(), hsub = lane >> 4, oc = lane & 15;
  const uint32_t off0 = ((uint32_t)hsub * n + t) * (D * 2) + oc * 16;
  uint4 x[NC];
  auto load_row = [&]() {
#pragma unroll
    for (int ch = 0; ch < NC; ++ch) x[ch] = GEAR_BUF_LOAD16(vb, off0 + (uint32_t)ch * 4u * n * (D * 2));
  };
  load_row();
  const bool filt = !per_head && (k_top > 0 || k_bot > 0);
  if (filt && !wave_ext_select<NC>(x, H, k_top, k_bot, raw, list)) {
#pragma unroll
    for (int ch = 0; ch < NC; ++ch) x[ch] = make_uint4(key16x2(x[ch].x), key16x2(x[ch].y), key16x2(x[ch].z), key16x2(x[ch].w));
    RegSource<NC> src{x};
    const ThreshPair tp = pack_thresh(wave_select(src, N, k_top, k_bot, list, true));
    const ThreshKeys tk = key_thresh(tp);
    const bool cut = __ballot(tk.cut) != 0ull;   // wave-uniform
#pragma unroll
    for (int ch = 0; ch < NC; ++ch) {
      reinterpret_cast<uint8_t*>(list)[(ch * 4 + hsub) * 16 + oc] =
          (uint8_t)(cut ? piece_bits(x[ch], (uint32_t)(ch * 512 + lane * 8), tp) : key_bits(x[ch], tk));
      GEAR_SCHED_FENCE();
    }
    wave_lds_sync();
    if (vsz) load_row();
  }
  if (filt && mask) store_token_mask(list, mask, b, H, n, t);
  if (vsz) {
    uint32_t mn = 0x7C007C00u, mx = 0xFC00FC00u;
#pragma unroll
    for (int ch = 0; ch < NC; ++ch) {
      uint32_t f = 0u;
      if (filt) f = reinterpret_cast<const uint8_t*>(list)[(ch * 4 + hsub) * 16 + oc];
      if (per_head) {
        const uint32_t kw[4] = {key16x2(x[ch].x), key16x2(x[ch].y), key16x2(x[ch].z), key16x2(x[ch].w)};
        const ThreshPair tp = row16_thresholds(kw, oc, k_top, k_bot);   // this head's own thresholds
        f = piece_bits(make_uint4(kw[0], kw[1], kw[2], kw[3]), (uint32_t)(oc * 8), tp);
      }
      if (ch * 4 + hsub < H) extend_extremes(drop_entries(x[ch], f), mx, mn);
    }
    mn = key16x2(mn);
    mx = key16x2(mx);
    uint32_t kmn = min(mn & 0xFFFFu, mn >> 16), kmx = max(mx & 0xFFFFu, mx >> 16);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      kmn = min(kmn, (uint32_t)__shfl_xor(kmn, o, 64));
      kmx = max(kmx, (uint32_t)__shfl_xor(kmx, o, 64));
    }
    if (lane == 0) vsz[(size_t)b * n + t] = group_bits(make_group(h2f(unkey16(kmn)), h2f(unkey16(kmx)), qmax));
  }
}

}  // namespace gear
