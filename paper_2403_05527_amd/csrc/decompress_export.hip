// gear_decompress (X-hat = D + A B^T + S, Algorithm 1) and the canonical export
// views of the stored components.
#include "gear_internal.h"
#include "gear_launch.h"

namespace gear {

__global__ void fill_u32_kernel(uint32_t* p, uint32_t v, size_t count) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x)
    p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t v, size_t count, hipStream_t st) {
  if (count == 0) return hipSuccess;
  size_t blocks = (count + 255) / 256;
  if (blocks > 65535) blocks = 65535;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, v, count);
  return hipGetLastError();
}

__device__ __forceinline__ uint32_t load_code(const SegView& sv, const Dims& dm, bool is_k, int slab, int t,
                                              int c) {
  const uint32_t cmask = (1u << dm.bits) - 1u;
  if (is_k) {
    const int per = 32 / dm.bits;
    const uint32_t w = sv.codes[((size_t)slab * sv.n_cap + t) * dm.wpr + c / per];
    return (w >> ((c % per) * dm.bits)) & cmask;
  }
  const int tgg = t / dm.tpw, i = t - tgg * dm.tpw;
  const uint32_t w =
      sv.codes[((size_t)slab * sv.nblk_cap + (tgg >> 2)) * 512 + ((tgg & 3) * 16 + (c & 15)) * 8 + (c >> 4)];
  return (w >> (i * dm.bits)) & cmask;
}
__device__ __forceinline__ uint32_t load_sz(const SegView& sv, const Dims& dm, bool is_k, int slab, int t, int c) {
  if (is_k) return sv.sz[((size_t)slab * sv.ng_cap + key_group(dm, t)) * D + c];
  return sv.sz[((size_t)slab * sv.n_cap + t) * (D / dm.g) + c / dm.g];
}

// Calls f(row in the tile, channel, fp16 bits) for every filled fixed slot of one
// 64-token tile; the slots are spread over the 256 threads of the block.
template <class F>
__device__ __forceinline__ void for_each_ell(const SegView& sv, int is_k, int slab, int tile, int tid, F&& f) {
  if (is_k) {
    for (int i = tid; i < TILE * ELL_K; i += 256) {
      const int tl = i / ELL_K, t = tile * TILE + tl;
      if (t >= sv.n) continue;
      const uint32_t en = sv.ell[((size_t)slab * sv.n_cap + t) * ELL_K + (i % ELL_K)];
      if (en & ELL_VALID) f(tl, (int)(en & 127u), en >> 16);
    }
  } else {
    for (int i = tid; i < D * ELL_V; i += 256) {
      const int c = i / ELL_V;
      const uint32_t en = sv.ell[(((size_t)slab * sv.ntile_cap + tile) * D + c) * ELL_V + (i % ELL_V)];
      if ((en & ELL_VALID) && tile * TILE + (int)(en & 63u) < sv.n) f((int)(en & 63u), c, en >> 16);
    }
  }
}

// ---- decompress: X-hat = D + A B^T + S of one 64-token tile ----
// The floor is HBM (2 bytes written per entry, about 0.45 read).  A thread owns eight neighbouring channels, i.e. one
// 16-byte piece of each of four or eight neighbouring rows; the 16 lanes of a row write its 256 bytes together.  A Value's tokens lie in
// one code word per channel: eight words give the row pieces, with no exchange between lanes.
// S goes through an fp16 tile in LDS (entries off its support are 0) because its slots and lists belong to rows (Keys)
// or channels (Values) and not to the piece's owner.  To keep the arithmetic under the write stream, codes become
// floats a byte at a time (no bit-field extract per entry) and the rank sum runs on the fp16 factors as they are
// stored, two ranks per instruction.  Every load that does not depend on the list table is requested before the first
// wait.
// What bounded it was the number of load instructions (26 for the four row pieces a thread had): so factors and Value parameters come in
// whole 16-byte pieces, and on a full chip a thread's channels' words and factors serve eight rows (decompress_rows).  Keys and Values together, four
// rows -> four rows with whole pieces -> eight rows: 16 x 32 heads x 4096 tokens of rank 4 (1.34 GB moved) at 2 bits 363 -> 321 -> 285 us (4.7 TB/s), at 4
// bits 358 -> 300 -> 261, 7 x 40 x 1777 at 4 bits 66 -> 56 -> 57, 32 x 32768 of rank 8 189 -> 179 -> 120, 64 x 8192 in groups of 32 88 -> 55 -> 57; stored
// without the non-temporal hint 289, 272, 75, 175, 80. A thread has two entries
// of the list in flight: large grids at 15 % outliers take 0.87 of the time that they took with one, those of up to 5 % 0.98 to 1.0 (four: 0.88, and 1.00 to 1.01).
// R: the rank rounded up to 0, 2, 4 or 8; NW = R / 2 words of two factors.
template <int R>
struct FactorRow {
  uint32_t w[R > 0 ? R / 2 : 1];
};
// Row `row` of a rank-`rank` factor through a view of its rows (zeros past the view); entries r >= rank are 0.
template <int R>
__device__ __forceinline__ FactorRow<R> load_factor(GEAR_BUF_T view, int row, int rank) {
  FactorRow<R> f;
  if constexpr (R == 0) {
    f.w[0] = 0u;
  } else if (rank == R) {   // (the same in every thread of the launch) one 4-, 8- or 16-byte read
    if constexpr (R == 2) {
      f.w[0] = GEAR_BUF_LOAD4(view, row * 4);
    } else if constexpr (R == 4) {
      const uint2 t = GEAR_BUF_LOAD8(view, row * 8);
      f.w[0] = t.x; f.w[1] = t.y;
    } else {
      const uint4 t = GEAR_BUF_LOAD16(view, row * 16);
      f.w[0] = t.x; f.w[1] = t.y; f.w[2] = t.z; f.w[3] = t.w;
    }
  } else {
    uint32_t h[R];
#pragma unroll
    for (int r = 0; r < R; ++r) h[r] = GEAR_BUF_LOAD2(view, (row * rank + r) * 2);
#pragma unroll
    for (int r = 0; r < R; r += 2) f.w[r / 2] = (r < rank ? h[r] : 0u) | ((r + 1 < rank ? h[r + 1] : 0u) << 16);
  }
  return f;
}
// N rows from `row` on (a multiple of N, N R / 8 a whole number or 1): in 16-byte reads where they are stored in a piece.  The view ends with a
// whole piece.
template <int R, int N>
__device__ __forceinline__ void load_factors(GEAR_BUF_T view, int row, int rank, FactorRow<R> (&f)[N]) {
  if constexpr (R == 2 || R == 4) {
    if (rank == R) {   // (the same in every thread of the launch)
      uint32_t w[N * R / 2];
#pragma unroll
      for (int i = 0; i < N * R / 8; ++i) {
        const uint4 t = GEAR_BUF_LOAD16(view, row * (2 * R) + 16 * i);
        w[4 * i] = t.x; w[4 * i + 1] = t.y; w[4 * i + 2] = t.z; w[4 * i + 3] = t.w;
      }
#pragma unroll
      for (int e = 0; e < N; ++e)
#pragma unroll
        for (int i = 0; i < R / 2; ++i) f[e].w[i] = w[e * (R / 2) + i];
      return;
    }
  }
#pragma unroll
  for (int e = 0; e < N; ++e) f[e] = load_factor<R>(view, row + e, rank);
}
// Eight entries of one row: code * scale + zero, + A B^T, + S, in fp32 in this order, then fp16.
// c0, c1: the codes of entries 0..3 and 4..7, one per byte.
template <int R>
__device__ __forceinline__ uint4 decompress_piece(uint32_t c0, uint32_t c1, const float (&dl)[8], const float (&mn)[8],
                                                  const FactorRow<R>& a, const FactorRow<R> (&bf)[8], const uint4& sp) {
  const uint32_t sw[4] = {sp.x, sp.y, sp.z, sp.w};
  uint32_t o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float v[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int e = 2 * j + h;
      float x = (float)(((e < 4 ? c0 : c1) >> (8 * (e & 3))) & 0xFFu) * dl[e] + mn[e];
      if constexpr (R > 0) {
#pragma unroll
        for (int i = 0; i < R / 2; ++i) x = GEAR_FDOT2(a.w[i], bf[e].w[i], x);
      }
      v[h] = x + h2f(h ? (sw[j] >> 16) : (sw[j] & 0xFFFFu));
    }
    const h2_t p = {(_Float16)v[0], (_Float16)v[1]};
    o[j] = __builtin_bit_cast(uint32_t, p);
  }
  return make_uint4(o[0], o[1], o[2], o[3]);
}
constexpr int SP_PITCH = D + 8;   // fp16 entries per row of the S tile (16-byte pieces of neighbouring rows in different banks)
constexpr int dec_threads(int rows) { return TILE * (D / 8) / rows; }   // rows: of a thread

// grid (ceil(n/64), B*H), block dec_threads(ROWS).
template <bool IS_K, int BITS, int R, int ROWS>
__global__ __launch_bounds__(dec_threads(ROWS)) void decompress_kernel(Dims dm, SegView sv, uint16_t* __restrict__ out, int n_total) {
  constexpr int THREADS = dec_threads(ROWS), TPW = 32 / BITS;
  constexpr int NWG = TILE / TPW;   // Values: code words of a channel in the tile
  constexpr uint32_t CMASK = BITS == 2 ? 0x03030303u : 0x0F0F0F0Fu;
  __shared__ __align__(16) uint16_t sp[TILE * SP_PITCH];
  const int slab = blockIdx.y, tile = blockIdx.x, t0 = tile * TILE;
  const int tid = threadIdx.x, oc = tid & 15, q = tid >> 4;
  const int lg = 31 - __clz(dm.g), lng = 7 - lg;   // log2 of the group size, of a Value row's groups
  const bool sparse = dm.ppm > 0;
  // the thread's rows of the tile: row0 .. row0 + ROWS - 1 (a Value's lie in one code word per channel: all of it, or a part)
  const int wg = q & (NWG - 1), part = q / NWG;   // Values
  const int row0 = IS_K ? ROWS * q : wg * TPW + ROWS * part;
  // views of the slab's rows: what lies past the last row is not written (up to a whole piece of the rows' parameters is read)
  const GEAR_BUF_T ob = GEAR_BUF_MAKE(out + ((size_t)slab * n_total + sv.t0) * D, (uint32_t)sv.n * (D * 2));
  const GEAR_BUF_T ab = GEAR_BUF_MAKE(sv.A + (size_t)slab * sv.n_cap * sv.rank, ((uint32_t)sv.n * sv.rank * 2 + 15u) & ~15u);
  const GEAR_BUF_T bb = GEAR_BUF_MAKE(sv.Bf + (size_t)slab * D * sv.rank, (uint32_t)(D * 2) * sv.rank);
  uint2 tab = make_uint2(0u, 0u);
  constexpr int SLOTS = TILE * ELL_K / THREADS;   // the thread's fixed slots of the tile
  static_assert(TILE * ELL_K == D * ELL_V && (SLOTS == 1 || SLOTS == 2), "one or two slots per thread");
  uint32_t slot[2] = {0u, 0u};
  if (sparse) {
    tab = sv.sp_table[(size_t)slab * sv.ntile_cap + tile];
    // (a Key segment's last rows may not all exist)
    const uint32_t* ell = sv.ell + ((size_t)slab * sv.ntile_cap + tile) * (D * ELL_V) + SLOTS * tid;   // Values
    const GEAR_BUF_T eb = GEAR_BUF_MAKE(sv.ell + (size_t)slab * sv.n_cap * ELL_K, (uint32_t)sv.n * (ELL_K * 4));
    if constexpr (SLOTS == 2) {
      uint2 t;
      if constexpr (IS_K) t = GEAR_BUF_LOAD8(eb, (t0 * ELL_K + 2 * tid) * 4);
      else t = *reinterpret_cast<const uint2*>(ell);
      slot[0] = t.x;
      slot[1] = t.y;
    } else {
      if constexpr (IS_K) slot[0] = GEAR_BUF_LOAD4(eb, (t0 * ELL_K + tid) * 4);
      else slot[0] = *ell;
    }
  }
  uint32_t cw[8];          // Keys: cw[k] the 8 codes of row k; Values: cw[e] the word of channel 8 oc + e
  uint32_t zv[ROWS];   // Values: (scale, zero) of the rows
  uint4 zk[2];             // Keys: (scale, zero) of the channels in the rows' group
  FactorRow<R> a[ROWS], bf[8];
  if constexpr (IS_K) {
    const GEAR_BUF_T cb = GEAR_BUF_MAKE(sv.codes + (size_t)slab * sv.n_cap * (4 * BITS), (uint32_t)sv.n * (16 * BITS));
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      const int t = t0 + row0 + k;
      cw[k] = BITS == 4 ? GEAR_BUF_LOAD4(cb, t * 64 + oc * 4) : GEAR_BUF_LOAD2(cb, t * 32 + oc * 2);
    }
    const int g0 = dm.kcvt ? 0 : (t0 + row0) >> lg;
    const GEAR_BUF_T zb = GEAR_BUF_MAKE(sv.sz + (size_t)slab * sv.ng_cap * D, (uint32_t)sv.ng_cap * (D * 4));
#pragma unroll
    for (int h = 0; h < 2; ++h) zk[h] = GEAR_BUF_LOAD16(zb, (g0 * D + oc * 8) * 4 + 16 * h);
  } else {
    // (a tile's last code block may lie past the segment: nothing of it is used then)
    const int blk = (t0 / TPW + wg) >> 2;
    const GEAR_BUF_T cb = GEAR_BUF_MAKE(sv.codes + (size_t)slab * sv.nblk_cap * 512, (uint32_t)sv.nblk_cap * 2048);
#pragma unroll
    for (int e = 0; e < 8; ++e) cw[e] = GEAR_BUF_LOAD4(cb, (blk * 512 + (wg & 3) * 128 + ((oc & 1) * 8 + e) * 8 + (oc >> 1)) * 4);
    const GEAR_BUF_T zb = GEAR_BUF_MAKE(sv.sz + (((size_t)slab * sv.n_cap) << lng), (((uint32_t)sv.n << lng) * 4 + 15u) & ~15u);
    const int G = (oc * 8) >> lg;
    if (lng == 0) {
#pragma unroll
      for (int k = 0; k < ROWS; k += 4) {
        const uint4 z = GEAR_BUF_LOAD16(zb, (t0 + row0 + k) * 4);
        zv[k] = z.x; zv[k + 1] = z.y; zv[k + 2] = z.z; zv[k + 3] = z.w;
      }
    } else if (lng == 1) {
#pragma unroll
      for (int k = 0; k < ROWS; k += 2) {
        const uint4 z = GEAR_BUF_LOAD16(zb, (t0 + row0 + k) * 8);
        zv[k] = G ? z.y : z.x;
        zv[k + 1] = G ? z.w : z.z;
      }
    } else {
#pragma unroll
      for (int k = 0; k < ROWS; ++k) zv[k] = GEAR_BUF_LOAD4(zb, (((t0 + row0 + k) << lng) + G) * 4);
    }
  }
  load_factors<R, ROWS>(ab, t0 + row0, sv.rank, a);
  load_factors<R, 8>(bb, oc * 8, sv.rank, bf);

  if (sparse) {
    for (int i = tid; i < TILE * SP_PITCH / 8; i += THREADS) reinterpret_cast<uint4*>(sp)[i] = make_uint4(0, 0, 0, 0);
    block_lds_sync();
    const uint32_t* lst = sv.sp_pool + (size_t)(IS_K ? slab : slab / dm.H) * sv.pool_cap + tab.x;
    auto place = [&](uint32_t en) { sp[((en & 0xFFFFu) >> 7) * SP_PITCH + (en & 127u)] = (uint16_t)(en >> 16); };
    for (uint32_t e = tid; e < tab.y; e += 2 * THREADS) {   // (two of a thread's entries in flight)
      const bool more = e + THREADS < tab.y;
      const uint32_t en = lst[e], en2 = more ? lst[e + THREADS] : 0u;
      place(en);
      if (more) place(en2);
    }
#pragma unroll
    for (int h = 0; h < SLOTS; ++h) {
      if (slot[h] & ELL_VALID) {
        const int i = SLOTS * tid + h, tl = IS_K ? i / ELL_K : (int)(slot[h] & 63u), c = IS_K ? (int)(slot[h] & 127u) : i / ELL_V;
        sp[tl * SP_PITCH + c] = (uint16_t)(slot[h] >> 16);
      }
    }
    block_lds_sync();
  }
  // Values: the codes of channels 4 h .. 4 h + 3 a byte position at a time: bytes of tokens row0 + 4 p .. (2 bits), row0 + 2 p .. (4 bits)
  constexpr int NB = IS_K ? 1 : ROWS * BITS / 8;
  uint32_t cb4[NB][2];
  if constexpr (!IS_K) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int p = 0; p < NB; p += 2) {   // bytes p, p + 1 of my part of the words
        const uint32_t s2 = 0x05010400u + 0x01010101u * (uint32_t)(NB * part + p);   // (lo[p], hi[p], lo[p + 1], hi[p + 1])
        const uint32_t x = GEAR_BYTE_PERM(cw[4 * h + 1], cw[4 * h], s2), y = GEAR_BYTE_PERM(cw[4 * h + 3], cw[4 * h + 2], s2);
        cb4[p][h] = GEAR_BYTE_PERM(y, x, 0x05040100u);
        if (p + 1 < NB) cb4[p + 1][h] = GEAR_BYTE_PERM(y, x, 0x07060302u);
      }
    }
  }
  float dl[8], mn[8];
  if constexpr (IS_K) {
    const uint32_t w[8] = {zk[0].x, zk[0].y, zk[0].z, zk[0].w, zk[1].x, zk[1].y, zk[1].z, zk[1].w};
#pragma unroll
    for (int e = 0; e < 8; ++e) { dl[e] = h2f(w[e] & 0xFFFFu); mn[e] = h2f(w[e] >> 16); }
  }
#pragma unroll
  for (int k = 0; k < ROWS; ++k) {
    const int tl = row0 + k;
    uint32_t c0, c1;
    if constexpr (IS_K) {
      if constexpr (BITS == 2) {
        // codes e = 0..3 in byte 0, 4..7 in byte 1: spread two bits per byte
        const uint32_t lo = cw[k] & 0xFFu, hi = cw[k] >> 8;
        c0 = (lo | (lo << 6) | (lo << 12) | (lo << 18)) & CMASK;
        c1 = (hi | (hi << 6) | (hi << 12) | (hi << 18)) & CMASK;
      } else {
        const uint32_t ev = cw[k] & CMASK, od = (cw[k] >> 4) & CMASK;   // codes 0 2 4 6 and 1 3 5 7
        c0 = GEAR_BYTE_PERM(od, ev, 0x05010400u);
        c1 = GEAR_BYTE_PERM(od, ev, 0x07030602u);
      }
    } else {
      const float d = h2f(zv[k] & 0xFFFFu), m = h2f(zv[k] >> 16);
#pragma unroll
      for (int e = 0; e < 8; ++e) { dl[e] = d; mn[e] = m; }
      constexpr int PER = 8 / BITS;   // tokens of a byte
      c0 = (cb4[k / PER][0] >> (BITS * (k % PER))) & CMASK;
      c1 = (cb4[k / PER][1] >> (BITS * (k % PER))) & CMASK;
    }
    const uint4 s4 = sparse ? *reinterpret_cast<const uint4*>(sp + tl * SP_PITCH + oc * 8) : make_uint4(0, 0, 0, 0);
    GEAR_BUF_STORE16_NT(ob, (uint32_t)(t0 + tl) * (D * 2) + oc * 16, decompress_piece<R>(c0, c1, dl, mn, a[k], bf, s4));
  }
}

// grid (ceil(n/64), B*H), block 256.
__global__ __launch_bounds__(256) void export_codes_kernel(Dims dm, SegView sv, int is_k, uint8_t* __restrict__ codes,
                                                           uint16_t* __restrict__ scale, uint16_t* __restrict__ zero,
                                                           int n_total, int ng_total) {
  const int slab = blockIdx.y, tile = blockIdx.x, tid = threadIdx.x;
  for (int i = tid; i < TILE * D; i += 256) {
    const int tl = i / D, c = i % D, t = tile * TILE + tl;
    if (t >= sv.n) break;
    codes[((size_t)slab * n_total + sv.t0 + t) * D + c] = (uint8_t)load_code(sv, dm, is_k, slab, t, c);
    const uint32_t sb = load_sz(sv, dm, is_k, slab, t, c);
    if (is_k) {
      if (dm.kcvt ? t == 0 : t % dm.g == 0) {
        const size_t o = ((size_t)slab * ng_total + sv.g0 + key_group(dm, t)) * D + c;
        scale[o] = (uint16_t)(sb & 0xFFFFu);
        zero[o] = (uint16_t)(sb >> 16);
      }
    } else if (c % dm.g == 0) {
      const size_t o = ((size_t)slab * n_total + sv.t0 + t) * (D / dm.g) + c / dm.g;
      scale[o] = (uint16_t)(sb & 0xFFFFu);
      zero[o] = (uint16_t)(sb >> 16);
    }
  }
}

// grid (ceil(n/64), B*H), block 256.  Outputs must be zero-filled beforehand.
__global__ __launch_bounds__(256) void export_sparse_kernel(Dims dm, SegView sv, int is_k, uint8_t* __restrict__ mask,
                                                            uint16_t* __restrict__ vals, int n_total) {
  const int slab = blockIdx.y, tile = blockIdx.x, tid = threadIdx.x;
  const int b = slab / dm.H;
  const uint2 oc = sv.sp_table[(size_t)slab * sv.ntile_cap + tile];
  const uint32_t* lst = sv.sp_pool + (size_t)(is_k ? slab : b) * sv.pool_cap + oc.x;
  for (uint32_t e = tid; e < oc.y; e += 256) {
    const uint32_t en = lst[e];
    const int t = tile * TILE + (int)((en & 0xFFFFu) >> 7), c = en & 127u;
    if (t < sv.n) {
      const size_t o = ((size_t)slab * n_total + sv.t0 + t) * D + c;
      mask[o] = 1;
      vals[o] = (uint16_t)(en >> 16);
    }
  }
  for_each_ell(sv, is_k, slab, tile, tid, [&](int tl, int c, uint32_t hb) {
    const size_t o = ((size_t)slab * n_total + sv.t0 + tile * TILE + tl) * D + c;
    mask[o] = 1;
    vals[o] = (uint16_t)hb;
  });
}

// ---- COO view of S: (linear index into [B, H, n_total, 128], fp16 value), sorted by index ----
// Pass 1 (count = 1) leaves the number of outliers of every token row in rowcnt[slab * n_total + t];
// after the prefix sums, pass 2 (count = 0) writes each row's entries in channel order from rowcnt[row]
// (then the row's first position).  grid (ceil(n/64), B*H), block 256: the tile's part of S is
// rebuilt in LDS as a bit per entry plus its value.
__global__ __launch_bounds__(256) void coo_tile_kernel(Dims dm, SegView sv, int is_k, int count, uint32_t* __restrict__ rowcnt,
                                                       long long* __restrict__ lin, uint16_t* __restrict__ vals, int n_total) {
  __shared__ uint32_t bits[TILE][4];
  __shared__ uint16_t val[TILE][D];
  const int slab = blockIdx.y, tile = blockIdx.x, tid = threadIdx.x;
  const int b = slab / dm.H;
  if (tid < TILE * 4) (&bits[0][0])[tid] = 0u;
  block_lds_sync();
  auto put = [&](int tl, int c, uint32_t hb) {
    atomicOr(&bits[tl][c >> 5], 1u << (c & 31));
    val[tl][c] = (uint16_t)hb;
  };
  if (dm.ppm > 0) {
    const uint2 oc = sv.sp_table[(size_t)slab * sv.ntile_cap + tile];
    const uint32_t* lst = sv.sp_pool + (size_t)(is_k ? slab : b) * sv.pool_cap + oc.x;
    for (uint32_t e = tid; e < oc.y; e += 256) {
      const uint32_t en = lst[e];
      const int tl = (int)((en & 0xFFFFu) >> 7);
      if (tile * TILE + tl < sv.n) put(tl, (int)(en & 127u), en >> 16);
    }
    for_each_ell(sv, is_k, slab, tile, tid, put);
  }
  block_lds_sync();
  if (tid < TILE && tile * TILE + tid < sv.n) {
    const size_t row = (size_t)slab * n_total + sv.t0 + tile * TILE + tid;
    if (count) {
      rowcnt[row] = __popc(bits[tid][0]) + __popc(bits[tid][1]) + __popc(bits[tid][2]) + __popc(bits[tid][3]);
    } else {
      size_t o = rowcnt[row];
      for (int w = 0; w < 4; ++w) {
        uint32_t m = bits[tid][w];
        while (m) {
          const int c = 32 * w + __ffs((int)m) - 1;
          m &= m - 1u;
          lin[o] = (long long)(row * D + c);
          vals[o] = val[tid][c];
          ++o;
        }
      }
    }
  }
}

// Exclusive prefix sums of v[0 .. count) in place, in three launches: sums of chunks of 1024,
// their prefix sums (one block), then each chunk's own scan.
__global__ __launch_bounds__(256) void scan_chunk_sums_kernel(const uint32_t* __restrict__ v, size_t count, uint32_t* __restrict__ sums) {
  __shared__ uint32_t red[4];
  const size_t base = (size_t)blockIdx.x * 1024;
  uint32_t s = 0;
  for (int i = threadIdx.x; i < 1024; i += 256)
    if (base + i < count) s += v[base + i];
  s = wave_sum_shfl(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  block_lds_sync();
  if (threadIdx.x == 0) sums[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}
__global__ __launch_bounds__(256) void scan_sums_kernel(uint32_t* __restrict__ sums, int nchunks) {   // one block
  __shared__ uint32_t wtot[4];
  __shared__ uint32_t carry_s;
  if (threadIdx.x == 0) carry_s = 0u;
  block_lds_sync();
  for (int i0 = 0; i0 < nchunks; i0 += 256) {
    const int i = i0 + threadIdx.x;
    const uint32_t x = i < nchunks ? sums[i] : 0u;
    const uint32_t inc = wave_incl_scan(x);
    if ((threadIdx.x & 63) == 63) wtot[threadIdx.x >> 6] = inc;
    block_lds_sync();
    uint32_t off = carry_s;
    for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) off += wtot[w];
    if (i < nchunks) sums[i] = off + inc - x;
    block_lds_sync();
    if (threadIdx.x == 255) carry_s = off + inc;
    block_lds_sync();
  }
}
__global__ __launch_bounds__(256) void scan_apply_kernel(uint32_t* __restrict__ v, size_t count, const uint32_t* __restrict__ sums) {
  __shared__ uint32_t wtot[4];
  const size_t base = (size_t)blockIdx.x * 1024 + (size_t)threadIdx.x * 4;
  uint32_t x[4], t = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[i] = base + i < count ? v[base + i] : 0u;
    t += x[i];
  }
  const uint32_t inc = wave_incl_scan(t);
  if ((threadIdx.x & 63) == 63) wtot[threadIdx.x >> 6] = inc;
  block_lds_sync();
  uint32_t off = sums[blockIdx.x] + inc - t;
  for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) off += wtot[w];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (base + i < count) v[base + i] = off;
    off += x[i];
  }
}

__global__ void export_lowrank_kernel(SegView sv, uint16_t* __restrict__ A, uint16_t* __restrict__ Bf, int slabs) {
  const size_t na = (size_t)slabs * sv.n * sv.rank, nb = (size_t)slabs * D * sv.rank;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < na + nb; i += (size_t)gridDim.x * blockDim.x) {
    if (i < na) {
      const size_t per = (size_t)sv.n * sv.rank;
      const size_t slab = i / per, r = i - slab * per;
      A[i] = sv.A[slab * sv.n_cap * sv.rank + r];
    } else {
      Bf[i - na] = sv.Bf[i - na];
    }
  }
}

template <bool IS_K, int BITS, int ROWS>
static void launch_decompress_t(const Dims& dm, const SegView& sv, uint16_t* out, int n_total, hipStream_t st) {
  const dim3 grid((sv.n + TILE - 1) / TILE, dm.B * dm.H), block(dec_threads(ROWS));
  if (sv.rank == 0) hipLaunchKernelGGL((decompress_kernel<IS_K, BITS, 0, ROWS>), grid, block, 0, st, dm, sv, out, n_total);
  else if (sv.rank <= 2) hipLaunchKernelGGL((decompress_kernel<IS_K, BITS, 2, ROWS>), grid, block, 0, st, dm, sv, out, n_total);
  else if (sv.rank <= 4) hipLaunchKernelGGL((decompress_kernel<IS_K, BITS, 4, ROWS>), grid, block, 0, st, dm, sv, out, n_total);
  else hipLaunchKernelGGL((decompress_kernel<IS_K, BITS, 8, ROWS>), grid, block, 0, st, dm, sv, out, n_total);
}
// Rows of a thread, 4 or 8.  Eight halve the loads of codes and factors, four have twice the waves and half the chain.  Times of four rows to those of
// eight, Keys and Values, nothing of the cache in the chip's caches; by tiles (of 64 tokens, all slabs):
//   tiles         up to 512      to 768      to 1024     to 1536     to 8192       more
//   rank 0        0.87 to 0.98   0.96        0.98        1.06        0.99 to 1.04  1.01; where the cache is near 0.91 to 0.99 up to 8192 tiles,
//                 0.98 to 1.0 at 16384, 1.01 to 1.07 from 30000 (64 x 2048 tokens at 5 % 14.2 : 15.2 us, 512 x 8192 484 : 458): hence its line
//   rank 1        0.87 to 0.98   1.05        1.06        1.09        1.13          1.32
//   rank 2, 4     0.75 to 0.97   0.88, 0.95  0.94, 0.98  1.02, 1.08  0.96 to 1.10  1.07
//   rank 8        0.76 to 0.89   0.92        0.99        1.03        0.99 to 1.10  1.22  (where the cache is near, 1.16 at 1024)
//   others        1.0 to 1.3 up to 256 tiles, 1.2 to 1.85 beyond, where the cache is near (a row's factors are several loads)
// The more entries in lists, which 128 threads fetch half as fast, the less eight gain where factors come in whole pieces: level at 15 % outliers (rank 0
// 0.93), and 149 : 178 us at 40 % (12 x 16 x 4052, rank 4).  Tiles of few rows (segments of up to 110 tokens) do not count as whole ones for these
// ranks: 0.90 to 0.97 up to 7000 of them.
static int decompress_rows(const Dims& dm, const SegView& sv) {
  const long long tiles = (long long)((sv.n + TILE - 1) / TILE) * dm.B * dm.H, rows = (long long)sv.n * dm.B * dm.H;
  switch (sv.rank) {
    case 0: return tiles > 24 * 1024 && dm.ppm <= 100000 ? 8 : 4;
    case 2: case 4: return rows > 1024 * TILE && dm.ppm <= 100000 ? 8 : 4;
    case 1: return tiles > 512 ? 8 : 4;
    case 8: return tiles > 768 ? 8 : 4;
    default: return 8;
  }
}
template <bool IS_K, int BITS>
static void launch_decompress_r(const Dims& dm, const SegView& sv, uint16_t* out, int n_total, hipStream_t st) {
  if (decompress_rows(dm, sv) == 4) launch_decompress_t<IS_K, BITS, 4>(dm, sv, out, n_total, st);
  else launch_decompress_t<IS_K, BITS, 8>(dm, sv, out, n_total, st);
}

hipError_t launch_decompress(const Dims& dm, const SegView& ks, const SegView& vs, uint16_t* Kout,
                             uint16_t* Vout, int n_total, hipStream_t st) {
  if (dm.bits == 2) {
    if (Kout) launch_decompress_r<true, 2>(dm, ks, Kout, n_total, st);
    if (Vout) launch_decompress_r<false, 2>(dm, vs, Vout, n_total, st);
  } else {
    if (Kout) launch_decompress_r<true, 4>(dm, ks, Kout, n_total, st);
    if (Vout) launch_decompress_r<false, 4>(dm, vs, Vout, n_total, st);
  }
  return hipGetLastError();
}

hipError_t launch_export_codes(const Dims& dm, const SegView& sv, bool is_k, uint8_t* codes, uint16_t* scale,
                               uint16_t* zero, int n_total, int ng_total, hipStream_t st) {
  dim3 grid((sv.n + TILE - 1) / TILE, dm.B * dm.H);
  hipLaunchKernelGGL(export_codes_kernel, grid, dim3(256), 0, st, dm, sv, is_k ? 1 : 0, codes, scale, zero,
                     n_total, ng_total);
  return hipGetLastError();
}

hipError_t launch_export_sparse(const Dims& dm, const SegView& sv, bool is_k, uint8_t* mask, uint16_t* vals,
                                int n_total, hipStream_t st) {
  if (dm.ppm == 0) return hipSuccess;
  dim3 grid((sv.n + TILE - 1) / TILE, dm.B * dm.H);
  hipLaunchKernelGGL(export_sparse_kernel, grid, dim3(256), 0, st, dm, sv, is_k ? 1 : 0, mask, vals, n_total);
  return hipGetLastError();
}

hipError_t launch_coo_tiles(const Dims& dm, const SegView& sv, bool is_k, bool count, uint32_t* rowcnt, long long* lin,
                            uint16_t* vals, int n_total, hipStream_t st) {
  dim3 grid((sv.n + TILE - 1) / TILE, dm.B * dm.H);
  hipLaunchKernelGGL(coo_tile_kernel, grid, dim3(256), 0, st, dm, sv, is_k ? 1 : 0, count ? 1 : 0, rowcnt, lin, vals, n_total);
  return hipGetLastError();
}

hipError_t launch_exclusive_scan(uint32_t* v, size_t count, uint32_t* sums, hipStream_t st) {
  const int nchunks = (int)((count + 1023) / 1024);
  if (nchunks == 0) return hipSuccess;
  hipLaunchKernelGGL(scan_chunk_sums_kernel, dim3(nchunks), dim3(256), 0, st, (const uint32_t*)v, count, sums);
  hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(256), 0, st, sums, nchunks);
  hipLaunchKernelGGL(scan_apply_kernel, dim3(nchunks), dim3(256), 0, st, v, count, (const uint32_t*)sums);
  return hipGetLastError();
}

hipError_t launch_export_lowrank(const Dims& dm, const SegView& sv, uint16_t* A, uint16_t* Bf, hipStream_t st) {
  if (sv.rank == 0) return hipSuccess;
  hipLaunchKernelGGL(export_lowrank_kernel, dim3(1024), dim3(256), 0, st, sv, A, Bf, dm.B * dm.H);
  return hipGetLastError();
}

}  // namespace gear
