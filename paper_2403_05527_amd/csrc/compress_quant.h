// Quant_b(X - S) (Eq. 2 / Eq. 5) of one tensor, its sparse matrix S in the stored form, and in the same pass the
// Gram matrix G = R^T R of the quantization residual R = X - S - D-hat that the power iteration works on (Algorithm 2:
// every round before the last maps B -> R^T (R B) = G B).
//
// The Filter kernels leave S as one bit per entry (16 bytes per token row), so this kernel reads X once and nothing
// between it and the last pass of the low-rank solver has the size of X: a filtered copy Y = X - S written here and
// read by a separate Gram pass made 4 tensor sizes of traffic out of 1 (Keys of 64 x 8 heads x 8192 tokens: 502 us for
// the quantizer that wrote Y plus 308 us for the Gram pass).
//
// A block walks a strip of tokens in tiles of 128 tokens x 128 channels.  Thread (r0 = tid / 16, oc = tid % 16) holds
// channels 8 oc .. 8 oc + 7 of the eight consecutive rows 8 r0 .. 8 r0 + 7:
//  * a Key group (32, 64 or 128 tokens of a channel) is 1, 2 or 4 whole waves, and min / max over a thread's rows are
//    packed fp16 instructions, two channels each; a Value group (32, 64 or 128 channels of a row) is 4, 8 or 16 lanes,
//    whose eight rows are reduced together, each exchange halving the rows a lane carries;
//  * the eight tokens of a channel that lie in one thread are consecutive, as the stored Value code words want them;
//  * as an MFMA operand, register j of "channel e" holds rows (2j, 2j+1) of channel 8 oc + e: operand e is the 16
//    channels {8 oc + e} x 32 tokens of the wave, and acc(e, f) += op_e^T op_f is one 16 x 16 tile of G: lane l,
//    register i <-> G[8 (4 (l/16) + i) + e][8 (l%16) + f].  Only the 36 tiles e <= f are computed (G is symmetric).
// The tile passes through LDS once, where the few outliers are looked up by row (Keys) or by channel (Values), put into
// their slots and lists, and zeroed: the arithmetic per entry then needs no mask.
//
// A residual entry enters the contraction as two fp16 numbers, its leading part and what that leaves (22 bits
// together), and a product as three MFMA terms (the lo lo' term is below fp32 resolution); accumulation is fp32.  The
// leading parts alone are not enough: without orthonormalisation between the rounds the weaker directions of
// G^(L-1) B0 are small differences of large numbers, and a relative error of 2^-11 in G is amplified by the square of
// the ratio of its leading eigenvalues.
#pragma once
#include "gear_internal.h"
#include "gear_select.h"
#include "gear_launch.h"

namespace gear {

constexpr int QT = 128;        // tokens per tile
constexpr int KLG_VEC = 15;    // Keys: "log2 of the group size" of the per-vector grouping (one group per segment)

typedef _Float16 quant_h8 __attribute__((ext_vector_type(8)));

// Exchanges between the two halves / the odd and even rows of 16 lanes of two registers: after lane_swap32 a holds
// (a of lanes 0..31, b of lanes 0..31), b holds (a of lanes 32..63, b of lanes 32..63); lane_swap16 does the same with
// the rows (0, 1) and (2, 3).
#ifndef GEAR_LANE_SWAP32
#define GEAR_LANE_SWAP32(a, b)                                                 \
  do {                                                                         \
    const auto r__ = __builtin_amdgcn_permlane32_swap((a), (b), false, false); \
    (a) = r__[0];                                                              \
    (b) = r__[1];                                                              \
  } while (0)
#define GEAR_LANE_SWAP16(a, b)                                                 \
  do {                                                                         \
    const auto r__ = __builtin_amdgcn_permlane16_swap((a), (b), false, false); \
    (a) = r__[0];                                                              \
    (b) = r__[1];                                                              \
  } while (0)
#endif

// (mx - mn) / (2^b - 1), correctly rounded: for these two divisors the product with the rounded reciprocal and one
// fused correction give the IEEE quotient for every normal fp32 numerator (checked over all mantissas).
template <int BITS>
__device__ __forceinline__ float div_levels(float x) {
#pragma clang fp contract(off)
  constexpr float q = (float)((1 << BITS) - 1);
  constexpr float y = 1.0f / q;
  const float q0 = __fmul_rn(x, y);
  float d = __builtin_fmaf(__builtin_fmaf(-q, q0, x), y, q0);
  GEAR_PIN_VGPR(d);   // (a conversion to fp16 that follows must see the fp32 value: fused with the last step it would round once)
  return d;
}
// make_group of gear_internal.h with the two divisions in their short forms (the same floats)
template <int BITS>
__device__ __forceinline__ GroupQ make_group_b(float mn, float mx) {
#pragma clang fp contract(off)
  GroupQ q;
  q.mn = mn + 0.0f;   // -0 -> +0
  q.delta = h2f(f2h(div_levels<BITS>(__fsub_rn(mx + 0.0f, q.mn))));
  q.inv = q.delta > 0.0f ? recip_of_half(q.delta) : 0.0f;
  return q;
}

struct QuantArgs {
  const uint16_t* X;     // [slab][n][128]
  SegView sv;
  Dims dm;
  int n, t_lr, strip;    // t_lr: rows before it take no part in the low-rank term; strip: tokens per block (a multiple of 128)
  uint4* mask;           // [slab][n]: bit c of a row = entry (row, c) belongs to S (Values with the Filter per head: written here)
  const uint32_t* vsz;   // Values, per-vector grouping: a token's (scale, zero)
  int k_top, k_bot;      // Values with the Filter per head: entries per vector
  uint32_t* pool_ctr;
  uint16_t* Yout;        // nullable: Y = X - S for the solvers that walk over it (short segments, a single round)
  float* gram;           // [slab][strip][36][4][64]
};

template <bool IS_K, int BITS, int LG>
struct QuantSmem;
template <int BITS, int LG>
struct QuantSmem<true, BITS, LG> {
  static constexpr int NG = LG >= 7 ? 1 : QT >> LG;   // groups per tile
  uint4 tile[QT][D / 8];
  uint4 rowmask[QT];
  uint4 slots[QT];
  uint32_t red_mn[4][D / 2], red_mx[4][D / 2];        // a wave's min / max of its 32 rows, two channels per word
  __attribute__((aligned(16))) uint2 par[NG][D];      // (scale, zero) as fp16, 1/scale
  uint32_t ovf_cnt[32], ovf_off[32];                  // overflow lists of the strip's 64-token tiles
};
template <int BITS, int LG>
struct QuantSmem<false, BITS, LG> {
  static constexpr int NG = D >> LG;                  // groups per row
  uint4 tile[QT][D / 8];
  uint4 rowmask[QT];
  uint4 colmask[D];                                   // bit t of channel c's 128 bits
  uint2 par[QT][NG];                                  // (scale, zero) as fp16, 1/scale
  uint4 codes[QT * D * BITS / 128];                   // code words in operand order
  uint32_t list_off[2];
};

template <bool IS_K, int BITS, int LG, bool GRAM>
union QuantLds {
  QuantSmem<IS_K, BITS, LG> s;
  float red[GRAM ? GRAM_FLOATS : 4];
};

// One block's strip of slab blockIdx.y, 256 threads.
template <bool IS_K, int BITS, int LG, bool GRAM>
__device__ __forceinline__ void quant_body(QuantLds<IS_K, BITS, LG, GRAM>& sm, const QuantArgs& a) {
  typedef QuantSmem<IS_K, BITS, LG> Smem;
  constexpr int NG = Smem::NG;
  constexpr float QMAX = (float)((1 << BITS) - 1);
  Smem& s = sm.s;
  const int slab = blockIdx.y, n = a.n;
  int tid = threadIdx.x;
  const int wave = GEAR_WAVE_UNIFORM(tid >> 6);
  int lane = tid & 63, r0 = tid >> 4, oc = tid & 15;
  const int t_begin = blockIdx.x * a.strip;
  const int t_end = t_begin + a.strip < n ? t_begin + a.strip : n;
  const bool filt = a.dm.ppm > 0;
  const bool vhead = !IS_K && a.dm.vhead != 0;
  const int b = slab / a.dm.H, h = slab - b * a.dm.H;
  const GEAR_BUF_T xb = GEAR_BUF_MAKE(a.X + (size_t)slab * n * D, (uint32_t)n * (D * 2));
  const GEAR_BUF_T mb = GEAR_BUF_MAKE(a.mask + (size_t)slab * n, filt && !vhead ? n * 16 : 0);   // (no bits yet: reads as 0)
  uint16_t* tile16 = reinterpret_cast<uint16_t*>(&s.tile[0][0]);
  float one = 1.0f;
  GEAR_PIN_SGPR(one);   // fma(fp16 value, one, float) is one mixed-precision instruction: conversion and addition together

  if constexpr (IS_K) {
    if (filt) {
      // where the overflow lists of the strip's 64-token tiles go: one allocation per strip
      const int ntile = (t_end - t_begin + TILE - 1) / TILE;
      for (int i = wave; i < ntile; i += 4) {
        const uint4 m = GEAR_BUF_LOAD16(mb, (t_begin + TILE * i + lane) * 16);
        const uint32_t tot = __popc(m.x) + __popc(m.y) + __popc(m.z) + __popc(m.w);
        const uint32_t sum = lane_bcast_u(wave_incl_scan(tot > ELL_K ? tot - ELL_K : 0u), 63);
        if (lane == 0) s.ovf_cnt[i] = sum;
      }
      block_lds_sync();
      if (wave == 0) {
        const uint32_t v = lane < ntile ? s.ovf_cnt[lane] : 0u;
        const uint32_t inc = wave_incl_scan(v);
        uint32_t off = 0;
        if (lane == 63) off = atomicAdd(&a.pool_ctr[slab], inc);
        off = lane_bcast_u(off, 63) + inc - v;
        if (lane < ntile) {
          s.ovf_off[lane] = off;
          a.sv.sp_table[(size_t)slab * a.sv.ntile_cap + t_begin / TILE + lane] = make_uint2(off, v);
        }
      }
    }
    if (LG == KLG_VEC) {   // per-vector grouping: the channel's one pair of this segment was found with its thresholds
      if (tid < D) {
        const GroupQ q = load_group(a.sv.sz[(size_t)slab * a.sv.ng_cap * D + tid]);
        s.par[0][tid] = make_uint2(group_bits(q), __float_as_uint(q.inv));
      }
      block_lds_sync();
    }
  }

  floatx4 acc[GRAM ? GRAM_TILES : 1];
#pragma unroll
  for (int i = 0; i < (GRAM ? GRAM_TILES : 1); ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};

  // the eight row pieces of a thread and half a row's mask; rows past the end read as 0
  uint32_t x[8][4];
  uint2 mk;
  auto load_row = [&](int base, int k) {
    const uint4 v = GEAR_BUF_LOAD16(xb, (base + 8 * r0 + k) * (D * 2) + oc * 16);
    x[k][0] = v.x; x[k][1] = v.y; x[k][2] = v.z; x[k][3] = v.w;
  };
  auto load_mask = [&](int base) { mk = GEAR_BUF_LOAD8(mb, base * 16 + tid * 8); };
#pragma unroll
  for (int k = 0; k < 8; ++k) load_row(t_begin, k);
  load_mask(t_begin);

  // Values: code words of the tile that starts at `base` from LDS to the arena (blocks of TB tokens, operand order);
  // every word of a block that holds at least one token is written (rows past n carry code 0)
  constexpr int TB = 128 / BITS;   // 64 (2 bits) or 32 (4 bits) tokens per block
  auto copy_codes = [&](int base) {
    if constexpr (!IS_K) {
      uint4* dst = reinterpret_cast<uint4*>(a.sv.codes + ((size_t)slab * a.sv.nblk_cap + base / TB) * 512);
#pragma unroll
      for (int i = 0; i < QT * D * BITS / 128 / 256; ++i) {
        const int p = tid + 256 * i;
        if (base + (p >> 7) * TB < n) dst[p] = s.codes[p];
      }
    }
  };

#pragma unroll 1
  for (int base = t_begin; base < t_end; base += QT) {
    const bool ragged = base + QT > n;   // block-uniform: only such a tile has rows past the end
    // (the addresses below are made anew in every tile: kept over the loop they would not fit next to the accumulators)
    GEAR_PIN_VGPR(tid);
    lane = tid & 63;
    r0 = tid >> 4;
    oc = tid & 15;
    if constexpr (!IS_K) {
      if (vhead && filt) {   // the Filter per head: the row's 16 lanes hold the whole vector
#pragma unroll 1
        for (int k = 0; k < 8; ++k) {
          // (the row pieces are read again: a loop over registers could not stay rolled)
          const uint4 v = GEAR_BUF_LOAD16(xb, (base + 8 * r0 + k) * (D * 2) + oc * 16);
          const uint32_t kw[4] = {key16x2(v.x), key16x2(v.y), key16x2(v.z), key16x2(v.w)};
          const ThreshPair tp = row16_thresholds(kw, oc, a.k_top, a.k_bot);
          uint32_t f = 0;
#pragma unroll
          for (int e = 0; e < 8; ++e) f |= (outlier(slot_key(kw, e), (uint32_t)(8 * oc + e), tp) ? 1u : 0u) << e;
          const int t = base + 8 * r0 + k;
          if (t >= n) f = 0u;
          else reinterpret_cast<uint8_t*>(a.mask + (size_t)slab * n + t)[oc] = (uint8_t)f;
          reinterpret_cast<uint8_t*>(&s.rowmask[8 * r0 + k])[oc] = (uint8_t)f;
        }
      }
    }
    if (!IS_K || filt) {
      if (filt) {
#pragma unroll
        for (int k = 0; k < 8; ++k) s.tile[8 * r0 + k][oc] = make_uint4(x[k][0], x[k][1], x[k][2], x[k][3]);
        if (!vhead) reinterpret_cast<uint2*>(s.rowmask)[tid] = mk;
        if (tid < QT) {
          uint32_t z = 0;
          GEAR_PIN_VGPR(z);   // (not a register quadruple of zeros over the whole loop)
          if constexpr (IS_K) s.slots[tid] = make_uint4(z, z, z, z);   // empty slots
          else s.colmask[tid] = make_uint4(z, z, z, z);
        }
      }
      block_lds_sync();
    }
    if constexpr (!IS_K) {
      if (base > t_begin) copy_codes(base - QT);
    }

    // ---- the tile's outliers: into slots and lists, and out of the tile
    if constexpr (IS_K) {
      // A token row: the first ELL_K in channel order take the row's fixed slots, the rest go to the 64-token tile's
      // overflow list, ordered (t, c).  Two threads per row, 64 channels each.
      if (filt) {
        static_assert(ELL_K == 4, "the row's slots are stored as one 16-byte word");
        const int row = tid >> 1, half = tid & 1;
        const uint4 m = s.rowmask[row];
        const uint32_t lo = __popc(m.x) + __popc(m.y), hi = __popc(m.z) + __popc(m.w);
        const uint32_t pre = half ? lo : 0u, cnt = half ? hi : lo;
        const uint32_t over = (pre + cnt > ELL_K ? pre + cnt - ELL_K : 0u) - (pre > ELL_K ? pre - ELL_K : 0u);
        uint32_t off = s.ovf_off[(base - t_begin) / TILE + (tid >> 7)] + wave_incl_scan(over) - over;
        if (wave & 1) {   // behind the entries of the tile's first 32 rows
          const uint4 p = s.rowmask[row - 32];
          const uint32_t tot = half ? 0u : __popc(p.x) + __popc(p.y) + __popc(p.z) + __popc(p.w);
          off += lane_bcast_u(wave_incl_scan(tot > ELL_K ? tot - ELL_K : 0u), 63);
        }
        uint32_t* pool = a.sv.sp_pool + (size_t)slab * a.sv.pool_cap;
        uint32_t* slots = reinterpret_cast<uint32_t*>(&s.slots[row]);
        uint32_t s_i = pre;
        uint64_t mm = half ? ((uint64_t)m.w << 32 | m.z) : ((uint64_t)m.y << 32 | m.x);
        while (mm != 0ull) {
          const int c = 64 * half + __ffsll((long long)mm) - 1;
          mm &= mm - 1ull;
          const uint32_t v = tile16[row * D + c];
          tile16[row * D + c] = 0;
          if (s_i < ELL_K) slots[s_i] = (uint32_t)c | ELL_VALID | (v << 16);
          else {
            if (off < a.sv.pool_cap) pool[off] = (uint32_t)((row & (TILE - 1)) * D + c) | (v << 16);
            ++off;
          }
          ++s_i;
        }
        block_lds_sync();
        if (tid < QT && base + tid < n)
          *reinterpret_cast<uint4*>(a.sv.ell + ((size_t)slab * a.sv.n_cap + base + tid) * ELL_K) = s.slots[tid];
      }
    } else {
      // A channel of a 64-token tile: the first ELL_V in token order take its fixed slots, the rest go to the tile's
      // overflow list, ordered (c, t).  The rows' bits are first sorted by channel.
      if (filt) {
        static_assert(ELL_V == 2, "the channel's slots are stored as one 8-byte word");
        {
          const int row = tid >> 1, half = tid & 1;
          const uint2 m = reinterpret_cast<const uint2*>(&s.rowmask[row])[half];
          uint64_t mm = (uint64_t)m.y << 32 | m.x;
          while (mm != 0ull) {
            const int c = 64 * half + __ffsll((long long)mm) - 1;
            mm &= mm - 1ull;
            atomicOr(&reinterpret_cast<uint32_t*>(&s.colmask[c])[row >> 5], 1u << (row & 31));
          }
        }
        block_lds_sync();
        const int c = tid & (D - 1), th = tid >> 7;
        const uint2 m = reinterpret_cast<const uint2*>(&s.colmask[c])[th];
        const uint2 mo = reinterpret_cast<const uint2*>(&s.colmask[c ^ 64])[th];   // what the other wave of the tile sees
        const uint32_t cnt = __popc(m.x) + __popc(m.y), cnto = __popc(mo.x) + __popc(mo.y);
        const uint32_t over = cnt > ELL_V ? cnt - ELL_V : 0u, overo = cnto > ELL_V ? cnto - ELL_V : 0u;
        const uint32_t inc = wave_incl_scan(over);
        const uint32_t other = lane_bcast_u(wave_incl_scan(overo), 63), tot = lane_bcast_u(inc, 63) + other;
        const int tl = base / TILE + th;
        if ((tid & (D - 1)) == 0) {
          // a list that fits takes the tile's reserved region; a longer one is allocated behind the regions
          const uint32_t off = tot <= VPOOL_FIXED ? (uint32_t)(h * a.sv.ntile_cap + tl) * VPOOL_FIXED
                                                  : (uint32_t)(a.dm.H * a.sv.ntile_cap) * VPOOL_FIXED + atomicAdd(&a.pool_ctr[b], tot);
          if (TILE * tl < n) a.sv.sp_table[(size_t)slab * a.sv.ntile_cap + tl] = make_uint2(off, tot);
          s.list_off[th] = off;
        }
        block_lds_sync();
        uint32_t off = s.list_off[th] + ((wave & 1) ? other : 0u) + inc - over;
        uint32_t* pool = a.sv.sp_pool + (size_t)b * a.sv.pool_cap;
        uint2 slot = make_uint2(0, 0);   // empty slots
        uint32_t s_i = 0;
        uint64_t mm = (uint64_t)m.y << 32 | m.x;
        while (mm != 0ull) {
          const int t = __ffsll((long long)mm) - 1;
          mm &= mm - 1ull;
          const int at = (TILE * th + t) * D + c;
          const uint32_t v = tile16[at];
          tile16[at] = 0;
          const uint32_t en = (uint32_t)t | ELL_VALID | (v << 16);
          if (s_i == 0u) slot.x = en;
          else if (s_i == 1u) slot.y = en;
          else {
            if (off < a.sv.pool_cap) pool[off] = (uint32_t)(t * D + c) | (v << 16);
            ++off;
          }
          ++s_i;
        }
        if (TILE * tl < n) *reinterpret_cast<uint2*>(a.sv.ell + (((size_t)slab * a.sv.ntile_cap + tl) * D + c) * ELL_V) = slot;
      }
      block_lds_sync();
    }
    if (filt) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const uint4 v = s.tile[8 * r0 + k][oc];
        x[k][0] = v.x; x[k][1] = v.y; x[k][2] = v.z; x[k][3] = v.w;
      }
    }
    if (a.Yout) {
      const GEAR_BUF_T yb = GEAR_BUF_MAKE(a.Yout + (size_t)slab * n * D, (uint32_t)n * (D * 2));
#pragma unroll
      for (int k = 0; k < 8; ++k)
        GEAR_BUF_STORE16_NT(yb, (base + 8 * r0 + k) * (D * 2) + oc * 16, make_uint4(x[k][0], x[k][1], x[k][2], x[k][3]));
    }

    // ---- min / max of the groups, (scale, zero)
    if constexpr (IS_K) {
      if constexpr (LG != KLG_VEC) {
        uint32_t mn[4], mx[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          mn[w] = mx[w] = x[0][w];
#pragma unroll
          for (int k = 1; k < 8; ++k) {
            mn[w] = pk_min_f16(mn[w], x[k][w]);
            mx[w] = pk_max_f16(mx[w], x[k][w]);
          }
        }
        if (ragged) {   // rows past the end take no part
          const int live = n - (base + 8 * r0);
          if (live < 8) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
              mn[w] = 0x7C007C00u;
              mx[w] = 0xFC00FC00u;
#pragma unroll
              for (int k = 0; k < 8; ++k) {
                mn[w] = pk_min_f16(mn[w], k < live ? x[k][w] : 0x7C007C00u);
                mx[w] = pk_max_f16(mx[w], k < live ? x[k][w] : 0xFC00FC00u);
              }
            }
          }
        }
        // over the wave's four rows of 16 lanes; row r of lanes ends up with word pi(r) = {0, 2, 1, 3}[r]
        GEAR_LANE_SWAP32(mn[0], mn[1]);
        GEAR_LANE_SWAP32(mn[2], mn[3]);
        GEAR_LANE_SWAP32(mx[0], mx[1]);
        GEAR_LANE_SWAP32(mx[2], mx[3]);
        uint32_t n01 = pk_min_f16(mn[0], mn[1]), n23 = pk_min_f16(mn[2], mn[3]);
        uint32_t x01 = pk_max_f16(mx[0], mx[1]), x23 = pk_max_f16(mx[2], mx[3]);
        GEAR_LANE_SWAP16(n01, n23);
        GEAR_LANE_SWAP16(x01, x23);
        const int w = ((lane >> 4) & 1) * 2 + (lane >> 5);
        s.red_mn[wave][oc * 4 + w] = pk_min_f16(n01, n23);
        s.red_mx[wave][oc * 4 + w] = pk_max_f16(x01, x23);
        block_lds_sync();
        constexpr int WPG = (1 << LG) / 32;   // waves per group
#pragma unroll
        for (int i0 = 0; i0 < NG * D; i0 += 256) {
          const int i = i0 + tid, gi = i >> 7, c = i & (D - 1);
          if (i < NG * D) {
            float fmn = INFINITY, fmx = -INFINITY;
#pragma unroll
            for (int wv = 0; wv < WPG; ++wv) {
              fmn = fminf(fmn, h2f(reinterpret_cast<const uint16_t*>(s.red_mn[gi * WPG + wv])[c]));
              fmx = fmaxf(fmx, h2f(reinterpret_cast<const uint16_t*>(s.red_mx[gi * WPG + wv])[c]));
            }
            const bool valid = base + (gi << LG) < n;
            const GroupQ q = make_group_b<BITS>(valid ? fmn : 0.0f, valid ? fmx : 0.0f);
            const uint32_t bits = group_bits(q);
            s.par[gi][c] = make_uint2(bits, __float_as_uint(q.inv));
            if (valid) a.sv.sz[((size_t)slab * a.sv.ng_cap + (base >> LG) + gi) * D + c] = bits;
          }
        }
        block_lds_sync();
      }
    } else {
      // word k: (min, -max) of the thread's piece of row k
      uint32_t u[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const uint32_t lo = pk_min_f16(pk_min_f16(x[k][0], x[k][1]), pk_min_f16(x[k][2], x[k][3]));
        const uint32_t hi = pk_max_f16(pk_max_f16(x[k][0], x[k][1]), pk_max_f16(x[k][2], x[k][3])) ^ 0x80008000u;
        u[k] = pk_min_f16(GEAR_BYTE_PERM(hi, lo, 0x05040100u), GEAR_BYTE_PERM(hi, lo, 0x07060302u));
      }
      // over the lanes of a group; every exchange halves the rows a lane carries
      constexpr int RPL = LG == 5 ? 2 : 1;   // rows a lane ends up with
      int j0;                                // the first of them
      const bool b0 = (lane & 1) != 0, b1 = (lane & 2) != 0, b2 = (lane & 4) != 0;
      uint32_t fin[RPL];
      if constexpr (LG == 5) {   // 4 lanes
        uint32_t p[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) p[k] = pk_min_f16(b1 ? u[k + 4] : u[k], dpp_u<DPP_XOR2>(b1 ? u[k] : u[k + 4]));
#pragma unroll
        for (int k = 0; k < 2; ++k) fin[k] = pk_min_f16(b0 ? p[k + 2] : p[k], dpp_u<DPP_XOR1>(b0 ? p[k] : p[k + 2]));
        j0 = (b1 ? 4 : 0) + (b0 ? 2 : 0);
      } else {                   // 8 or 16 lanes: lane i with lane 7 - i, then inside the quad
        uint32_t p[4], q[2];
#pragma unroll
        for (int k = 0; k < 4; ++k) p[k] = pk_min_f16(b2 ? u[k + 4] : u[k], dpp_u<DPP_HALF_MIRROR>(b2 ? u[k] : u[k + 4]));
#pragma unroll
        for (int k = 0; k < 2; ++k) q[k] = pk_min_f16(b1 ? p[k + 2] : p[k], dpp_u<DPP_XOR2>(b1 ? p[k] : p[k + 2]));
        fin[0] = pk_min_f16(b0 ? q[1] : q[0], dpp_u<DPP_XOR1>(b0 ? q[0] : q[1]));
        if constexpr (LG == 7) fin[0] = pk_min_f16(fin[0], dpp_u<DPP_ROR8>(fin[0]));
        j0 = lane & 7;
      }
      const int G = (oc * 8) >> LG;
#pragma unroll
      for (int i = 0; i < RPL; ++i) {
        const int row = 8 * r0 + j0 + i, t = base + row;
        const float lo = h2f(fin[i] & 0xFFFFu), hi = -h2f(fin[i] >> 16);
        GroupQ q;
        if (a.dm.kcvt) q = load_group(t < n ? a.vsz[(size_t)b * n + t] : 0u);
        else q = make_group_b<BITS>(lo, hi);
        if (LG != 7 || (lane & 8) == 0) {
          s.par[row][G] = make_uint2(group_bits(q), __float_as_uint(q.inv));
          if (t < n) a.sv.sz[((size_t)slab * a.sv.n_cap + t) * NG + G] = group_bits(q);
        }
      }
      wave_lds_sync();   // (a wave makes the parameters of its own 32 rows)
    }

    // ---- codes, and the residuals as fp16 operands: leading part, and what it leaves
    uint32_t oph[GRAM ? 8 : 1][4], opl[GRAM ? 8 : 1][4];
    {
#pragma clang fp contract(off)
      const int gi = IS_K ? (LG >= 7 ? 0 : (8 * r0) >> (LG < 7 ? LG : 7)) : 0;
      constexpr int CPS = 16 / BITS;     // codes per 16 bits
      float cw[8];                       // Keys: 16 bits of codes of my row pieces
      const GEAR_BUF_T cbuf = GEAR_BUF_MAKE(a.sv.codes + (size_t)slab * a.sv.n_cap * (4 * BITS), IS_K ? (uint32_t)n * (16 * BITS) : 0u);
#pragma unroll
      for (int w = 0; w < 4; ++w) {      // channels 2 w, 2 w + 1
        uint2 kp[2];                     // Keys: their parameters
        if constexpr (IS_K) {
          const uint4 p = *reinterpret_cast<const uint4*>(&s.par[gi][oc * 8 + 2 * w]);
          kp[0] = make_uint2(p.x, p.y);
          kp[1] = make_uint2(p.z, p.w);
        }
        float cv[2][2];                  // Values: the codes of the two channels in my eight tokens, 16 bits each
#pragma unroll
        for (int j = 0; j < 4; ++j) {    // rows 2 j, 2 j + 1
          uint2 vp[2];                   // Values: parameters of the two rows' channel group
          if constexpr (!IS_K) {
            vp[0] = s.par[8 * r0 + 2 * j][(oc * 8) >> LG];
            vp[1] = s.par[8 * r0 + 2 * j + 1][(oc * 8) >> LG];
          }
#pragma unroll
          for (int e2 = 0; e2 < 2; ++e2) {
            const int e = 2 * w + e2;
            float res[2];
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
              const int k = 2 * j + kk;
              const uint2 par = IS_K ? kp[e2] : vp[kk];
              const float mn = h2f(par.x >> 16), inv = __uint_as_float(par.y), dl = h2f(par.x & 0xFFFFu);
              // y - zero, 1/scale times it, nearest code: the quantizer's own sequence (y >= zero, so only the upper
              // end needs a clamp)
              const float ym = __builtin_fmaf(h2f(e2 ? x[k][w] >> 16 : x[k][w] & 0xFFFFu), one, -mn);
              const float c = fminf(rintf(__fmul_rn(ym, inv)), QMAX);
              res[kk] = __builtin_fmaf(-c, dl, ym);
              const int i = (IS_K ? e : k) % CPS;   // place of the code in its 16 bits
              float& acc16 = IS_K ? cw[k] : cv[e2][k / CPS];
              acc16 = i == 0 ? c : __builtin_fmaf(c, (float)(1u << (BITS * i)), acc16);
              if (IS_K && i == CPS - 1)   // (rows past the end fall outside the view)
                GEAR_BUF_STORE2(cbuf, (uint32_t)(base + 8 * r0 + k) * (16 * BITS) + oc * BITS + 2 * (e / CPS), (uint32_t)acc16);
            }
            if constexpr (GRAM) {
              const uint32_t hi = pack_h2(res[0], res[1]);
              oph[e][j] = hi;
              opl[e][j] = pack_h2(__builtin_fmaf(h2f(hi & 0xFFFFu), -one, res[0]), __builtin_fmaf(h2f(hi >> 16), -one, res[1]));
            }
          }
          if (GRAM && (IS_K || (j & 1))) GEAR_SCHED_FENCE();   // interleaved, the temporaries would not fit next to the accumulators
        }
        if constexpr (!IS_K) {
#pragma unroll
          for (int e2 = 0; e2 < 2; ++e2) {
            // word (kg*16 + c%16)*8 + c/16 of a block holds channel c = 8 oc + e for the 32/b tokens of lane group kg
            const int c16 = 8 * (oc & 1) + 2 * w + e2;
            if (BITS == 2) {
              const int word = (((r0 >> 1) & 3) * 16 + c16) * 8 + (oc >> 1);
              reinterpret_cast<uint16_t*>(s.codes)[((r0 >> 3) * 512 + word) * 2 + (r0 & 1)] = (uint16_t)(uint32_t)cv[e2][0];
            } else {
              const int word = ((r0 & 3) * 16 + c16) * 8 + (oc >> 1);
              reinterpret_cast<uint32_t*>(s.codes)[(r0 >> 2) * 512 + word] = (uint32_t)cv[e2][0] | ((uint32_t)cv[e2][1] << 16);
            }
          }
        }
      }
    }

    // ---- the 36 tiles of G: r r' = hi hi' + hi lo' + lo hi'; the next tile's rows are requested as registers fall free
    if constexpr (GRAM) {
      const int t0 = base + 8 * r0;
      if (ragged || base < a.t_lr) {   // block-uniform: rows past the end, rows that take no part in the low-rank term
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool live0 = t0 + 2 * j < n && t0 + 2 * j >= a.t_lr, live1 = t0 + 2 * j + 1 < n && t0 + 2 * j + 1 >= a.t_lr;
          const uint32_t keep = (live0 ? 0xFFFFu : 0u) | (live1 ? 0xFFFF0000u : 0u);
#pragma unroll
          for (int e = 0; e < 8; ++e) { oph[e][j] &= keep; opl[e][j] &= keep; }
        }
      }
      const bool more = base + QT < t_end;   // block-uniform
      GEAR_SCHED_FENCE();
      int ti = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const quant_h8 ah = __builtin_bit_cast(quant_h8, make_uint4(oph[e][0], oph[e][1], oph[e][2], oph[e][3]));
        const quant_h8 al = __builtin_bit_cast(quant_h8, make_uint4(opl[e][0], opl[e][1], opl[e][2], opl[e][3]));
#pragma unroll
        for (int f = e; f < 8; ++f) {
          const quant_h8 bh = __builtin_bit_cast(quant_h8, make_uint4(oph[f][0], oph[f][1], oph[f][2], oph[f][3]));
          const quant_h8 bl = __builtin_bit_cast(quant_h8, make_uint4(opl[f][0], opl[f][1], opl[f][2], opl[f][3]));
          acc[ti] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, bh, acc[ti], 0, 0, 0);
          acc[ti] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, bl, acc[ti], 0, 0, 0);
          acc[ti] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, bh, acc[ti], 0, 0, 0);
          ++ti;
        }
        GEAR_SCHED_FENCE();
        if (more && e >= 4) {   // two, one, one and four rows after e = 4 .. 7 (the operands of e and below are dead by then)
          const int first = e == 4 ? 0 : e - 3, last = e == 7 ? 8 : e - 2;
#pragma unroll
          for (int k = 0; k < 8; ++k)
            if (k >= first && k < last) load_row(base + QT, k);
        }
      }
      if (more) load_mask(base + QT);
    }
  }
  if constexpr (!IS_K) {
    block_lds_sync();
    copy_codes(((t_end - 1 - t_begin) & ~(QT - 1)) + t_begin);
  }

  // ---- the four waves' tiles, added in wave order (a fixed order: results do not vary from run to run); a few tiles
  // at a time, so that the LDS reads in flight stay few
  if constexpr (GRAM) {
    float* red = sm.red;
    float* out = a.gram + ((size_t)slab * gridDim.x + blockIdx.x) * GRAM_FLOATS;
    block_lds_sync();
    if (wave == 0) {
#pragma unroll
      for (int ti = 0; ti < GRAM_TILES; ++ti)
#pragma unroll
        for (int i = 0; i < 4; ++i) red[ti * 256 + i * 64 + lane] = acc[ti][i];
    }
    block_lds_sync();
#pragma unroll 1
    for (int w = 1; w < 3; ++w) {
      if (wave == w) {
#pragma unroll
        for (int ti = 0; ti < GRAM_TILES; ++ti) {
          float v[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = red[ti * 256 + i * 64 + lane];
#pragma unroll
          for (int i = 0; i < 4; ++i) red[ti * 256 + i * 64 + lane] = v[i] + acc[ti][i];
          GEAR_PIN_VGPR(v[0]);   // keeps the tiles' reads from being hoisted above each other's writes en bloc
        }
      }
      block_lds_sync();
    }
    if (wave == 3) {
#pragma unroll
      for (int ti = 0; ti < GRAM_TILES; ++ti) {
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = red[ti * 256 + i * 64 + lane];
#pragma unroll
        for (int i = 0; i < 4; ++i) out[ti * 256 + i * 64 + lane] = v[i] + acc[ti][i];
        GEAR_PIN_VGPR(v[0]);
      }
    }
  }
}

// One tensor, with Y for the solvers that go one tensor at a time.  grid (ceil(n / 128), B*H), block 256.
template <bool IS_K, int BITS, int LG>
__global__ __launch_bounds__(256, 3) void quant_kernel(QuantArgs a) {
  __shared__ QuantLds<IS_K, BITS, LG, false> sm;
  quant_body<IS_K, BITS, LG, false>(sm, a);
}

// Keys and Values of a call whose low-rank terms are solved together: the blocks of z = 0 take the Keys, those of z = 1 the
// Values.  A short prompt or a flushed buffer has fewer blocks than the chip has slots, and a block's time is the latency of
// its chain, so the second tensor rides along: 512 tokens of 32 heads took 15 + 15 us one after the other (a whole request of
// 24 steps 398 us, now 374 with the last round's projection taken together too; 7 x 40 heads x 1777 tokens compressed and read back
// 565 -> 520).  With the chip full it makes no difference (64 x 8 heads x 8192 tokens: 2640 and 2635 us).  grid (ceil(n / strip), B*H, 2), block 256.
template <int BITS, int KLG, int VLG, bool GRAM>
__global__ __launch_bounds__(256, (GRAM ? 2 : 3)) void quant_pair_kernel(QuantArgs k, QuantArgs v) {
  __shared__ union {
    QuantLds<true, BITS, KLG, GRAM> k;
    QuantLds<false, BITS, VLG, GRAM> v;
  } sm;
  if (blockIdx.z == 0) quant_body<true, BITS, KLG, GRAM>(sm.k, k);
  else quant_body<false, BITS, VLG, GRAM>(sm.v, v);
}

template <bool IS_K, int BITS, int LG>
static hipError_t launch_quant_t(const QuantArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((quant_kernel<IS_K, BITS, LG>), dim3((a.n + a.strip - 1) / a.strip, a.dm.B * a.dm.H), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace gear
