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
// What bounds it: vector issue (0.48 of the time under the profiler; 13 to 14 instructions per entry) next to the matrix cores (0.20), with two waves per
// SIMD, which is what the accumulators leave room for; some 170 of 800 us (64 x 8 heads x 8192 tokens, 2 % outliers) go to the loops over
// the outliers' bits.  So little may wait: a wave's 32 rows are copied straight into LDS while it works on the tile before (a copy
// needs no registers, of which there are none left), and nearly all of a tile's work is a wave's own: the four waves meet once per Key
// tile (the extremes of groups of 64 and 128 tokens) and twice per Value tile (the bits by channel, the list).  With the rows in
// registers and four or five barriers per tile 872 -> 800 us, 16 x 32 heads x 4096 tokens 449 -> 408, 7 x 40 x 1777 at 4 bits 160 -> 138.
// (Slower: two outliers of a lane per step instead of one, 806 with a loop per lane, 835 with one for the wave: more branches.)
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
  static constexpr int WPG = LG >= 7 ? 4 : LG == 6 ? 2 : 1;   // waves (of 32 rows) that share a group
  uint4 slots[QT];
  // a wave's (min, max) of its 32 rows, two channels per word; of this tile, of the last.  (None with one group per vector: four blocks fit a
  // CU without them.  1024 slabs x 20 tokens at 40 % outliers, 15.6 us with three blocks and 11.5 with four.)
  uint2 red[LG == KLG_VEC ? 1 : 2 * 4 * D / 2];
  __attribute__((aligned(16))) uint2 par[4][D];       // per wave: (scale, zero) as fp16, 1/scale
  uint32_t ovf_cnt[64], ovf_off[64];                  // overflow entries of the strip's stretches of 32 rows
};
static_assert(4 * (QT * D * 2 + sizeof(QuantSmem<true, 2, KLG_VEC>)) <= 160 * 1024, "four blocks per CU");
template <int BITS, int LG>
struct QuantSmem<false, BITS, LG> {
  static constexpr int NG = D >> LG;                  // groups per row
  uint2 rowmask[2 * QT];                              // the Filter per head
  uint32_t colmask[4][D];                             // per wave: bit t of channel c's word = its row t
  __attribute__((aligned(16))) uint2 par[NG * QT];    // [group][row]: (scale, zero) as fp16, 1/scale
  uint4 codes[4][QT * D * BITS / 512];                // per wave: code words in operand order
  uint32_t list_off[2];
};

// One block's strip of slab blockIdx.y, 256 threads.  tile: LDS of its own (not part of s), which the next tile is copied into
// while this one is worked on: with the two in one variable the compiler would wait for the copy at every access to s.
template <bool IS_K, int BITS, int LG, bool GRAM>
__device__ __forceinline__ void quant_body(uint4 (&tile)[QT][D / 8], QuantSmem<IS_K, BITS, LG>& s, const QuantArgs& a) {
  constexpr float QMAX = (float)((1 << BITS) - 1);
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
  uint16_t* tile16 = reinterpret_cast<uint16_t*>(&tile[0][0]);
  float one = 1.0f;
  GEAR_PIN_SGPR(one);   // fma(fp16 value, one, float) is one mixed-precision instruction: conversion and addition together

  // A wave fetches its own 32 rows, straight into LDS, and each thread the bits of half a row (row tid / 2); no other wave touches
  // them.  (Rows past the end: the last row once more, or nothing where a wave has no others; they are zeroed when they are read.)
  uint2 mk;
  auto fetch = [&](int base) {
    mk = GEAR_BUF_LOAD8(mb, base * 16 + tid * 8);
    if (!GRAM && base + 32 * wave >= n) return;   // wave-uniform (1536 slabs x 64 tokens without outliers or a low-rank term 19.1 -> 17.9 us)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int t = base + 32 * wave + 4 * i + (lane >> 4);
      GEAR_DMA16(xb, (uint32_t)(t < n ? t : n - 1) * (D * 2) + oc * 16, &tile[32 * wave + 4 * i][0]);
    }
  };
  fetch(t_begin);

  if constexpr (IS_K) {
    if (filt) {
      // where the overflow entries of the strip's stretches of 32 rows go: one allocation per strip, a list per 64 rows
      const int ntile = (t_end - t_begin + TILE - 1) / TILE;
      for (int i = wave; i < ntile; i += 4) {
        const uint4 m = GEAR_BUF_LOAD16(mb, (t_begin + TILE * i + lane) * 16);
        const uint32_t tot = __popc(m.x) + __popc(m.y) + __popc(m.z) + __popc(m.w);
        const uint32_t inc = wave_incl_scan(tot > ELL_K ? tot - ELL_K : 0u);
        const uint32_t first = lane_bcast_u(inc, 31), both = lane_bcast_u(inc, 63);
        if (lane < 2) s.ovf_cnt[2 * i + lane] = lane == 0 ? first : both - first;
      }
      block_lds_sync();
      if (wave == 0) {
        const uint32_t v = lane < 2 * ntile ? s.ovf_cnt[lane] : 0u;
        const uint32_t inc = wave_incl_scan(v), pair = v + dpp_u<DPP_XOR1>(v);
        uint32_t off = 0;
        if (lane == 63) off = atomicAdd(&a.pool_ctr[slab], inc);
        off = lane_bcast_u(off, 63) + inc - v;
        if (lane < 2 * ntile) {
          s.ovf_off[lane] = off;
          if ((lane & 1) == 0) a.sv.sp_table[(size_t)slab * a.sv.ntile_cap + t_begin / TILE + (lane >> 1)] = make_uint2(off, pair);
        }
      }
      block_lds_sync();
    }
    if (LG == KLG_VEC) {   // per-vector grouping: the channel's one pair of this segment was found with its thresholds
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const GroupQ q = load_group(a.sv.sz[(size_t)slab * a.sv.ng_cap * D + lane + 64 * i]);
        s.par[wave][lane + 64 * i] = make_uint2(group_bits(q), __float_as_uint(q.inv));
      }
    }
  }

  floatx4 acc[GRAM ? GRAM_TILES : 1];
#pragma unroll
  for (int i = 0; i < (GRAM ? GRAM_TILES : 1); ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};

#pragma unroll 1
  for (int base = t_begin; base < t_end; base += QT) {
    const bool ragged = base + QT > n;   // block-uniform: only such a tile has rows past the end
    // (the addresses below are made anew in every tile: kept over the loop they would not fit next to the accumulators)
    GEAR_PIN_VGPR(tid);
    lane = tid & 63;
    r0 = tid >> 4;
    oc = tid & 15;
    GEAR_DMA_WAIT();

    // ---- the tile's outliers: into slots and lists, and out of the tile
    if constexpr (IS_K) {
      // A token row: the first ELL_K in channel order take the row's fixed slots, the rest go to the 64-token tile's
      // overflow list, ordered (t, c).  Two threads per row, 64 channels each.
      if (filt) {
        static_assert(ELL_K == 4, "the row's slots are stored as one 16-byte word");
        const int row = tid >> 1, half = tid & 1;
        reinterpret_cast<uint2*>(s.slots)[tid] = make_uint2(0, 0);   // empty slots
        const uint32_t cnt = __popc(mk.x) + __popc(mk.y), other = dpp_u<DPP_XOR1>(cnt);
        const uint32_t pre = half ? other : 0u;
        const uint32_t over = (pre + cnt > ELL_K ? pre + cnt - ELL_K : 0u) - (pre > ELL_K ? pre - ELL_K : 0u);
        uint32_t off = s.ovf_off[(base - t_begin) / 32 + wave] + wave_incl_scan(over) - over;
        uint32_t* pool = a.sv.sp_pool + (size_t)slab * a.sv.pool_cap;
        uint32_t* slots = reinterpret_cast<uint32_t*>(&s.slots[row]);
        uint32_t s_i = pre;
        uint64_t mm = (uint64_t)mk.y << 32 | mk.x;
        wave_lds_sync();
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
        wave_lds_sync();
        const int t = 32 * wave + lane;
        if (lane < 32 && base + t < n) *reinterpret_cast<uint4*>(a.sv.ell + ((size_t)slab * a.sv.n_cap + base + t) * ELL_K) = s.slots[t];
      }
    } else {
      // A channel of a 64-token tile: the first ELL_V in token order take its fixed slots, the rest go to the tile's
      // overflow list, ordered (c, t).  Two waves share the tile; each sorts the bits of its 32 rows by channel, and takes the
      // entries of its rows.
      if (vhead && filt) {   // the Filter per head: the row's 16 lanes hold the whole vector
#pragma unroll 1
        for (int k = 0; k < 8; ++k) {
          const uint4 v = tile[8 * r0 + k][oc];
          const uint32_t kw[4] = {key16x2(v.x), key16x2(v.y), key16x2(v.z), key16x2(v.w)};
          const ThreshPair tp = row16_thresholds(kw, oc, a.k_top, a.k_bot);
          uint32_t f = 0;
#pragma unroll
          for (int e = 0; e < 8; ++e) f |= (outlier(slot_key(kw, e), (uint32_t)(8 * oc + e), tp) ? 1u : 0u) << e;
          const int t = base + 8 * r0 + k;
          if (t >= n) f = 0u;
          else reinterpret_cast<uint8_t*>(a.mask + (size_t)slab * n + t)[oc] = (uint8_t)f;
          reinterpret_cast<uint8_t*>(&s.rowmask[2 * (8 * r0 + k)])[oc] = (uint8_t)f;
        }
        wave_lds_sync();
        mk = s.rowmask[tid];
      }
      if (filt) {
        static_assert(ELL_V == 2, "the channel's slots are one or the other of two words");
        s.colmask[wave][lane] = s.colmask[wave][lane + 64] = 0u;
        wave_lds_sync();
        {
          uint64_t mm = (uint64_t)mk.y << 32 | mk.x;
          while (mm != 0ull) {
            const int c = 64 * (lane & 1) + __ffsll((long long)mm) - 1;
            mm &= mm - 1ull;
            atomicOr(&s.colmask[wave][c], 1u << (lane >> 1));
          }
        }
        GEAR_DMA_BARRIER();
        const int th = wave >> 1, odd = wave & 1;
        const uint32_t lo0 = s.colmask[2 * th][lane], hi0 = s.colmask[2 * th + 1][lane];             // channel lane
        const uint32_t lo1 = s.colmask[2 * th][lane + 64], hi1 = s.colmask[2 * th + 1][lane + 64];   // channel lane + 64
        const uint32_t cnt0 = __popc(lo0) + __popc(hi0), cnt1 = __popc(lo1) + __popc(hi1);
        const uint32_t over0 = cnt0 > ELL_V ? cnt0 - ELL_V : 0u, over1 = cnt1 > ELL_V ? cnt1 - ELL_V : 0u;
        const uint32_t inc0 = wave_incl_scan(over0), inc1 = lane_bcast_u(inc0, 63) + wave_incl_scan(over1);
        const int tl = base / TILE + th;
        if (odd == 0 && lane == 63) {
          const uint32_t tot = inc1;
          // a list that fits takes the tile's reserved region; a longer one is allocated behind the regions
          const uint32_t off = tot <= VPOOL_FIXED ? (uint32_t)(h * a.sv.ntile_cap + tl) * VPOOL_FIXED
                                                  : (uint32_t)(a.dm.H * a.sv.ntile_cap) * VPOOL_FIXED + atomicAdd(&a.pool_ctr[b], tot);
          if (TILE * tl < n) a.sv.sp_table[(size_t)slab * a.sv.ntile_cap + tl] = make_uint2(off, tot);
          s.list_off[th] = off;
        }
        // my rows' entries of the two channels, in their order; s_i, off: the next one's place among the channel's, in the list
        // by_channel: only these two waves have rows (a flushed buffer of up to 64 tokens): they take a lane's first and second channel with
        // all of its rows.  By rows, the second wave has little to do (4 x 32 heads x 33 tokens at 40 %, rank 2, 42.7 -> 39.9 us).
        const bool by_channel = !GRAM && n - base <= TILE;   // block-uniform
        const uint32_t before0 = odd && !by_channel ? __popc(lo0) : 0u, before1 = odd && !by_channel ? __popc(lo1) : 0u;
        uint64_t mm = odd ? ((uint64_t)hi1 << 32 | hi0) : ((uint64_t)lo1 << 32 | lo0);
        if (by_channel) mm = odd ? ((uint64_t)hi1 << 32 | lo1) : ((uint64_t)hi0 << 32 | lo0);
        GEAR_DMA_BARRIER();
        const uint32_t list = s.list_off[th];
        uint32_t off = list + inc0 - over0 + (before0 > ELL_V ? before0 - ELL_V : 0u), s_i = before0;
        const uint32_t off1 = list + inc1 - over1 + (before1 > ELL_V ? before1 - ELL_V : 0u);
        uint32_t* pool = a.sv.sp_pool + (size_t)b * a.sv.pool_cap;
        uint2 slot[2] = {make_uint2(0, 0), make_uint2(0, 0)};   // empty slots
        uint32_t second = 0;   // at channel lane + 64
        if (by_channel && odd) {
          second = 1u;
          off = off1;
        }
        while (mm != 0ull) {
          const uint32_t bit = (uint32_t)__ffsll((long long)mm) - 1u;
          mm &= mm - 1ull;
          if (!by_channel && bit >= 32u && second == 0u) {
            second = 1u;
            off = off1;
            s_i = before1;
          }
          const int t = by_channel ? (int)bit : 32 * odd + (int)(bit & 31u), c = lane + 64 * (int)second, at = (TILE * th + t) * D + c;
          const uint32_t v = tile16[at];
          tile16[at] = 0;
          const uint32_t en = (uint32_t)t | ELL_VALID | (v << 16);
          if (s_i >= ELL_V) {
            if (off < a.sv.pool_cap) pool[off] = (uint32_t)(t * D + c) | (v << 16);
            ++off;
          } else if (second == 0u) {
            if (s_i == 0u) slot[0].x = en;
            else slot[0].y = en;
          } else {
            if (s_i == 0u) slot[1].x = en;
            else slot[1].y = en;
          }
          ++s_i;
        }
        if (by_channel) GEAR_DMA_BARRIER();   // (a wave's entries are in the other's rows too)
        else wave_lds_sync();
        if (TILE * tl < n) {
          // of a channel's two slots the wave of the first rows stores those that its entries take, the other wave the rest
          uint2* ell = reinterpret_cast<uint2*>(a.sv.ell + (((size_t)slab * a.sv.ntile_cap + tl) * D + lane) * ELL_V);
          auto store = [&](uint2* p, uint32_t first, uint2 both) {   // first: entries of the first 32 rows
            if (first >= 2u) {
              if (!odd) *p = both;
            } else if (first == 1u) {
              reinterpret_cast<uint32_t*>(p)[odd] = odd ? both.y : both.x;
            } else if (odd) {
              *p = both;
            }
          };
          if (by_channel) ell[64 * odd] = odd ? slot[1] : slot[0];
          else {
            store(ell, __popc(lo0), slot[0]);
            store(ell + 64, __popc(lo1), slot[1]);
          }
        }
      }
    }
    uint32_t x[8][4];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint4 v = tile[8 * r0 + k][oc];
      x[k][0] = v.x; x[k][1] = v.y; x[k][2] = v.z; x[k][3] = v.w;
    }
    if constexpr (IS_K) {
      GEAR_LDS_DRAIN();
      if (base + QT < t_end) fetch(base + QT);   // block-uniform
    }
    if (ragged) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const uint32_t keep = (uint32_t)((base + 8 * r0 + k - n) >> 31);   // all ones: a row before the end
#pragma unroll
        for (int w = 0; w < 4; ++w) x[k][w] &= keep;
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
        const int w = ((lane >> 4) & 1) * 2 + (lane >> 5), wpg = QuantSmem<true, BITS, LG>::WPG;
        const int buf = (((base - t_begin) / QT) & 1) * (2 * D);
        int at = buf + wave * (D / 2) + oc * 4 + w;
        GEAR_PIN_VGPR(at);   // (one step from the array to the element, see quant_body's head)
        s.red[at] = make_uint2(pk_min_f16(n01, n23), pk_max_f16(x01, x23));
        // each wave makes the parameters of its own group, two channels per lane: what the next barrier would cost is more than
        // that they are made by all waves of the group
        if constexpr (wpg > 1) GEAR_DMA_BARRIER();
        else wave_lds_sync();
        const int first = wave & ~(wpg - 1), grp = (base + 32 * first) >> LG;
        at = buf + first * (D / 2) + lane;
        GEAR_PIN_VGPR(at);
        uint2 ext = s.red[at];
#pragma unroll
        for (int wv = 1; wv < wpg; ++wv) {
          const uint2 o = s.red[at + wv * (D / 2)];
          ext = make_uint2(pk_min_f16(ext.x, o.x), pk_max_f16(ext.y, o.y));
        }
        const bool valid = base + 32 * first < n;
        if (!valid) ext = make_uint2(0, 0);
        const GroupQ q0 = make_group_b<BITS>(h2f(ext.x & 0xFFFFu), h2f(ext.y & 0xFFFFu)), q1 = make_group_b<BITS>(h2f(ext.x >> 16), h2f(ext.y >> 16));
        const uint2 bits = make_uint2(group_bits(q0), group_bits(q1));
        *reinterpret_cast<uint4*>(&s.par[wave][2 * lane]) = make_uint4(bits.x, __float_as_uint(q0.inv), bits.y, __float_as_uint(q1.inv));
        if (valid && wave == first) *reinterpret_cast<uint2*>(a.sv.sz + ((size_t)slab * a.sv.ng_cap + grp) * D + 2 * lane) = bits;
        wave_lds_sync();
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
          s.par[G * QT + row] = make_uint2(group_bits(q), __float_as_uint(q.inv));
          if (t < n) a.sv.sz[((size_t)slab * a.sv.n_cap + t) * (D >> LG) + G] = group_bits(q);
        }
      }
      wave_lds_sync();   // (a wave makes the parameters of its own 32 rows)
    }

    // ---- codes, and the residuals as fp16 operands: leading part, and what it leaves
    uint32_t oph[GRAM ? 8 : 1][4], opl[GRAM ? 8 : 1][4];
    {
#pragma clang fp contract(off)
      constexpr int CPS = 16 / BITS;     // codes per 16 bits
      float cw[8];                       // Keys: 16 bits of codes of my row pieces
      // Values: where my code words begin (2 bits: half words)
      int code_at = BITS == 2 ? wave * 512 + ((((r0 >> 1) & 1) * 16 + 8 * (oc & 1)) * 8 + (oc >> 1)) * 2 + (r0 & 1)
                              : wave * 512 + ((r0 & 3) * 16 + 8 * (oc & 1)) * 8 + (oc >> 1);
      const int par_at = IS_K ? 0 : ((oc * 8) >> LG) * QT + 8 * r0;   // Values: my first row's parameters
      if (!IS_K) GEAR_PIN_VGPR(code_at);
      const GEAR_BUF_T cbuf = GEAR_BUF_MAKE(a.sv.codes + (size_t)slab * a.sv.n_cap * (4 * BITS), IS_K ? (uint32_t)n * (16 * BITS) : 0u);
#pragma unroll
      for (int w = 0; w < 4; ++w) {      // channels 2 w, 2 w + 1
        uint2 kp[2];                     // Keys: their parameters
        if constexpr (IS_K) {
          const uint4 p = *reinterpret_cast<const uint4*>(&s.par[wave][oc * 8 + 2 * w]);
          kp[0] = make_uint2(p.x, p.y);
          kp[1] = make_uint2(p.z, p.w);
        }
        float cv[2][2];                  // Values: the codes of the two channels in my eight tokens, 16 bits each
#pragma unroll
        for (int j = 0; j < 4; ++j) {    // rows 2 j, 2 j + 1
          uint2 vp[2];                   // Values: parameters of the two rows' channel group
          if constexpr (!IS_K) {
            const uint4 p = *reinterpret_cast<const uint4*>(s.par + par_at + 2 * j);
            vp[0] = make_uint2(p.x, p.y);
            vp[1] = make_uint2(p.z, p.w);
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
              if (!IS_K) GEAR_PIN_VGPR(opl[e][j]);   // (here, and not behind the code words: the residuals would have to be kept)
            }
          }
          if (GRAM && (IS_K || (j & 1))) GEAR_SCHED_FENCE();   // interleaved, the temporaries would not fit next to the accumulators
        }
        if constexpr (!IS_K) {
#pragma unroll
          for (int e2 = 0; e2 < 2; ++e2) {
            // word (kg*16 + c%16)*8 + c/16 of a block holds channel c = 8 oc + e for the 32/b tokens of lane group kg: the wave's
            // 32 rows are two lane groups of a block of 64 (2 bits), or a block (4 bits)
            if (BITS == 2) {
              const int word = (2 * w + e2) * 8;
              reinterpret_cast<uint16_t*>(s.codes)[code_at + word * 2] = (uint16_t)(uint32_t)cv[e2][0];
            } else {
              const int word = (2 * w + e2) * 8;
              reinterpret_cast<uint32_t*>(s.codes)[code_at + word] = (uint32_t)cv[e2][0] | ((uint32_t)cv[e2][1] << 16);
            }
          }
        }
      }
    }
    if constexpr (!IS_K) {
      // the wave's code words; every word of a block that holds at least one token is written (rows past n carry code 0)
      wave_lds_sync();
      constexpr int TB = 128 / BITS, WPB = TB / 32;   // tokens of a block: 64 (2 bits) or 32 (4 bits); waves that share it
      const int blk = base / TB + wave / WPB;
      uint4* dst = reinterpret_cast<uint4*>(a.sv.codes + ((size_t)slab * a.sv.nblk_cap + blk) * 512) + (wave % WPB) * (128 / WPB);
      if (blk * TB < n) {
#pragma unroll
        for (int i = 0; i < 2 / WPB; ++i) dst[lane + 64 * i] = s.codes[wave][lane + 64 * i];
      }
      // (from here on the tile's work touches no LDS: the compiler, which for the Values does not tell the copy from its reads of the
      // parameters, would wait for the copy there)
      GEAR_LDS_DRAIN();
      if (base + QT < t_end) fetch(base + QT);   // block-uniform
    }

    // ---- the 36 tiles of G: r r' = hi hi' + hi lo' + lo hi'
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
      GEAR_SCHED_FENCE();
      // (a tile's three terms are as far apart as the order allows: the next one on the same accumulators would wait for the last)
#pragma unroll
      for (int e0 = 0; e0 < 8; e0 += 4) {   // operands e0 .. e0 + 3 with all from them on: 26 and 10 tiles
#pragma unroll
        for (int term = 0; term < 3; ++term) {
#pragma unroll
          for (int e = e0; e < e0 + 4; ++e) {
            const auto& oa = term == 2 ? opl : oph;
            const quant_h8 va = __builtin_bit_cast(quant_h8, make_uint4(oa[e][0], oa[e][1], oa[e][2], oa[e][3]));
#pragma unroll
            for (int f = e; f < 8; ++f) {
              const auto& ob = term == 1 ? opl : oph;
              const quant_h8 vb = __builtin_bit_cast(quant_h8, make_uint4(ob[f][0], ob[f][1], ob[f][2], ob[f][3]));
              const int ti = e * 8 - e * (e - 1) / 2 + f - e;
              acc[ti] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va, vb, acc[ti], 0, 0, 0);
            }
          }
          GEAR_SCHED_FENCE();
        }
      }
    }
  }

  // ---- the four waves' tiles, added in wave order (a fixed order: results do not vary from run to run): four tiles at a time, those of
  // the next round into the other half of the LDS
  if constexpr (GRAM) {
    float* red = reinterpret_cast<float*>(&tile[0][0]);   // [2][4][1024]
    float* out = a.gram + ((size_t)slab * gridDim.x + blockIdx.x) * GRAM_FLOATS;
    static_assert(GRAM_TILES % 4 == 0 && sizeof(tile) == 2 * 4 * 1024 * sizeof(float), "two rounds of four tiles of four waves");
    GEAR_DMA_BARRIER();
#pragma unroll
    for (int r = 0; r < GRAM_TILES / 4; ++r) {
      float* part = red + (r & 1) * 4096;
#pragma unroll
      for (int ti = 0; ti < 4; ++ti)
#pragma unroll
        for (int i = 0; i < 4; ++i) part[wave * 1024 + ti * 256 + i * 64 + lane] = acc[4 * r + ti][i];
      GEAR_DMA_BARRIER();
      floatx4 sum = *reinterpret_cast<const floatx4*>(part + 4 * tid);
#pragma unroll
      for (int w = 1; w < 4; ++w) sum += *reinterpret_cast<const floatx4*>(part + w * 1024 + 4 * tid);
      *reinterpret_cast<floatx4*>(out + r * 1024 + 4 * tid) = sum;
    }
  }
}

// One tensor, with Y for the solvers that go one tensor at a time.  grid (ceil(n / 128), B*H), block 256.
template <bool IS_K, int BITS, int LG>
__global__ __launch_bounds__(256, 3) void quant_kernel(QuantArgs a) {
  __shared__ uint4 tile[QT][D / 8];
  __shared__ QuantSmem<IS_K, BITS, LG> s;
  quant_body<IS_K, BITS, LG, false>(tile, s, a);
}

// Keys and Values of a call whose low-rank terms are solved together: the blocks of z = 0 take the Keys, those of z = 1 the
// Values.  A short prompt or a flushed buffer has fewer blocks than the chip has slots, and a block's time is the latency of
// its chain, so the second tensor rides along: 512 tokens of 32 heads took 15 + 15 us one after the other (a whole request of
// 24 steps 398 us, now 374 with the last round's projection taken together too; 7 x 40 heads x 1777 tokens compressed and read back
// 565 -> 520).  With the chip full it makes no difference (64 x 8 heads x 8192 tokens: 2640 and 2635 us).  grid (ceil(n / strip), B*H, 2), block 256.
template <int BITS, int KLG, int VLG, bool GRAM>
__global__ __launch_bounds__(256, (GRAM ? 2 : 3)) void quant_pair_kernel(QuantArgs k, QuantArgs v) {
  __shared__ uint4 tile[QT][D / 8];
  __shared__ union {
    QuantSmem<true, BITS, KLG> k;
    QuantSmem<false, BITS, VLG> v;
  } s;
  if (blockIdx.z == 0) quant_body<true, BITS, KLG, GRAM>(tile, s.k, k);
  else quant_body<false, BITS, VLG, GRAM>(tile, s.v, v);
}

template <bool IS_K, int BITS, int LG>
static hipError_t launch_quant_t(const QuantArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((quant_kernel<IS_K, BITS, LG>), dim3((a.n + a.strip - 1) / a.strip, a.dm.B * a.dm.H), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace gear
