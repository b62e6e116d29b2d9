// Filter_s (Eq. 4) of vectors that lie in registers as raw fp16 values, by the extremes of groups of entries.
//
// S holds a few per cent of a vector, so most entries only have to be seen to lie well inside it.  The entries of a lane are
// taken in groups (8 to 20 of them); if k groups have a maximum of at least T, then at least k entries are >= T, so the k-th
// largest group maximum, rounded down, is a threshold that every one of the k largest entries passes and few others do: of
// 1024 entries in groups of 16, 11 of which are wanted, about 13 pass; of 4096, 41 of which are wanted, about 46.  The
// survivors of both ends are put on a list in LDS and ranked exactly there, index and all.  Per pair of entries that is two
// packed instructions for the extremes and five for the test, against a histogram add in LDS per entry and two scans of 256
// counters per end in the two-level radix selection (gear_select.h).  That stays as the way out for vectors whose candidates
// do not fit the list: many entries equal to a threshold, or a ratio close to one entry in two.  Value rows: 64 x 8192 tokens
// of 1024 entries 504 -> 240 us (vector issue 0.86), 16 x 4096 of 4096 entries 240 -> 130, 32768 of 4096 entries 134 -> 70 (3.9 to
// 4.5 TB/s; the floor is one read); a flushed buffer of 4 x 20 tokens 17 -> 7.
#pragma once
#include "gear_internal.h"
#include "gear_select.h"

namespace gear {

constexpr int EXT_LIST = 512;       // candidates per wave: the words of the histograms that the way out needs (SELECT_LDS_WORDS)
constexpr int EXT_ROW_LIST = 128;   // ... per row of 16 lanes, where a wave works on four vectors

// The fp16 values next to the two rough thresholds, on the inside, in both halves: an entry is a candidate iff the clamp to
// [lo, hi] changes it.  tt, tb: candidates are the keys >= tt and those with 0xFFFF - key >= tb; 0x10000: none on that side.
// (-0 counts as changed where lo is +0: candidates may be too many, never too few.)
struct RoughBounds {
  uint32_t lo, hi;
};
__device__ __forceinline__ RoughBounds rough_bounds(uint32_t tt, uint32_t tb) {
  const uint32_t khi = tt - 1u < 0xFC00u ? tt - 1u : 0xFC00u;             // (no finite value lies beyond the infinities)
  const uint32_t klo = tb < 0xFC00u ? 0x10000u - tb : 0x0400u;
  return RoughBounds{unkey16(klo) * 0x00010001u, unkey16(khi) * 0x00010001u};
}
// Whether two rough thresholds can be used: enough groups on both sides (lanes without entries count as infinities of the
// wrong sign, keys 0x0400 and 0xFC00), and at least one key between them.
__device__ __forceinline__ bool rough_usable(uint32_t tt, uint32_t tb) { return tt > 0x0400u && tb > 0x0400u && tt + tb > 0x10000u; }
// bit j and bit 16 + j of f: the halves of word j (0..15) of a run of words that the clamp changes
__device__ __forceinline__ uint32_t outside_bits(uint32_t x, const RoughBounds& b, int j) {
  return nonzero_u16x2(x ^ pk_max_f16(pk_min_f16(x, b.hi), b.lo)) << j;
}
// Largest / smallest of the row pieces `w`, added to a running pair (even and odd entries apart).
__device__ __forceinline__ void extend_extremes(const uint4& v, uint32_t& mx, uint32_t& mn) {
  mx = pk_max_f16(pk_max_f16(mx, v.x), pk_max_f16(pk_max_f16(v.y, v.z), v.w));
  mn = pk_min_f16(pk_min_f16(mn, v.x), pk_min_f16(pk_min_f16(v.y, v.z), v.w));
}

// ------------------------------------------------------------------ one vector per wave
// Largest X such that k of the wave's words are >= X (k >= 1; the words that are not 0 are distinct, and at least k of them
// are >= rough << 16).  Counts are ballots: the search is scalar code but for one compare per step and register.
template <int R>
__device__ __forceinline__ uint32_t wave_kth_largest(const uint32_t (&c)[R], uint32_t k, uint32_t rough) {
  auto count = [&](uint32_t x) {
    uint32_t n = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) n += (uint32_t)__popcll(__ballot(c[i] >= x));
    return n;
  };
  uint32_t key = rough;
  // (the rough threshold is rarely more than a few steps of its own grid below the exact one)
  int b = rough + 512u <= 0xFFFFu && count((rough + 512u) << 16) >= k ? 15 : 8;
#pragma unroll 1
  for (; b >= 0; --b) {
    const uint32_t t = key + (1u << b);
    if (t <= 0xFFFFu && count(t << 16) >= k) key = t;
  }
  uint32_t x = key << 16;
  if (count(x) != k) {   // several entries equal the threshold: the lower halves (complements of the indices) decide
#pragma unroll 1
    for (b = 15; b >= 0; --b)
      if (count(x + (1u << b)) >= k) x += 1u << b;
  }
  return x;
}
// The same through a histogram of the distances of the keys from the rough threshold (two keys per counter; hist: 256 words of LDS
// private to the wave): the counter at which k is reached holds one to three entries as a rule, and those too many are dropped
// one by one.  Where many entries share the threshold, a second histogram finds the index among them (the lower halves are complements of
// indices below `rows`).  A chain of some 700 cycles each, where the search above takes 10 to 26 dependent steps of 100 to 200: it is
// what is left for lists whose threshold lies further off.  key_only: the lower half of the result does not matter.
template <int R>
__device__ __forceinline__ uint32_t wave_kth_by_bins(const uint32_t (&c)[R], uint32_t k, uint32_t rough, uint32_t* hist, int rows,
                                                     bool key_only = false) {
  const int lane = lane_id();
  wave_lds_sync();
  *reinterpret_cast<uint4*>(hist + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
  wave_lds_sync();
  uint32_t bin[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    bin[i] = 0xFFFFu;   // below the rough threshold, or nothing there
    if (c[i] >= rough << 16) {
      bin[i] = min(((c[i] >> 16) - rough) >> 1, 255u);
      atomicAdd(&hist[bin[i]], 1u);
    }
  }
  wave_lds_sync();
  int at;
  uint32_t above;
  scan_from_top(hist, k, at, above);
  const uint32_t spare = (uint32_t)GEAR_WAVE_UNIFORM((int)hist[at]) - (k - above);   // entries of that counter that are too many
  if (__builtin_expect(at == 255, 0)) return wave_kth_largest<R>(c, k, rough);
  uint32_t x = 0u;
  if (__builtin_expect(spare <= 6u, 1)) {
#pragma unroll 1
    for (uint32_t i = 0; i <= spare; ++i) {   // the least of the counter's entries above the last one
      uint32_t m = 0xFFFFFFFFu;
#pragma unroll
      for (int r = 0; r < R; ++r) m = min(m, bin[r] == (uint32_t)at && c[r] > x ? c[r] : 0xFFFFFFFFu);
      m = row16_min_u(m);
      x = min(min(lane_bcast_u(m, 0), lane_bcast_u(m, 16)), min(lane_bcast_u(m, 32), lane_bcast_u(m, 48)));
    }
    return x;
  }
  auto count = [&](uint32_t y) {
    uint32_t n = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) n += (uint32_t)__popcll(__ballot(c[i] >= y));
    return n;
  };
  uint32_t key = rough + 2u * (uint32_t)at + 1u;   // which of the counter's two keys
  const uint32_t upper = count(key << 16);
  if (upper < k) --key;
  if (key_only) return key << 16;
  const uint32_t need = k - (upper < k ? upper : above);
  const int shift = rows > 256 ? 24 - __clz(rows - 1) : 0;   // 256 counters for the indices
  wave_lds_sync();
  *reinterpret_cast<uint4*>(hist + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
  wave_lds_sync();
  uint32_t low = (256u << shift) - 0x10000u, from = key << 16;   // (lower halves lie in the last 256 << shift of theirs)
  GEAR_PIN_VGPR(low);
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const uint32_t off = c[i] - from;
    if (off <= 0xFFFFu) atomicAdd(&hist[(off + low) >> shift], 1u);
    GEAR_SCHED_FENCE();
  }
  wave_lds_sync();
  scan_from_top(hist, need, at, above);
  x = key << 16 | (0xFFFFu - ((256u - (uint32_t)at) << shift) + 1u);   // the last index of the counter
#pragma unroll 1
  for (int b = shift - 1; b >= 0; --b)
    if (count(x + (1u << b)) >= k) x += 1u << b;
  return x;
}
// list: `total` words (index | fp16 value << 16).  Leaves the selected entries as bits of smask (which may overlap the list).
template <int R>
__device__ __forceinline__ void wave_rank_list(uint32_t* list, uint32_t total, int k_top, int k_bot, uint32_t tt, uint32_t tb,
                                               uint32_t* smask, int mask_words) {
  const int lane = lane_id();
  uint32_t ct[R], cb[R];   // composites that grow towards the top / the bottom, ties towards the lower index
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const uint32_t p = (uint32_t)(lane + 64 * i);
    ct[i] = cb[i] = 0u;
    if (p < total) {
      const uint32_t e = list[p], c = key16(e >> 16) << 16 | (e & 0xFFFFu);
      ct[i] = c ^ 0xFFFFu;
      cb[i] = ~c;
    }
  }
  const uint32_t xt = k_top > 0 ? wave_kth_by_bins<R>(ct, (uint32_t)k_top, tt, list, 32 * mask_words) : 0xFFFFFFFFu;
  const uint32_t xb = k_bot > 0 ? wave_kth_by_bins<R>(cb, (uint32_t)k_bot, tb, list, 32 * mask_words) : 0xFFFFFFFFu;
  wave_lds_sync();
  for (int i = lane; i < mask_words; i += 64) smask[i] = 0u;
  wave_lds_sync();
#pragma unroll
  for (int i = 0; i < R; ++i)
    if (ct[i] >= xt || cb[i] >= xb) {
      const uint32_t idx = 0xFFFFu - (ct[i] & 0xFFFFu);
      atomicOr(&smask[idx >> 5], 1u << (idx & 31u));
    }
  wave_lds_sync();
}

// The vector of a Value token: chunk ch, lane l, entry e <-> index ch * 512 + l * 8 + e, H heads of 128 entries (lanes past the
// last head hold zeros).  raw: NC * 64 pieces of LDS private to the wave; list: EXT_LIST words.  The set's bits are left in
// list[0 .. 4 H) (bit i of the vector: word i / 32), for all lanes to see.  Returns false, with nothing done, where the
// candidates do not fit (wave-uniform).
template <int NC>
__device__ __forceinline__ bool wave_ext_select(const uint4 (&x)[NC], int H, int k_top, int k_bot, uint4* raw, uint32_t* list) {
  constexpr int NS = NC <= 2 ? 1 : NC >= 16 ? 4 : 2, CS = NC / NS;   // sets of CS chunks, two groups (even, odd entries) each
  static_assert(NS * CS == NC, "whole sets");
  const int lane = lane_id(), hsub = lane >> 4;
#pragma unroll
  for (int ch = 0; ch < NC; ++ch) raw[ch * 64 + lane] = x[ch];
  uint32_t gx[2 * NS], gn[2 * NS];   // keys of the groups' maxima, complements of those of the minima
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    uint32_t mx = 0xFC00FC00u, mn = 0x7C007C00u;
#pragma unroll
    for (int i = 0; i < CS; ++i) {
      const int ch = s * CS + i;
      if (ch * 4 + 4 <= H) extend_extremes(x[ch], mx, mn);   // wave-uniform: a chunk of whole heads
      else if (ch * 4 + hsub < H) extend_extremes(x[ch], mx, mn);
    }
    const uint32_t kx = key16x2(mx), kn = ~key16x2(mn);
    gx[2 * s] = kx & 0xFFFFu;
    gx[2 * s + 1] = kx >> 16;
    gn[2 * s] = kn & 0xFFFFu;
    gn[2 * s + 1] = kn >> 16;
  }
  uint32_t tt = 0u, tb = 0u;
#pragma unroll 1
  for (int b = 15; b >= 6; --b) {   // ten bits: 1/16 of an octave
    uint32_t nt = 0, nb = 0;
    const uint32_t qt = tt | 1u << b, qb = tb | 1u << b;
#pragma unroll
    for (int i = 0; i < 2 * NS; ++i) {
      nt += (uint32_t)__popcll(__ballot(gx[i] >= qt));
      nb += (uint32_t)__popcll(__ballot(gn[i] >= qb));
    }
    if (nt >= (uint32_t)k_top) tt = qt;
    if (nb >= (uint32_t)k_bot) tb = qb;
  }
  if (k_top == 0) tt = 0x10000u;
  if (k_bot == 0) tb = 0x10000u;
  if (!rough_usable(tt, tb)) return false;
  const RoughBounds rb = rough_bounds(tt, tb);
  constexpr int NF = (NC * 4 + 15) / 16;
  uint32_t f[NF], cnt = 0;
#pragma unroll
  for (int q = 0; q < NF; ++q) f[q] = 0u;
#pragma unroll
  for (int ch = 0; ch < NC; ++ch) {
    const int q = ch / 4, j = (ch % 4) * 4;
    const uint32_t z = outside_bits(x[ch].x, rb, j) | outside_bits(x[ch].y, rb, j + 1) | outside_bits(x[ch].z, rb, j + 2) |
                       outside_bits(x[ch].w, rb, j + 3);
    if (ch * 4 + 4 <= H || ch * 4 + hsub < H) f[q] |= z;
  }
#pragma unroll
  for (int q = 0; q < NF; ++q) cnt += (uint32_t)__popc(f[q]);
  const uint32_t inc = wave_incl_scan(cnt), total = lane_bcast_u(inc, 63);
  if (total > EXT_LIST) return false;
  uint32_t pos = inc - cnt;
  wave_lds_sync();
#pragma unroll
  for (int q = 0; q < NF; ++q) {
    while (f[q] != 0u) {   // bit p: entry p / 16 of word p % 16 of the sixteen words of chunks 4 q ..
      const uint32_t p = (uint32_t)__ffs((int)f[q]) - 1u, w = p & 15u, half = p >> 4;
      f[q] &= f[q] - 1u;
      const uint32_t ch = 4u * q + (w >> 2), e = 2u * (w & 3u) + half;
      const uint32_t v = reinterpret_cast<const uint16_t*>(raw + ch * 64u + lane)[e];
      list[pos++] = (ch * 512u + lane * 8u + e) | v << 16;
    }
  }
  wave_lds_sync();
  if (total <= 128u) wave_rank_list<2>(list, total, k_top, k_bot, tt, tb, list, 4 * H);
  else if (total <= 256u) wave_rank_list<4>(list, total, k_top, k_bot, tt, tb, list, 4 * H);
  else wave_rank_list<8>(list, total, k_top, k_bot, tt, tb, list, 4 * H);
  return true;
}

// ------------------------------------------------------------------ four vectors per wave, one per row of 16 lanes
__device__ __forceinline__ uint32_t row16_sum_u(uint32_t v) {
  v += dpp_u<DPP_XOR1>(v);
  v += dpp_u<DPP_XOR2>(v);
  v += dpp_u<DPP_HALF_MIRROR>(v);
  v += dpp_u<DPP_MIRROR>(v);
  return v;
}
// As wave_rank_list for the four rows side by side; total: of my row.  The rough thresholds let a few entries too many
// through: they are dropped one by one, the least extreme first (a step costs the row's minimum, four lane exchanges).
template <int R>
__device__ __forceinline__ void row_rank_list(const uint32_t* list, uint32_t total, int k_top, int k_bot, uint32_t tt, uint32_t tb,
                                              uint32_t* smask) {
  const int i16 = lane_id() & 15;
  uint32_t ct[R], cb[R];
  uint32_t nt = 0, nb = 0;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const uint32_t p = (uint32_t)(i16 + 16 * i);
    ct[i] = 0xFFFFFFFFu;   // not a top candidate
    cb[i] = 0u;            // not a bottom candidate
    if (p < total) {
      const uint32_t e = list[p], key = key16(e >> 16), c = key << 16 | (e & 0xFFFFu);
      if (key >= tt) { ct[i] = c ^ 0xFFFFu; ++nt; }
      if (0xFFFFu - key >= tb) { cb[i] = c; ++nb; }
    }
  }
  const uint32_t both = row16_sum_u(nt | nb << 16);
  nt = both & 0xFFFFu;
  nb = both >> 16;
  while (__ballot(nt > (uint32_t)k_top || nb > (uint32_t)k_bot) != 0ull) {   // wave-uniform
    uint32_t m = ct[0], M = cb[0];
#pragma unroll
    for (int i = 1; i < R; ++i) {
      m = min(m, ct[i]);
      M = max(M, cb[i]);
    }
    m = row16_min_u(m);
    M = row16_max_u(M);
    const bool dt = nt > (uint32_t)k_top, db = nb > (uint32_t)k_bot;   // the same in the lanes of a row
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (dt && ct[i] == m) ct[i] = 0xFFFFFFFFu;
      if (db && cb[i] == M) cb[i] = 0u;
    }
    nt -= dt ? 1u : 0u;
    nb -= db ? 1u : 0u;
  }
  wave_lds_sync();   // (every lane has its entries: the mask may take the list's place)
  *reinterpret_cast<uint2*>(smask + 2 * i16) = make_uint2(0u, 0u);
  wave_lds_sync();
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const bool top = ct[i] != 0xFFFFFFFFu, bot = cb[i] != 0u;
    const uint32_t idx = top ? 0xFFFFu - (ct[i] & 0xFFFFu) : cb[i] & 0xFFFFu;
    if (top || bot) atomicOr(&smask[idx >> 5], 1u << (idx & 31u));
  }
  wave_lds_sync();
}

// Lane i of a row, piece h, entry e <-> index 128 h + 8 i + e of the row's vector, H <= 8 pieces in use.  raw: 8 * 64 pieces of LDS
// private to the wave; list: EXT_LIST words, of which a row takes EXT_ROW_LIST.  The sets' bits are left in smask =
// list[32 row .. 32 row + 4 H).  valid: whether my row has a vector.  Returns false where some row's candidates do not fit
// (wave-uniform).
__device__ __forceinline__ bool row_ext_select(const uint4 (&x)[8], int H, int k_top, int k_bot, bool valid, uint4* raw, uint32_t* list) {
  const int lane = lane_id(), row = lane >> 4, i16 = lane & 15;
  uint32_t w[4];   // two sets of four heads, two groups each: (key of the maximum, complement of the key of the minimum)
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    uint32_t mx = 0xFC00FC00u, mn = 0x7C007C00u;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * s + i < H) extend_extremes(x[4 * s + i], mx, mn);   // wave-uniform
    const uint32_t kx = key16x2(mx), kn = ~key16x2(mn);
    w[2 * s] = GEAR_BYTE_PERM(kn, kx, 0x05040100u);
    w[2 * s + 1] = GEAR_BYTE_PERM(kn, kx, 0x07060302u);
  }
  const uint32_t km1 = (uint32_t)(k_top > 1 ? k_top - 1 : 0) | (uint32_t)(k_bot > 1 ? k_bot - 1 : 0) << 16;
  uint32_t t2 = 0u;   // both thresholds, one per half
#pragma unroll
  for (int b = 15; b >= 7; --b) {   // nine bits: 1/8 of an octave
    const uint32_t q = t2 + (0x00010001u << b) - 0x00010001u;   // an entry counts iff it is > q, half by half
    uint32_t n = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) n += nonzero_u16x2(sub_sat_u16x2(w[i], q));
    n = row16_sum_u(n);
    t2 += nonzero_u16x2(sub_sat_u16x2(n, km1)) << b;
  }
  const uint32_t tt = k_top > 0 ? t2 & 0xFFFFu : 0x10000u, tb = k_bot > 0 ? t2 >> 16 : 0x10000u;
  const RoughBounds rb = rough_bounds(tt, tb);
  uint32_t f[2] = {0u, 0u};
#pragma unroll
  for (int h = 0; h < 8; ++h)
    if (h < H) {   // wave-uniform
      raw[h * 64 + lane] = x[h];
      const int j = (h & 3) * 4;
      f[h >> 2] |= outside_bits(x[h].x, rb, j) | outside_bits(x[h].y, rb, j + 1) | outside_bits(x[h].z, rb, j + 2) |
                   outside_bits(x[h].w, rb, j + 3);
    }
  if (!valid) f[0] = f[1] = 0u;
  const uint32_t cnt = (uint32_t)(__popc(f[0]) + __popc(f[1]));
  const uint32_t inc = row16_incl_prefix(cnt), total = row16_sum_u(cnt);
  wave_lds_sync();   // (the way out reuses both arrays)
  if (__ballot(valid && (!rough_usable(tt, tb) || total > EXT_ROW_LIST)) != 0ull) return false;
  uint32_t* mine = list + row * EXT_ROW_LIST;
  uint32_t pos = inc - cnt;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    while (f[q] != 0u) {
      const uint32_t p = (uint32_t)__ffs((int)f[q]) - 1u, wd = p & 15u, half = p >> 4;
      f[q] &= f[q] - 1u;
      const uint32_t h = 4u * q + (wd >> 2), e = 2u * (wd & 3u) + half;
      const uint32_t v = reinterpret_cast<const uint16_t*>(raw + h * 64u + lane)[e];
      mine[pos++] = (128u * h + 8u * i16 + e) | v << 16;
    }
  }
  wave_lds_sync();
  const int most = max(max((int)lane_bcast_u(total, 0), (int)lane_bcast_u(total, 16)), max((int)lane_bcast_u(total, 32), (int)lane_bcast_u(total, 48)));
  uint32_t* smask = list + row * 32;
  if (most <= 32) row_rank_list<2>(mine, total, k_top, k_bot, tt, tb, smask);
  else if (most <= 64) row_rank_list<4>(mine, total, k_top, k_bot, tt, tb, smask);
  else row_rank_list<8>(mine, total, k_top, k_bot, tt, tb, smask);
  return true;
}

}  // namespace gear
