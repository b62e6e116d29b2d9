// Value side of gear_compress: Filter_s (Eq. 4), i.e. which entries of every Value token vector (the token's row over ALL
// heads' channels, index j = h*128 + c) go into S, one wave (or one row of 16 lanes) per token with the vector in registers,
// and the launch of the quantization kernel (compress_quant.h).  The result of the Filter is a bit per entry, 16 bytes per
// token row of a head.  (With the Filter per head the quantization kernel finds the entries by itself: a row's 16 lanes
// hold the whole vector there.)
#include <type_traits>
#include "gear_internal.h"
#include "gear_select.h"
#include "gear_select_rows.h"
#include "gear_select_ext.h"
#include "compress_select.h"
#include "gear_launch.h"
#include "compress_quant.h"

namespace gear {

// Tokens of a Value block of select_pair_kernel: as many waves as have room next to the Keys' LDS.
constexpr int pair_tokens(bool tiny, int nc) { return tiny ? 2 : nc <= 4 ? 8 : 4; }

// grid (ceil(n / 4), B); block 256, one token per wave.
template <int NC>
__global__ __launch_bounds__(256, (NC <= 8 ? 4 : NC <= 10 ? 3 : 2)) void v_select_kernel(const uint16_t* __restrict__ V, int H, int n, int k_top,
                                                       int k_bot, uint4* __restrict__ mask, uint32_t* __restrict__ vsz,
                                                       float qmax, int per_head) {
  __shared__ __align__(16) uint4 raw_all[4 * NC * 64];
  __shared__ __align__(16) uint32_t list_all[4 * EXT_LIST];
  const int wave = GEAR_WAVE_UNIFORM((int)(threadIdx.x >> 6)), t = blockIdx.x * 4 + wave;
  if (t >= n) return;   // (waves are independent)
  v_select_token<NC>(raw_all + wave * (NC * 64), list_all + wave * EXT_LIST, V, blockIdx.y, t, H, n, k_top, k_bot, mask, vsz, qmax, per_head);
}

// Both selections of a call with few blocks, in one launch: the first kblocks blocks take the Keys, the others WAVES tokens each.  Of a
// flushed buffer (TINY) or of a segment of up to 1024 tokens, each is a launch's latency and a short chain.
template <bool TINY, int NC>
__global__ __launch_bounds__(TINY ? 128 : 512, 4) void select_pair_kernel(const uint16_t* __restrict__ K, const uint16_t* __restrict__ V, int H, int n,
                                                                      int nslab, int k_top, int k_bot, int v_top, int v_bot,
                                                                      uint4* __restrict__ maskK, uint4* __restrict__ maskV,
                                                                      uint32_t* __restrict__ zero, int zero_count, uint32_t* __restrict__ ksz,
                                                                      int ng_cap, uint32_t* __restrict__ vsz, float qmax, int per_head) {
  constexpr int WAVES = pair_tokens(TINY, NC);
  __shared__ __align__(16) union {
    std::conditional_t<TINY, KTinySmem, KRegSmem<2>> k;
    struct {
      uint4 raw[WAVES][NC * 64];
      uint32_t list[WAVES][EXT_LIST];
    } v;
  } sm;
  const int kblocks = TINY ? nslab : (D / 8) * nslab;
  const int block = (int)blockIdx.x - kblocks;
  if (block < 0) {
    if constexpr (TINY) k_select_tiny_block(sm.k, K, blockIdx.x, nslab, n, k_top, k_bot, maskK, zero, zero_count, ksz, ng_cap, qmax);
    else k_select_reg_block<2>(sm.k, K, blockIdx.x, n, nslab, k_top, k_bot, maskK, zero, zero_count, ksz, ng_cap, qmax);
    return;
  }
  const int wave = GEAR_WAVE_UNIFORM((int)(threadIdx.x >> 6)), per = (n + WAVES - 1) / WAVES, b = block / per, t = (block - b * per) * WAVES + wave;
  if (wave >= WAVES || t >= n) return;   // (waves are independent)
  v_select_token<NC>(sm.v.raw[wave], sm.v.list[wave], V, b, t, H, n, v_top, v_bot, maskV, vsz, qmax, per_head);
}

// The same for token rows of at most 1024 entries (up to eight KV heads), four tokens per
// wave: row r of 16 lanes takes token 4 (4 blockIdx.x + wave) + r, lane i of the row the
// 16-byte piece i (channels 8 i .. 8 i + 7) of each head.  grid (ceil(n / 16), B),
// block 256.  vsz: nullptr unless the per-vector grouping is on.
__global__ __launch_bounds__(256, 4) void v_select_rows_kernel(const uint16_t* __restrict__ V, int H, int n,
                                                               int k_top, int k_bot, uint4* __restrict__ mask,
                                                               uint32_t* __restrict__ vsz, float qmax) {
  __shared__ __align__(16) uint4 raw_all[4 * 8 * 64];
  __shared__ __align__(16) uint32_t list_all[4 * EXT_LIST];
  static_assert(8 * 64 * 4 >= 4 * SELECT_ROW_LDS_WORDS, "the histograms of the way out take the raw values' place");
  const int b = blockIdx.y;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, row = lane >> 4;
  uint4* raw = raw_all + wave * (8 * 64);
  uint32_t* list = list_all + wave * EXT_LIST;
  // a view of the batch element's H * n rows; a lane whose token does not exist reads past it (zeros)
  const GEAR_BUF_T vb = GEAR_BUF_MAKE(V + (size_t)b * H * n * D, (uint32_t)H * n * (D * 2));
  const int i = tid & 15;
  const int t0 = (blockIdx.x * 4 + wave) * 4, t = t0 + row;
  if (t0 >= n) return;   // (waves are independent)
  const bool tvalid = t < n;
  const uint32_t off0 = tvalid ? (uint32_t)t * (D * 2) + i * 16 : 0xFFFFFF00u;
  uint4 x[8];
  auto load_rows = [&]() {
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      x[h] = make_uint4(0, 0, 0, 0);
      if (h < H) x[h] = GEAR_BUF_LOAD16(vb, tvalid ? off0 + (uint32_t)h * n * (D * 2) : off0);
    }
  };
  load_rows();
  const bool filt = k_top > 0 || k_bot > 0;
  if (filt && !row_ext_select(x, H, k_top, k_bot, tvalid, raw, list)) {
#pragma unroll
    for (int h = 0; h < 8; ++h) x[h] = make_uint4(key16x2(x[h].x), key16x2(x[h].y), key16x2(x[h].z), key16x2(x[h].w));
    const ThreshPair tp = pack_thresh(row_select(x, H, k_top, k_bot, reinterpret_cast<uint32_t*>(raw) + row * SELECT_ROW_LDS_WORDS));
    const ThreshKeys tk = key_thresh(tp);
    const bool cut = __ballot(tk.cut) != 0ull;   // wave-uniform
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      if (h < H)
        reinterpret_cast<uint8_t*>(list + row * 32)[h * 16 + i] =
            (uint8_t)(cut ? piece_bits(x[h], (uint32_t)(128 * h + 8 * i), tp) : key_bits(x[h], tk));
      GEAR_SCHED_FENCE();
    }
    wave_lds_sync();
    if (vsz) load_rows();
  }
  if (filt && mask) {   // lane 4 h + r stores the 16 bytes of head h of the wave's token r
    const int h = lane >> 2, r = lane & 3;
    if (h < H && t0 + r < n) mask[((size_t)b * H + h) * n + t0 + r] = *reinterpret_cast<const uint4*>(list + r * 32 + h * 4);
  }
  if (vsz) {   // per-vector grouping: the token's (scale, zero), outliers counted as 0
    uint32_t mn = 0x7C007C00u, mx = 0xFC00FC00u;
#pragma unroll
    for (int h = 0; h < 8; ++h)
      if (h < H) {
        const uint32_t f = filt ? reinterpret_cast<const uint8_t*>(list + row * 32)[h * 16 + i] : 0u;
        extend_extremes(drop_entries(x[h], f), mx, mn);
      }
    mn = key16x2(mn);
    mx = key16x2(mx);
    const uint32_t kmn = row16_min_u(min(mn & 0xFFFFu, mn >> 16)), kmx = row16_max_u(max(mx & 0xFFFFu, mx >> 16));
    if (tvalid && i == 0) vsz[(size_t)b * n + t] = group_bits(make_group(h2f(unkey16(kmn)), h2f(unkey16(kmx)), qmax));
  }
}

// ------------------------------------------------------------------ launchers
template <int NC>
static hipError_t launch_vsel(const uint16_t* V, const Dims& dm, int n, int k_top, int k_bot, uint4* mask, uint32_t* vsz,
                              hipStream_t st) {
  hipLaunchKernelGGL(v_select_kernel<NC>, dim3((n + 3) / 4, dm.B), dim3(256), 0, st, V, dm.H, n, k_top, k_bot, mask,
                     dm.kcvt ? vsz : (uint32_t*)nullptr, dm.qmax, dm.vhead);
  return hipGetLastError();
}

hipError_t launch_v_select(const uint16_t* V, const Dims& dm, int n, int k_top, int k_bot, uint4* mask, uint32_t* vsz,
                           hipStream_t st) {
  // the pass over whole token rows: the per-token Filter, and a token's (scale, zero) under the per-vector grouping
  if (!((dm.ppm > 0 && !dm.vhead) || dm.kcvt)) return hipSuccess;
  const int kt = dm.ppm > 0 ? k_top : 0, kb = dm.ppm > 0 ? k_bot : 0;
  if (dm.ppm == 0 || dm.vhead) mask = nullptr;
  const int nc = (dm.H + 3) / 4;
  const long long tokens = (long long)dm.B * n;
  // short token rows: four tokens per wave (a flushed buffer has too few tokens to fill the chip that way)
  if (dm.H <= 8 && !dm.vhead && tokens >= GEAR_ROWS_MIN_TOKENS) {
    // (the (scale, zero) array exists only under the per-vector grouping)
    hipLaunchKernelGGL(v_select_rows_kernel, dim3((n + 15) / 16, dm.B), dim3(256), 0, st, V, dm.H, n,
                       kt, kb, mask, dm.kcvt ? vsz : (uint32_t*)nullptr, dm.qmax);
    return hipGetLastError();
  }
  if (nc <= 2) return launch_vsel<2>(V, dm, n, kt, kb, mask, vsz, st);
  if (nc <= 4) return launch_vsel<4>(V, dm, n, kt, kb, mask, vsz, st);
  if (nc <= 8) return launch_vsel<8>(V, dm, n, kt, kb, mask, vsz, st);
  if (nc <= 10) return launch_vsel<10>(V, dm, n, kt, kb, mask, vsz, st);
  return launch_vsel<16>(V, dm, n, kt, kb, mask, vsz, st);
}

template <bool TINY, int NC>
static hipError_t launch_pair(const uint16_t* K, const uint16_t* V, const Dims& dm, int n, int k_top, int k_bot, int v_top, int v_bot,
                              uint4* maskK, uint4* maskV, uint32_t* zero, int zero_count, const SegView& ks, uint32_t* vsz, hipStream_t st) {
  constexpr int W = pair_tokens(TINY, NC);
  const int slabs = dm.B * dm.H;
  hipLaunchKernelGGL((select_pair_kernel<TINY, NC>), dim3((TINY ? 1 : D / 8) * slabs + dm.B * ((n + W - 1) / W)), dim3(TINY ? 128 : 512), 0, st, K, V,
                     dm.H, n, slabs, k_top, k_bot, v_top, v_bot, maskK, maskV, zero, zero_count, dm.kcvt ? ks.sz : (uint32_t*)nullptr,
                     ks.ng_cap, dm.kcvt ? vsz : (uint32_t*)nullptr, dm.qmax, dm.vhead);
  return hipGetLastError();
}
// A flushed buffer's selections go together at every number of slabs (a call of rank 2, launch after launch -> together: 32 slabs x 20 tokens
// 25.2 -> 21.1 us, 512 x 20 36.2 -> 32.0, 2048 x 20 90.9 -> 88.1, 256 x 64 46.1 -> 39.0), those of up to 1024 tokens while they leave the
// chip half empty (a call of rank 4, 32 x 512 48.8 -> 45.5, 64 x 1000 71.9 -> 68.3, but 128 x 512 72.5 -> 74.6, 256 x 800 level: the Value
// blocks hold the Keys' LDS and half of the waves).
constexpr int PAIR_SLABS = 64;
bool selects_in_pairs(const Dims& dm, int n) {
  if (!((dm.ppm > 0 && !dm.vhead) || dm.kcvt)) return false;   // no pass over the Values
  if (dm.H > 32 || (dm.H <= 8 && !dm.vhead && (long long)dm.B * n >= GEAR_ROWS_MIN_TOKENS)) return false;   // (other Value kernels)
  return n <= KSEL_TINY_ROWS || (n <= 1024 && dm.B * dm.H <= PAIR_SLABS);
}
hipError_t launch_select_pair(const uint16_t* K, const uint16_t* V, const Dims& dm, int n, int k_top, int k_bot, int v_top, int v_bot,
                              uint4* maskK, uint4* maskV, uint32_t* zero, int zero_count, const SegView& ks, uint32_t* vsz, hipStream_t st) {
  if (dm.ppm == 0) {
    k_top = k_bot = v_top = v_bot = 0;
    maskK = maskV = nullptr;
  }
  if (dm.vhead) maskV = nullptr;
  const int nc = (dm.H + 3) / 4;
#define GEAR_PAIR(TINY)                                                                                                                      \
  do {                                                                                                                                       \
    if (nc <= 2) return launch_pair<TINY, 2>(K, V, dm, n, k_top, k_bot, v_top, v_bot, maskK, maskV, zero, zero_count, ks, vsz, st);            \
    if (nc <= 4) return launch_pair<TINY, 4>(K, V, dm, n, k_top, k_bot, v_top, v_bot, maskK, maskV, zero, zero_count, ks, vsz, st);            \
    return launch_pair<TINY, 8>(K, V, dm, n, k_top, k_bot, v_top, v_bot, maskK, maskV, zero, zero_count, ks, vsz, st);                         \
  } while (0)
  if (n <= KSEL_TINY_ROWS) GEAR_PAIR(true);
  GEAR_PAIR(false);
#undef GEAR_PAIR
}

template <int BITS>
static hipError_t launch_v_quant_b(const QuantArgs& a, hipStream_t st) {
  if (a.dm.g == 128) return launch_quant_t<false, BITS, 7>(a, st);
  if (a.dm.g == 64) return launch_quant_t<false, BITS, 6>(a, st);
  return launch_quant_t<false, BITS, 5>(a, st);
}
hipError_t launch_v_quant(const uint16_t* V, const SegView& sv, const Dims& dm, int n, int t_lr, int k_top, int k_bot, uint4* mask,
                          const uint32_t* vsz, uint32_t* pool_ctr, uint16_t* Yout, hipStream_t st) {
  const QuantArgs a{V, sv, dm, n, t_lr, QT, mask, vsz, k_top, k_bot, pool_ctr, Yout, nullptr};
  return dm.bits == 2 ? launch_v_quant_b<2>(a, st) : launch_v_quant_b<4>(a, st);
}

template <int BITS, int KLG, int VLG>
static hipError_t launch_quant_pair_t(const QuantArgs& k, const QuantArgs& v, hipStream_t st) {
  const dim3 grid((k.n + k.strip - 1) / k.strip, k.dm.B * k.dm.H, 2);
  if (k.gram) hipLaunchKernelGGL((quant_pair_kernel<BITS, KLG, VLG, true>), grid, dim3(256), 0, st, k, v);
  else hipLaunchKernelGGL((quant_pair_kernel<BITS, KLG, VLG, false>), grid, dim3(256), 0, st, k, v);
  return hipGetLastError();
}
template <int BITS>
static hipError_t launch_quant_pair_b(const QuantArgs& k, const QuantArgs& v, hipStream_t st) {
  if (k.dm.kcvt) return launch_quant_pair_t<BITS, KLG_VEC, 7>(k, v, st);   // (a Value row's one group: all 128 channels of a head)
  if (k.dm.g == 128) return launch_quant_pair_t<BITS, 7, 7>(k, v, st);
  if (k.dm.g == 64) return launch_quant_pair_t<BITS, 6, 6>(k, v, st);
  return launch_quant_pair_t<BITS, 5, 5>(k, v, st);
}
hipError_t launch_quant_pair(const QuantTensor& k, const QuantTensor& v, const Dims& dm, int n, int t_lr, int v_top, int v_bot,
                             const uint32_t* vsz, int strip, hipStream_t st) {
  const QuantArgs ka{k.X, k.sv, dm, n, t_lr, strip, k.mask, nullptr, 0, 0, k.pool_ctr, k.Yout, k.gram};
  const QuantArgs va{v.X, v.sv, dm, n, t_lr, strip, v.mask, vsz, v_top, v_bot, v.pool_ctr, v.Yout, v.gram};
  return dm.bits == 2 ? launch_quant_pair_b<2>(ka, va, st) : launch_quant_pair_b<4>(ka, va, st);
}

}  // namespace gear
