// Value side of gear_compress: Filter_s (Eq. 4), i.e. which entries of every Value token vector (the token's row over ALL
// heads' channels, index j = h*128 + c) go into S, one wave (or one row of 16 lanes) per token with the vector in registers,
// and the launch of the quantization kernel (compress_quant.h).  The result of the Filter is a bit per entry, 16 bytes per
// token row of a head.  (With the Filter per head the quantization kernel finds the entries by itself: a row's 16 lanes
// hold the whole vector there.)
#include "gear_internal.h"
#include "gear_select.h"
#include "gear_select_rows.h"
#include "gear_select_ext.h"
#include "gear_launch.h"
#include "compress_quant.h"

namespace gear {

template <int NC>
struct RegSource {  // the vector lives in the wave's registers
  static constexpr int kMaxChunks = NC;
  const uint4* x;
  __device__ __forceinline__ uint4 operator()(int ch) const { return x[ch]; }
};

// The mask of a token from the bits of its vector, which the selection leaves in LDS: lane h stores head h's 16 bytes.
__device__ __forceinline__ void store_token_mask(const uint32_t* smask, uint4* mask, int b, int H, int n, int t) {
  const int h = lane_id();
  if (h < H) mask[((size_t)b * H + h) * n + t] = *reinterpret_cast<const uint4*>(smask + 4 * h);
}

// grid (ceil(n / 4), B); block 256, one token per wave.
// lane l, chunk ch  <->  head 4*ch + l/16, channels 8*(l%16)..+7, i.e. in-vector index
// ch*512 + l*8 + e.
// Under the per-vector grouping (vsz != nullptr) the kernel also leaves the token's (scale, zero):
// its one Value group spans the whole vector, outliers counted as 0.  per_head: the Filter ranks
// each head's 128 channels (the 16 lanes of a row) on their own; the mask is then not stored (the quantization kernel
// finds the entries again, they cost less than their round trip).
template <int NC>
__global__ __launch_bounds__(256, (NC <= 8 ? 4 : NC <= 10 ? 3 : 2)) void v_select_kernel(const uint16_t* __restrict__ V, int H, int n, int k_top,
                                                       int k_bot, uint4* __restrict__ mask, uint32_t* __restrict__ vsz,
                                                       float qmax, int per_head) {
  __shared__ __align__(16) uint4 raw_all[4 * NC * 64];
  __shared__ __align__(16) uint32_t list_all[4 * EXT_LIST];
  static_assert(EXT_LIST >= SELECT_LDS_WORDS, "the histograms of the way out take the list's place");
  const int b = blockIdx.y;
  const int tid = threadIdx.x, wave = tid >> 6;
  const int N = H * D;
  uint4* raw = raw_all + wave * (NC * 64);
  uint32_t* list = list_all + wave * EXT_LIST;
  // (a view of the batch element's H * n rows: heads past H read as 0)
  const GEAR_BUF_T vb = GEAR_BUF_MAKE(V + (size_t)b * H * n * D, (uint32_t)H * n * (D * 2));
  const int lane = tid & 63, hsub = lane >> 4, oc = lane & 15;
  const int t = blockIdx.x * 4 + wave;
  if (t >= n) return;   // (waves are independent)
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
