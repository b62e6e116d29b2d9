// Value side of gear_compress: Filter_s (Eq. 4), i.e. which entries of every Value token vector (the token's row over ALL
// heads' channels, index j = h*128 + c) go into S, one wave (or one row of 16 lanes) per token with the vector in registers,
// and the launch of the quantization kernel (compress_quant.h).  The result of the Filter is a bit per entry, 16 bytes per
// token row of a head.  (With the Filter per head the quantization kernel finds the entries by itself: a row's 16 lanes
// hold the whole vector there.)
#include "gear_internal.h"
#include "gear_select.h"
#include "gear_select_rows.h"
#include "gear_launch.h"
#include "compress_quant.h"

namespace gear {

template <int NC>
struct RegSource {  // the vector lives in the wave's registers
  static constexpr int kMaxChunks = NC;
  const uint4* x;
  __device__ __forceinline__ uint4 operator()(int ch) const { return x[ch]; }
};

// grid (ceil(n / (4 * tpw)), B); block 256: tpw tokens per wave, one after another.
// lane l, chunk ch  <->  head 4*ch + l/16, channels 8*(l%16)..+7, i.e. in-vector index
// ch*512 + l*8 + e.
// Under the per-vector grouping (vsz != nullptr) the kernel also leaves the token's (scale, zero):
// its one Value group spans the whole vector, outliers counted as 0.  per_head: the Filter ranks
// each head's 128 channels (the 16 lanes of a row) on their own; the mask is then not stored (the quantization kernel
// finds the entries again, they cost less than their round trip).
template <int NC>
__global__ __launch_bounds__(256, (NC <= 8 ? 5 : NC <= 10 ? 4 : 2)) void v_select_kernel(const uint16_t* __restrict__ V, int H, int n, int tpw, int k_top,
                                                       int k_bot, uint4* __restrict__ mask, uint32_t* __restrict__ vsz,
                                                       float qmax, int per_head) {
  __shared__ uint32_t hist[4 * SELECT_LDS_WORDS];
  const int b = blockIdx.y;
  const int tid = threadIdx.x, wave = tid >> 6;
  const int N = H * D;
  for (int i = 0; i < tpw; ++i) {
    int lane = tid & 63;
    GEAR_PIN_VGPR(lane);   // (indices made from it are not kept over the loop)
    const int hsub = lane >> 4, oc = lane & 15;
    const int t = (blockIdx.x * tpw + i) * 4 + wave;
    const bool tvalid = t < n;
    // (a view of the batch element's H * n rows: heads past H read as 0; entries past N are
    // never looked at by the selection, they only have to be defined)
    const GEAR_BUF_T vb = GEAR_BUF_MAKE(V + (size_t)b * H * n * D, tvalid ? (uint32_t)H * n * (D * 2) : 0u);
    const uint32_t off0 = ((uint32_t)hsub * n + t) * (D * 2) + oc * 16;
    uint4 x[NC];
#pragma unroll
    for (int ch = 0; ch < NC; ++ch) {
      const uint4 raw = GEAR_BUF_LOAD16(vb, off0 + (uint32_t)ch * 4u * n * (D * 2));
      x[ch] = make_uint4(key16x2(raw.x), key16x2(raw.y), key16x2(raw.z), key16x2(raw.w));
    }
    ThreshPair tp = pack_thresh(thresh_none());
    if (!per_head) {
      RegSource<NC> src{x};
      const Thresh th = wave_select(src, N, k_top, k_bot, hist + wave * SELECT_LDS_WORDS, tvalid);
      tp = pack_thresh(th);
      if (tvalid && mask) {
        const ThreshKeys tk = key_thresh(tp);
        const bool cut = __ballot(tk.cut) != 0ull;   // wave-uniform
#pragma unroll
        for (int ch = 0; ch < NC; ++ch) {
          if (ch * 4 + hsub < H)
            reinterpret_cast<uint8_t*>(mask + ((size_t)b * H + ch * 4 + hsub) * n + t)[oc] =
                (uint8_t)(cut ? piece_bits(x[ch], (uint32_t)(ch * 512 + lane * 8), tp) : key_bits(x[ch], tk));
          GEAR_SCHED_FENCE();
        }
      }
    }
    if (vsz) {
      uint32_t kmn = 0xFFFFu, kmx = 0u;
#pragma unroll
      for (int ch = 0; ch < NC; ++ch) {
        const uint32_t kw[4] = {x[ch].x, x[ch].y, x[ch].z, x[ch].w};
        uint32_t idx0 = (uint32_t)(ch * 512 + lane * 8);          // index in the token's row over all heads
        if (per_head) {
          tp = row16_thresholds(kw, oc, k_top, k_bot);            // this head's own thresholds,
          idx0 = (uint32_t)(oc * 8);                              // on the index inside the head
        }
        if (ch * 512 + lane * 8 < N) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const uint32_t k = slot_key(kw, e), y = outlier(k, idx0 + e, tp) ? 0x8000u : k;
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
      if (tvalid && lane == 0) vsz[(size_t)b * n + t] = group_bits(make_group(h2f(unkey16(kmn)), h2f(unkey16(kmx)), qmax));
    }
  }
}

// The same thresholds for token rows of at most 1024 entries (up to eight KV heads), four tokens per
// wave: row r of 16 lanes takes token 4 (4 (blockIdx.x tpw + it) + wave) + r, lane i of the row the
// 16-byte piece i (channels 8 i .. 8 i + 7) of each head (gear_select_rows.h).  grid (ceil(n / (16 tpw)), B),
// block 256, 2 KB of LDS per row.  vsz: nullptr unless the per-vector grouping is on.
__global__ __launch_bounds__(256, 4) void v_select_rows_kernel(const uint16_t* __restrict__ V, int H, int n, int tpw,
                                                               int k_top, int k_bot, uint4* __restrict__ mask,
                                                               uint32_t* __restrict__ vsz, float qmax) {
  __shared__ __attribute__((aligned(16))) uint32_t hist[16 * SELECT_ROW_LDS_WORDS];
  const int b = blockIdx.y;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, row = lane >> 4;
  uint32_t* hrow = hist + (wave * 4 + row) * SELECT_ROW_LDS_WORDS;
  // a view of the batch element's H * n rows; a lane whose token does not exist reads past it (zeros)
  const GEAR_BUF_T vb = GEAR_BUF_MAKE(V + (size_t)b * H * n * D, (uint32_t)H * n * (D * 2));
  for (int it = 0; it < tpw; ++it) {
    int i = tid & 15;
    GEAR_PIN_VGPR(i);   // (indices made from it are not kept over the loop)
    const int t = ((blockIdx.x * tpw + it) * 4 + wave) * 4 + row;
    const bool tvalid = t < n;
    const uint32_t off0 = tvalid ? (uint32_t)t * (D * 2) + i * 16 : 0xFFFFFF00u;
    uint4 x[8];
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      x[h] = make_uint4(0, 0, 0, 0);
      if (h < H) {
        const uint4 raw = GEAR_BUF_LOAD16(vb, tvalid ? off0 + (uint32_t)h * n * (D * 2) : off0);
        x[h] = make_uint4(key16x2(raw.x), key16x2(raw.y), key16x2(raw.z), key16x2(raw.w));
      }
    }
    ThreshPair tp = pack_thresh(thresh_none());
    if (k_top > 0 || k_bot > 0) {
      tp = pack_thresh(row_select(x, H, k_top, k_bot, hrow));
      const ThreshKeys tk = key_thresh(tp);
      const bool cut = __ballot(tk.cut) != 0ull;   // wave-uniform
      if (tvalid && mask) {
#pragma unroll
        for (int h = 0; h < 8; ++h) {
          if (h < H)
            reinterpret_cast<uint8_t*>(mask + ((size_t)b * H + h) * n + t)[i] =
                (uint8_t)(cut ? piece_bits(x[h], (uint32_t)(128 * h + 8 * i), tp) : key_bits(x[h], tk));
          GEAR_SCHED_FENCE();
        }
      }
    }
    if (vsz) {   // per-vector grouping: the token's (scale, zero), outliers counted as 0
      uint32_t kmn = 0xFFFFu, kmx = 0u;
#pragma unroll
      for (int h = 0; h < 8; ++h)
        if (h < H) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const uint32_t k = slot16(x[h], e), y = outlier(k, (uint32_t)(128 * h + 8 * i + e), tp) ? 0x8000u : k;
            kmn = min(kmn, y);
            kmx = max(kmx, y);
          }
        }
      kmn = row16_min_u(kmn);
      kmx = row16_max_u(kmx);
      if (tvalid && i == 0) vsz[(size_t)b * n + t] = group_bits(make_group(h2f(unkey16(kmn)), h2f(unkey16(kmx)), qmax));
    }
  }
}

// ------------------------------------------------------------------ launchers
template <int NC>
static hipError_t launch_vsel(const uint16_t* V, const Dims& dm, int n, int k_top, int k_bot, uint4* mask, uint32_t* vsz,
                              hipStream_t st) {
  // four tokens per wave, or one when the call has few tokens (a flushed buffer)
  const int tpw = (long long)n * dm.B >= 16384 ? 4 : 1;
  dim3 grid((n + 4 * tpw - 1) / (4 * tpw), dm.B);
  hipLaunchKernelGGL(v_select_kernel<NC>, grid, dim3(256), 0, st, V, dm.H, n, tpw, k_top, k_bot, mask,
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
    const int tpw = tokens >= (1 << 18) ? 4 : tokens >= (1 << 16) ? 2 : 1;   // >= 4096 blocks before a block takes more tokens
    // (the (scale, zero) array exists only under the per-vector grouping)
    hipLaunchKernelGGL(v_select_rows_kernel, dim3((n + 16 * tpw - 1) / (16 * tpw), dm.B), dim3(256), 0, st, V, dm.H, n, tpw,
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
