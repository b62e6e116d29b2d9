// Key side of gear_compress: Filter_s (Eq. 4), i.e. which entries of every Key channel vector (over the call's tokens) go
// into S, and the launch of the quantization kernel (compress_quant.h).  The result of the Filter is a bit per entry,
// 16 bytes per token row.
//   k_select_tiny_kernel   segments of at most 64 tokens (a flushed buffer): one thread per vector
//   (it and k_select_reg_kernel's shortest segments mostly go together with the Values: select_pair_kernel)
//   k_select_stream_kernel more than 1024 tokens: candidates collected by blocks of 8 or 16 channels and 512 or 1024 threads, then ranked
//                          (gear_select_stream.h)
//   k_select_reg_kernel    otherwise up to 8192 tokens: one wave per vector, the vector in registers
//   k_select_long_kernel   otherwise: one wave per vector, from a channel-major copy of the keys
#include <math.h>
#include <atomic>
#include "gear_internal.h"
#include "gear_select.h"
#include "gear_launch.h"
#include "gear_select_stream.h"
#include "compress_select.h"
#include "compress_quant.h"

namespace gear {

// ------------------------------------------------------------------ K select, segments of at most 64 tokens
// grid (B*H), block 128.
__global__ __launch_bounds__(128) void k_select_tiny_kernel(const uint16_t* __restrict__ K, int n, int k_top, int k_bot,
                                                            uint4* __restrict__ mask, uint32_t* __restrict__ zero,
                                                            int zero_count, uint32_t* __restrict__ ksz, int ng_cap, float qmax) {
  __shared__ KTinySmem sm;
  k_select_tiny_block(sm, K, blockIdx.x, gridDim.x, n, k_top, k_bot, mask, zero, zero_count, ksz, ng_cap, qmax);
}

// ------------------------------------------------------------------ K select, segments of more than 8192 tokens
// Such a vector fits neither the registers of a wave nor, eight channels at a time, the LDS of a block, and
// read one channel at a time from the [token][channel] tensor every 2-byte value costs a whole memory
// sector.  So the keys are first written channel-major ([slab][channel][stride] u16, stride = n rounded up
// to 8) into scratch memory, and the selection then reads every vector contiguously, straight from global
// memory, once per pass.  LDS holds the histograms and the block's eight channels of outlier bits (32 KB).
struct GlobalKeySource {   // one vector stored contiguously in global memory as 16-bit keys
  static constexpr int kMaxChunks = -1;
  GEAR_BUF_T buf;          // view of the vector's stride keys; reads past it return 0
  __device__ __forceinline__ uint4 operator()(int ch) const { return GEAR_BUF_LOAD16(buf, (ch * 64 + lane_id()) * 16); }
};

// grid (ceil(n / 128), B*H), block 256: thread (rg, oc) takes the 16-byte pieces (8 channels) of rows
// 8 rg .. 8 rg + 7 of the tile, turns the values into keys, transposes the 8 x 8 block in registers and
// stores 8 tokens of each of its 8 channels with one 16-byte store.  Rows past n are written as the key of 0.
__global__ __launch_bounds__(256) void k_transpose_keys_kernel(const uint16_t* __restrict__ K, int n, int stride,
                                                               uint16_t* __restrict__ KT) {
  const int slab = blockIdx.y, tid = threadIdx.x, rg = tid >> 4, oc = tid & 15;
  const int row0 = blockIdx.x * 128 + rg * 8;
  const GEAR_BUF_T xb = GEAR_BUF_MAKE(K + (size_t)slab * n * D, n * (D * 2));
  uint32_t w[8][4];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const uint4 t4 = GEAR_BUF_LOAD16(xb, (row0 + k) * (D * 2) + oc * 16);
    w[k][0] = key16x2(t4.x); w[k][1] = key16x2(t4.y); w[k][2] = key16x2(t4.z); w[k][3] = key16x2(t4.w);
  }
  if (row0 >= stride) return;   // (stride is a multiple of 8: the 8 tokens lie inside or outside together)
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int j = c >> 1;
    const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;   // the high / the low halves of two words
    const uint4 o = make_uint4(GEAR_BYTE_PERM(w[1][j], w[0][j], sel), GEAR_BYTE_PERM(w[3][j], w[2][j], sel),
                               GEAR_BYTE_PERM(w[5][j], w[4][j], sel), GEAR_BYTE_PERM(w[7][j], w[6][j], sel));
    *reinterpret_cast<uint4*>(KT + ((size_t)slab * D + oc * 8 + c) * stride + row0) = o;
  }
}

// 1-D grid of 16 * nslab blocks of 512 threads, decoded like that of k_select_reg_kernel: one wave per channel vector.
__global__ __launch_bounds__(512) void k_select_long_kernel(const uint16_t* __restrict__ KT, int n, int stride, int nslab, int k_top,
                                                            int k_bot, uint4* __restrict__ mask,
                                                            uint32_t* __restrict__ zero, int zero_count,
                                                            uint32_t* __restrict__ ksz, int ng_cap, float qmax) {
  __shared__ uint32_t hist_all[8 * SELECT_LDS_WORDS];
  __shared__ __align__(16) uint32_t bits[32768 / 4];
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < zero_count; i += gridDim.x * blockDim.x) zero[i] = 0u;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int slab, cb;
  slab_and_column_block(blockIdx.x, nslab, D / 8, slab, cb);
  const int v = slab * D + cb * 8 + wave;   // vector: slab, channel
  const GlobalKeySource src{GEAR_BUF_MAKE(KT + (size_t)v * stride, stride * 2)};
  const Thresh th = wave_select(src, n, k_top, k_bot, hist_all + wave * SELECT_LDS_WORDS, true);
  const ThreshPair tp = pack_thresh(th);
  if (ksz) {
    // per-vector grouping: (scale, zero) of the channel's one group, from min and max of X - S
    uint32_t kmn = 0xFFFFu, kmx = 0u;
    for_each_chunk(src, (n + 511) >> 9, [&](int ch, const uint4& v4) {
      const int base = ch * 512 + lane * 8;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t k = slot16(v4, e);
        if (base + e < n) {
          const uint32_t y = outlier(k, (uint32_t)(base + e), tp) ? 0x8000u : k;
          kmn = min(kmn, y);
          kmx = max(kmx, y);
        }
      }
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      kmn = min(kmn, (uint32_t)__shfl_xor(kmn, o, 64));
      kmx = max(kmx, (uint32_t)__shfl_xor(kmx, o, 64));
    }
    if (lane == 0)
      ksz[(size_t)(v / D) * ng_cap * D + (v % D)] = group_bits(make_group(h2f(unkey16(kmn)), h2f(unkey16(kmx)), qmax));
  }
  if (!mask) return;
  const ThreshKeys tk = key_thresh(tp);
  for_each_chunk(src, (n + 511) >> 9, [&](int ch, const uint4& v4) { mark_chunk(v4, ch, bits, tp, tk); });
  block_lds_sync();
  store_mask_bytes(bits, mask + (size_t)slab * n, n, cb);
}

// ------------------------------------------------------------------ K select, vectors in registers
// grid 16 * nslab, block 512.
template <int NC>
__global__ __launch_bounds__(512, (NC <= 8 ? 4 : 2)) void k_select_reg_kernel(const uint16_t* __restrict__ K, int n, int nslab,
                                                                            int k_top, int k_bot, uint4* __restrict__ mask,
                                                                            uint32_t* __restrict__ zero, int zero_count,
                                                                            uint32_t* __restrict__ ksz, int ng_cap, float qmax) {
  __shared__ KRegSmem<NC> sm;
  k_select_reg_block<NC>(sm, K, blockIdx.x, n, nslab, k_top, k_bot, mask, zero, zero_count, ksz, ng_cap, qmax);
}

// ------------------------------------------------------------------ launchers
template <int NC>
static hipError_t launch_k_select_reg(const uint16_t* K, const Dims& dm, int n, int k_top, int k_bot, uint4* mask,
                                      uint32_t* zero, int zero_count, const SegView& sv, hipStream_t st) {
  hipLaunchKernelGGL(k_select_reg_kernel<NC>, dim3((D / 8) * dm.B * dm.H), dim3(512), 0, st, K, n, dm.B * dm.H, k_top, k_bot, mask,
                     zero, zero_count, dm.kcvt ? sv.sz : (uint32_t*)nullptr, sv.ng_cap, dm.qmax);
  return hipGetLastError();
}

template <int PC, int NB, bool ONCE, int T>
static hipError_t launch_k_select_stream(const uint16_t* K, const Dims& dm, int n, int k_top, int k_bot, const StreamPlan& p, uint4* mask,
                                         uint32_t* zero, int zero_count, const SegView& sv, hipStream_t st) {
  static std::atomic<uint64_t> lds_raised{0};
  const hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(k_select_stream_kernel<PC, NB, ONCE, T>), lds_raised, p.lds, LDS_PER_CU);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_select_stream_kernel<PC, NB, ONCE, T>), dim3((D / (8 * PC)) * dm.B * dm.H), dim3(T), p.lds, st, K, n, p.L, dm.B * dm.H,
                     k_top, k_bot, p.j_top, p.j_bot, p.cap, mask, zero, zero_count, dm.kcvt ? sv.sz : (uint32_t*)nullptr, sv.ng_cap,
                     dm.qmax);
  return hipGetLastError();
}

hipError_t launch_k_select(const uint16_t* K, const Dims& dm, int n, int k_top, int k_bot, uint4* mask,
                           uint32_t* zero, int zero_count, const SegView& sv, uint16_t* kt_scratch, hipStream_t st) {
  if (dm.ppm == 0) mask = nullptr;
  // Lists of candidates, where they fit (a ratio of a few per cent) and the work fills the chip.  A call at rank 0 and 2 %, before
  // and after: 512 slabs x 8192 tokens 1382 -> 1239 us, 128 x 20000 1184 -> 855, 32 x 32768 514 -> 421, 512 x 4096 630 -> 596, 1280 x 2048
  // 763 -> 731; 8 x 8192 64 -> 67 and 32 x 2048 42.5 -> 43, hence the bound on the rows.  Up to 1024 tokens the barriers between the phases
  // of a short vector cost more than its histograms do (512 x 1024: 164 against 178).  Up to 8192 tokens, where the other way reads the
  // column once too, the line lies between 5 % (512 x 8192: 1947 and 1952, 256 x 6000 898 -> 844) and 10 % (256 x 6000 928 against 954,
  // 1024 x 3000 1496 against 1588); beyond, 5 % is 893 -> 764 for 128 x 12000.
  StreamPlan p;
  const int slabs = dm.B * dm.H;
  if (mask && (n > 8192 || (n > 1024 && (long long)slabs * n > GEAR_STREAM_MIN_ROWS && 100LL * (k_top + k_bot) <= 6LL * n))) {
    const bool rest = dm.kcvt != 0;
    // (blocks of 8 channels where those of 16 are too few to go round: 3 x 9000 tokens 64.4 -> 53.6, 61.0 from a channel-major copy)
    const bool wide = n <= 8192 || 8 * slabs >= 128;
#define GEAR_STREAM(PC, NB, ONCE, T, LDS)                                                       \
  do {                                                                                       \
    if (stream_plan(PC, NB, ONCE, T, n, k_top, k_bot, rest, LDS, p))                                  \
      return launch_k_select_stream<PC, NB, ONCE, T>(K, dm, n, k_top, k_bot, p, mask, zero, zero_count, sv, st); \
  } while (0)
    // One block of 1024 threads and 16 channels per CU, whose lists may take all of its LDS, where these blocks come out nearly even: a
    // lone round of them beats half as many threads (32 slabs x 9000 at 2 % 116 -> 110 us, x 5000 at 5 % 116 -> 105, 10 x 8192 75 -> 72, but
    // 40 x 8192 135 -> 152), and blocks of 8 channels, which fetch each line twice as often, wherever the lists of two blocks per CU do not
    // fit (32 x 32768 at 1 % 381 -> 345, 24 x 20000 at 2 % 201 -> 184, 52 x 16000 376 -> 360, 128 x 20000 847 -> 816).  In a last
    // round that is a quarter empty the smaller blocks are level or ahead (48 slabs of 16000 to 32768 tokens 0.99 to 1.03, 40 1.01 to 1.04),
    // and so they are where the larger ones are at most half a round (16 slabs x 32768 207 against 223, 8 x 9001 60 against 68, 10 x 8000 at
    // 4 % 74 against 79).  Long lists keep a lone block at its ranking, which nothing then hides: from 4 % on several rounds of the
    // smaller blocks win (128 x 8000 at 4 % 450 against 475, 80 x 8504 at 5 % 375 against 403), at 3 % where the last round is an eighth empty
    // (80 x 11000 369 against 378, but 64 x 16000 448 against 434).
    if (n <= 2048) GEAR_STREAM(2, 8, true, 512, 80 * 1024);
    else if (n <= 4096) GEAR_STREAM(2, 16, true, 512, 80 * 1024);
    else {
      const int blocks = 8 * slabs, rounds = (blocks + GEAR_STREAM_CUS - 1) / GEAR_STREAM_CUS;
      const bool pairs = wide && stream_plan(2, 8, false, 512, n, k_top, k_bot, rest, 80 * 1024, p);
      const bool lone = rounds == 1 && (pairs || blocks > GEAR_STREAM_CUS / 2);
      const bool even = 200LL * (k_top + k_bot) <= 5LL * n ? 32 * blocks >= 25 * rounds * GEAR_STREAM_CUS
                                                           : 200LL * (k_top + k_bot) <= 7LL * n && 8 * blocks >= 7 * rounds * GEAR_STREAM_CUS;
      if (lone || (rounds > 1 && !pairs && even)) GEAR_STREAM(2, 8, false, 1024, LDS_PER_CU);
      if (pairs) GEAR_STREAM(2, 8, false, 512, 80 * 1024);
    }
    GEAR_STREAM(1, 8, false, 512, LDS_PER_CU);
#undef GEAR_STREAM
  }
  // segments of more than 8192 tokens: through a channel-major copy of the keys
  if (n > 8192) {
    const int stride = (n + 7) & ~7;
    hipLaunchKernelGGL(k_transpose_keys_kernel, dim3((n + 127) / 128, dm.B * dm.H), dim3(256), 0, st, K, n, stride, kt_scratch);
    hipLaunchKernelGGL(k_select_long_kernel, dim3(dm.B * dm.H * (D / 8)), dim3(512), 0, st, (const uint16_t*)kt_scratch, n,
                       stride, dm.B * dm.H, k_top, k_bot, mask, zero, zero_count, dm.kcvt ? sv.sz : (uint32_t*)nullptr, sv.ng_cap, dm.qmax);
    return hipGetLastError();
  }
  // a flushed buffer: one thread per channel vector
  if (n <= KSEL_TINY_ROWS) {
    hipLaunchKernelGGL(k_select_tiny_kernel, dim3(dm.B * dm.H), dim3(128), 0, st, K, n, k_top, k_bot, mask, zero, zero_count,
                       dm.kcvt ? sv.sz : (uint32_t*)nullptr, sv.ng_cap, dm.qmax);
    return hipGetLastError();
  }
  // otherwise the channel vectors live in registers
  if (n > 4096) return launch_k_select_reg<16>(K, dm, n, k_top, k_bot, mask, zero, zero_count, sv, st);
  if (n > 2048) return launch_k_select_reg<8>(K, dm, n, k_top, k_bot, mask, zero, zero_count, sv, st);
  if (n > 1024) return launch_k_select_reg<4>(K, dm, n, k_top, k_bot, mask, zero, zero_count, sv, st);
  return launch_k_select_reg<2>(K, dm, n, k_top, k_bot, mask, zero, zero_count, sv, st);
}

template <int BITS>
static hipError_t launch_k_quant_b(const QuantArgs& a, hipStream_t st) {
  if (a.dm.kcvt) return launch_quant_t<true, BITS, KLG_VEC>(a, st);
  if (a.dm.g == 128) return launch_quant_t<true, BITS, 7>(a, st);
  if (a.dm.g == 64) return launch_quant_t<true, BITS, 6>(a, st);
  return launch_quant_t<true, BITS, 5>(a, st);
}
hipError_t launch_k_quant(const uint16_t* K, const SegView& sv, const Dims& dm, int n, int t_lr, uint4* mask, uint32_t* pool_ctr,
                          uint16_t* Yout, hipStream_t st) {
  const QuantArgs a{K, sv, dm, n, t_lr, QT, mask, nullptr, 0, 0, pool_ctr, Yout, nullptr};
  return dm.bits == 2 ? launch_k_quant_b<2>(a, st) : launch_k_quant_b<4>(a, st);
}

}  // namespace gear
