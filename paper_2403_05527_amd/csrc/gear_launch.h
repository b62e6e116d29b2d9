// Host-side launch functions of the kernel translation units.
#pragma once
#include <atomic>
#include "gear_internal.h"

namespace gear {

// Lets a kernel be launched with up to `bytes` of dynamic LDS on the current device, where the launch asks for more (`need`) than any
// kernel may have without it.  The attribute belongs to a device's copy of the kernel, so every device that a process works on gets it.
// `raised`: one per kernel instance, a bit per device; two threads may both raise it: harmless.
inline hipError_t raise_dynamic_lds(const void* kernel, std::atomic<uint64_t>& raised, size_t need, size_t bytes) {
  if (need <= 64 * 1024) return hipSuccess;
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0ull;   // (further devices: raised on each call)
  if (raised.load(std::memory_order_relaxed) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) raised.fetch_or(bit, std::memory_order_relaxed);
  return e;
}
// A kernel without static LDS is raised to what a CU has, at once: were it raised to the size of each larger call, of two threads the
// one with the smaller size could set it last, below what the other is about to launch with.
constexpr size_t LDS_PER_CU = 160 * 1024;

// Chunk segments live in equally sized regions; view j = view 0 advanced by
// j * stride bytes on every pointer.
struct ChunkSet {
  SegView k0, v0;       // views of chunk 0 (n / rank filled per chunk on the device)
  uint64_t stride;      // bytes between consecutive chunk regions
  int n_chunks;
  uint8_t n[GEAR_MAX_CHUNKS];
  uint8_t rank[GEAR_MAX_CHUNKS];
};

hipError_t launch_fill_u32(uint32_t* p, uint32_t v, size_t count, hipStream_t st);

// mask: [slab][n], 16 bytes per token row: bit c = entry (row, c) belongs to S (Filter_s, Eq. 4); not written when ppm is 0.
// The Key kernel also clears zero[0 .. zero_count) (the list counters of the call); under the per-vector grouping it also
// writes every channel's (scale, zero) of the segment sv
hipError_t launch_k_select(const uint16_t* K, const Dims& dm, int n, int k_top, int k_bot, uint4* mask,
                           uint32_t* zero, int zero_count, const SegView& sv, uint16_t* kt_scratch, hipStream_t st);
// Both selections in one launch, where selects_in_pairs says so (the arguments of launch_k_select and launch_v_select).
bool selects_in_pairs(const Dims& dm, int n);
hipError_t launch_select_pair(const uint16_t* K, const uint16_t* V, const Dims& dm, int n, int k_top, int k_bot, int v_top, int v_bot,
                              uint4* maskK, uint4* maskV, uint32_t* zero, int zero_count, const SegView& ks, uint32_t* vsz, hipStream_t st);
// k_top / k_bot: per Value vector (the token's row over all heads); vsz: [B][n] words, a token's (scale, zero) under the
// per-vector grouping
hipError_t launch_v_select(const uint16_t* V, const Dims& dm, int n, int k_top, int k_bot, uint4* mask, uint32_t* vsz,
                           hipStream_t st);
// Quantization of one tensor given its mask (compress_quant.h).  Yout (nullable): [slab][n][128] fp16, Y = X - S, from which
// the low-rank solvers that walk over it re-derive the residual R = Y - D-hat.  k_top / k_bot (Values with the Filter per
// head, which this launch finds by itself): per head's vector.
constexpr int GRAM_TILES = 36;
constexpr int GRAM_FLOATS = GRAM_TILES * 256;
hipError_t launch_k_quant(const uint16_t* K, const SegView& sv, const Dims& dm, int n, int t_lr, uint4* mask, uint32_t* pool_ctr,
                          uint16_t* Yout, hipStream_t st);
hipError_t launch_v_quant(const uint16_t* V, const SegView& sv, const Dims& dm, int n, int t_lr, int k_top, int k_bot, uint4* mask,
                          const uint32_t* vsz, uint32_t* pool_ctr, uint16_t* Yout, hipStream_t st);
// Both tensors of a call in one launch.  gram != nullptr (in both): the same pass leaves the partial Gram matrices of the
// residual, [slab][strip of `strip` tokens][GRAM_FLOATS]; otherwise Yout as above.
struct QuantTensor {
  const uint16_t* X;
  SegView sv;
  uint4* mask;
  uint32_t* pool_ctr;
  uint16_t* Yout;
  float* gram;
};
hipError_t launch_quant_pair(const QuantTensor& k, const QuantTensor& v, const Dims& dm, int n, int t_lr, int v_top, int v_bot,
                             const uint32_t* vsz, int strip, hipStream_t st);

int pi_padded_rank(int rank);
// Tokens per strip of the pass that quantizes and forms the Gram matrices.  A strip is one block's work and leaves one partial
// matrix (36 KB) per tensor, which the solve kernel, one block per slab, adds up: the longest strips whose blocks, those of both
// tensors, fill the resident slots one and a quarter times (just above once, the few blocks of the second round cost as much as
// the first: 280 slabs of 1777 tokens in one strip each, 560 blocks, 524 us for a compress and decompress against 516 in two
// strips).  Counting one tensor only, with strips down to 128 tokens, took 160 us for a call on 5 x 8 slabs of 3001 tokens (now
// 140), 106 on 4 x 32 of 512 (95), 82 on 32 of 1003 (78), and twice the partials' memory.
// A grid that stays under an eighth of the slots with 256-token strips is a few blocks' latency: strips of 128 tokens halve the
// block's chain (8 slabs of 512 tokens 56 against 58 us).  Above that they gain a microsecond at most (32 slabs of 300 tokens 67
// against 68) or lose (32 of 512: 72 against 70), and their partials would be the largest array of such a cache.
constexpr int STRIP_BLOCKS = GEAR_BLOCK_SLOTS + GEAR_BLOCK_SLOTS / 4;
constexpr long long STRIP_ROWS_FEW = 256ll * (GEAR_BLOCK_SLOTS / 8);   // token rows of both tensors
inline int pi_gram_strip(int n, int slabs) {
  for (int strip = 2048; strip > 256; strip >>= 1)
    if (2ll * slabs * ((n + strip - 1) / strip) >= STRIP_BLOCKS) return strip;
  return 2ll * slabs * n >= STRIP_ROWS_FEW ? 256 : 128;
}
// The most strips per slab any segment of up to n_max tokens gets.  The strip length grows with n, and for one length the count
// does: the maximum lies at n_max or at the last n before a longer strip.
inline int pi_gram_strips_max(int n_max, int slabs) {
  const long long per = (STRIP_BLOCKS - 1) / (2ll * slabs);   // strips per slab that are too few
  int most = 0;
  auto take = [&](long long n) {
    if (n < 1) return;
    if (n > n_max) n = n_max;
    const int strip = pi_gram_strip((int)n, slabs), count = ((int)n + strip - 1) / strip;
    most = count > most ? count : most;
  };
  take(n_max);
  for (int strip = 512; strip <= 2048; strip <<= 1) take(strip * per);
  take((STRIP_ROWS_FEW - 1) / (2ll * slabs));
  return most;
}
// whether a segment of n tokens is solved on its Gram matrix (from X and its mask instead of Y)
inline bool pi_on_gram(int n, int rank, int iters) { return rank > 0 && iters > 1 && n > 256; }
// whether Keys and Values of a segment are solved together, launch by launch: on their Gram matrices, or (a flushed
// buffer, whose Y tensors are small) with the residual in LDS.  The other solvers work through the same scratch arrays,
// sized for one tensor, one tensor after the other.
constexpr int PI_TINY_ROWS = 64;
inline bool pi_paired(int n, int rank, int iters) { return rank > 0 && (n <= PI_TINY_ROWS || pi_on_gram(n, rank, iters)); }
// One tensor of a call.  sb: the start matrices of its slabs; X and mask (nullptr: nothing filtered) for the solver on
// the Gram matrix, Y = X - S for the others.
struct PiTensor {
  const uint16_t* X;
  const uint4* mask;
  const uint16_t* Y;
  SegView sv;
  StartB sb;
};
// t_lr: first token of the segment that takes part in the low-rank term (rows before it get A = 0)
// Bcur: [2][slab][128][padded rank]; gram: [2][slab][nstrips][GRAM_FLOATS], Keys first; the solver writes to both for its last pass
hipError_t launch_power_iteration_pair(const PiTensor& k, const PiTensor& v, const Dims& dm, int n, int t_lr, int iters, float* Bcur,
                                       float* gram, int nstrips, hipStream_t st);
hipError_t launch_power_iteration(bool is_k, const PiTensor& x, const Dims& dm, int n, int t_lr, int iters, float* Bcur, float* partial,
                                  float* Atmp, float* cmat, hipStream_t st);

constexpr int DECODE_SPLIT = 512;        // prefill tokens per split block
constexpr int DECODE_REC = 2 + D;        // floats per partial record: m, l, o[128]
// q: [B, H_q, q_len, 128]; q_len a power of two with (H_q / H) * q_len <= 8; causal: query row j sees the buffer
// rows 0 .. n_buf - q_len + j; partial: B * H_q * q_len * (records per row) * DECODE_REC floats
hipError_t launch_decode(const Dims& dm, const SegView& k0, const SegView& v0, const ChunkSet& cs,
                         const uint16_t* q, const uint16_t* Kbuf, const uint16_t* Vbuf, int n_buf,
                         int n_buf_cap, int rank_cap, int q_len, int causal, uint16_t* out, float* partial,
                         hipStream_t st);

hipError_t launch_decompress(const Dims& dm, const SegView& ks, const SegView& vs, uint16_t* Kout,
                             uint16_t* Vout, int n_total, hipStream_t st);
hipError_t launch_export_codes(const Dims& dm, const SegView& sv, bool is_k, uint8_t* codes, uint16_t* scale,
                               uint16_t* zero, int n_total, int ng_total, hipStream_t st);
hipError_t launch_export_sparse(const Dims& dm, const SegView& sv, bool is_k, uint8_t* mask, uint16_t* vals,
                                int n_total, hipStream_t st);
// COO view of S: count = true writes every token row's outlier count to rowcnt[slab * n_total + t]; count = false
// writes the rows' entries from the positions rowcnt then holds (launch_exclusive_scan in between; sums: scratch of
// ceil(count / 1024) words)
hipError_t launch_coo_tiles(const Dims& dm, const SegView& sv, bool is_k, bool count, uint32_t* rowcnt, long long* lin,
                            uint16_t* vals, int n_total, hipStream_t st);
hipError_t launch_exclusive_scan(uint32_t* v, size_t count, uint32_t* sums, hipStream_t st);
hipError_t launch_export_lowrank(const Dims& dm, const SegView& sv, uint16_t* A, uint16_t* Bf, hipStream_t st);

}  // namespace gear
