// gear_decode_attn: single-query attention (Eq. 1) read directly from the
// compressed cache.  K-hat and V-hat are never materialised:
//   score_t = q . D_K[t] + (q^T B_K) . A_K[t] + q . S_K[t]
//   out     = sum_t p_t D_V[t] + (p^T A_V) B_V^T + p^T S_V
// (the low-rank term as a down- then up-projection, as the paper's
// implementation notes describe), followed by the fp16 buffer rows.
//
// Split-KV: block (split, b*H_kv + h) handles DECODE_SPLIT tokens of the prefill
// segment for all query heads of the KV head on the matrix cores
// (decode_mfma.h); the last split index handles the appended chunk segments and
// the fp16 buffer (decode_tail.h).  Every block writes one partial softmax
// record (m, l, o) per query head; decode_combine merges the records.
// A cache of few pieces is read by one block per slab instead, in one launch
// (decode_single_kernel, chosen by read_plan).
#include <atomic>
#include "gear_internal.h"
#include "gear_launch.h"
#include "decode_mfma.h"
#include "decode_tail.h"

namespace gear {

static_assert(MFMA_TS == DECODE_SPLIT, "split size is part of the workspace layout");

// grid (nsplit + ncb + 1, B*H_kv << lparts), block 256: a slab's query columns are shared by 2^lparts blocks, GQ
// columns each (read_plan).  Blocks [0, nsplit): 512 prefill tokens each;
// blocks [nsplit, nsplit + ncb): four pieces of appended chunks each (one piece = up to 128
// rows of one chunk, pp pieces per chunk), through the same code as the prefill; the
// last block: the fp16 streaming-buffer rows.
template <int BITS, int GQ, int LG>
__global__ __launch_bounds__(256, (GQ == 8 ? 3 : (BITS == 2 && (GQ <= 2 || (GQ == 4 && LG >= 6))) ? 5 : 4)) void decode_split_kernel(Dims dm, SegView k0, SegView v0, ChunkSet cs,
                                                              const uint16_t* __restrict__ q,
                                                              const uint16_t* __restrict__ Kbuf,
                                                              const uint16_t* __restrict__ Vbuf, int n_buf,
                                                              int n_buf_cap, int nsplit, int pp, int rank_cap,
                                                              int odd_rank, int q_len, int causal, int lparts,
                                                              float* __restrict__ partial) {
  GEAR_DYN_LDS(smem_raw);
  const int slab = blockIdx.y >> lparts, split = blockIdx.x;
  const int nrec = (int)gridDim.x;
  const int b = slab / dm.H;
  const int row0 = (int)blockIdx.y * GQ;   // the block's first query row: the columns of a slab, and the slabs, lie in a row
  float* rec_base = partial + ((size_t)row0 * nrec + split) * DECODE_REC;
  const int rec_stride = nrec * DECODE_REC;
  const uint16_t* qg = q + (size_t)row0 * D;
  const int wave = GEAR_WAVE_UNIFORM((int)(threadIdx.x >> 6));
  if (split == nrec - 1) {
    buffer_block<GQ>(*reinterpret_cast<TailSmem<GQ>*>(smem_raw), qg, Kbuf + (size_t)slab * n_buf_cap * D,
                     Vbuf + (size_t)slab * n_buf_cap * D, n_buf, q_len, causal, row0, rec_base, rec_stride);
    return;
  }
  // one call site: the prefill segment for every wave, or one chunk piece per wave
  // (piece i = 4 * (split - nsplit) + wave covers rows [128 * (i % pp), ...) of chunk i / pp)
  SegView kw_ = k0, vw_ = v0;
  int tw0 = split * MFMA_TS + WTOK * wave, nw = k0.n - tw0;
  if (split >= nsplit) {
    const int item = 4 * (split - nsplit) + wave;
    const int j = pp == 2 ? item >> 1 : item, part = item - j * pp;   // pp is 1 or 2
    int n_j = 0, r_j = 0;
    if (j < cs.n_chunks) {
      n_j = cs.n[j];
      r_j = cs.rank[j];
    }
    kw_ = chunk_view(cs.k0, cs.stride, j < cs.n_chunks ? j : 0, n_j, r_j);
    vw_ = chunk_view(cs.v0, cs.stride, j < cs.n_chunks ? j : 0, n_j, r_j);
    tw0 = WTOK * part;
    nw = n_j - tw0;
  }
  mfma_block<BITS, GQ, LG, false>(smem_raw, dm, kw_, vw_, qg, slab, b, tw0, nw, k0.rank, v0.rank, rank_cap, odd_rank != 0,
                                  split < nsplit, rec_base, rec_stride, 0, 0, 0);
}

// The whole read of a slab (or of a part of its query columns) in one block, for caches of few pieces (read_plan): grid
// (B*H_kv << lparts), a wave per 128 prefill tokens, then one per chunk piece, then one per 32 buffer rows.  The states meet in
// LDS and the block writes the result itself: no records and no second launch.  Bound by one wave's chain of dependent steps and the launch; each wave adds its own zero-point
// and low-rank terms, so that the merge behind the barrier is one plane read per wave.
template <int BITS, int GQ, int LG>
__global__ __launch_bounds__(64 * SINGLE_WAVES<GQ>) void decode_single_kernel(Dims dm, SegView k0, SegView v0, ChunkSet cs,
                                                                              const uint16_t* __restrict__ q,
                                                                              const uint16_t* __restrict__ Kbuf,
                                                                              const uint16_t* __restrict__ Vbuf, int n_buf,
                                                                              int n_buf_cap, int npw, int ncw, int pp, int rank_cap,
                                                                              int odd_rank, int q_len, int causal, int lparts,
                                                                              uint16_t* __restrict__ out) {
  GEAR_DYN_LDS(smem_raw);
  const int slab = blockIdx.x >> lparts, b = slab / dm.H;
  const int row0 = (int)blockIdx.x * GQ;   // the block's first query row
  const uint16_t* qg = q + (size_t)row0 * D;
  const int wave = GEAR_WAVE_UNIFORM((int)(threadIdx.x >> 6)), nthreads = (int)blockDim.x, nwaves = nthreads >> 6;
  const MfmaLayout L = mfma_layout<GQ>(BITS, 1 << LG, k0.rank, v0.rank, rank_cap, odd_rank != 0, nwaves, ncw);
  if (wave >= npw + ncw) {
    buffer_wave<GQ>(smem_raw, L, qg, Kbuf + (size_t)slab * n_buf_cap * D, Vbuf + (size_t)slab * n_buf_cap * D, n_buf,
                    (wave - npw - ncw) * BUF_WAVE_ROWS, q_len, causal, row0, wave, nthreads);
  } else {
    SegView kw_ = k0, vw_ = v0;
    int tw0 = WTOK * wave, nw = k0.n - tw0;
    const int item = wave - npw;
    if (item >= 0) {
      const int j = pp == 2 ? item >> 1 : item, part = item - j * pp;   // pp is 1 or 2
      kw_ = chunk_view(cs.k0, cs.stride, j, cs.n[j], cs.rank[j]);
      vw_ = chunk_view(cs.v0, cs.stride, j, cs.n[j], cs.rank[j]);
      tw0 = WTOK * part;
      nw = cs.n[j] - tw0;
    }
    mfma_block<BITS, GQ, LG, true>(smem_raw, dm, kw_, vw_, qg, slab, b, tw0, nw, k0.rank, v0.rank, rank_cap, odd_rank != 0, item < 0,
                                   nullptr, 0, nwaves, ncw, item);
  }
  block_lds_sync();
  const MfmaMisc<GQ, SINGLE_WAVES<GQ>>& M = *reinterpret_cast<const MfmaMisc<GQ, SINGLE_WAVES<GQ>>*>(smem_raw + L.misc);
  for (int i = threadIdx.x; i < GQ * D; i += nthreads) {
    const int c = i / GQ, hq = i % GQ;   // the lanes of a wave read consecutive plane entries
    float Mx = -INFINITY;
#pragma unroll
    for (int w = 0; w < SINGLE_WAVES<GQ>; ++w)
      if (w < nwaves) Mx = fmaxf(Mx, M.wstat[w][hq][0]);
    float o = 0.0f, l = 0.0f;
#pragma unroll 4
    for (int w = 0; w < nwaves; ++w) {
      const float2 st = *reinterpret_cast<const float2*>(&M.wstat[w][hq][0]);
      const float f = st.x == -INFINITY ? 0.0f : __expf(st.x - Mx);   // a wave none of whose rows the column sees
      o += f * reinterpret_cast<const float*>(smem_raw + L.wave0 + (size_t)w * L.wave_stride + L.osp)[i];
      l += f * st.y;
    }
    out[((size_t)row0 + hq) * D + c] = (uint16_t)f2h(o / l);
  }
}

// grid (B*H_q), block 128: thread c merges channel c of the row's nrec records, AT_ONCE (16, 32 or 64) records per round.
// Lane s of every wave fetches (m, l) of record s, so the weights of a round's records come from one
// round of loads, and the thread's channel of all of them is requested along with it: the kernel is one load latency and a short
// chain, which registers alone exchange lanes in.  Eight records at a time behind the weights, with shuffles through LDS, a read took a
// microsecond more (16 x 32 heads x 4096 tokens, 11 records, 58.2 -> 57.2 us, 32 x 32768, 66 records, 33.9 -> 33.0, 40 slabs x 3001 23.9 -> 23.5).
// Records past the last read as 0 through the buffer view.
template <int AT_ONCE>
__global__ __launch_bounds__(128) void decode_combine_kernel(const float* __restrict__ partial, int nrec,
                                                             uint16_t* __restrict__ out) {
  const int row = blockIdx.x, c = threadIdx.x, lane = threadIdx.x & 63;
  const GEAR_BUF_T rb = GEAR_BUF_MAKE(partial + (size_t)row * nrec * DECODE_REC, nrec * (DECODE_REC * 4));
  float M = -INFINITY, L = 0.0f, o = 0.0f;
  for (int s0 = 0; s0 < nrec; s0 += AT_ONCE) {
    const int cnt = nrec - s0 < AT_ONCE ? nrec - s0 : AT_ONCE;
    const uint2 ml = GEAR_BUF_LOAD8(rb, (s0 + lane) * (DECODE_REC * 4));
    float v[AT_ONCE];
#pragma unroll
    for (int b = 0; b < AT_ONCE; b += 8) {
      if (b < cnt) {   // block-uniform
#pragma unroll
        for (int u = 0; u < 8; ++u) v[b + u] = __uint_as_float(GEAR_BUF_LOAD4(rb, ((s0 + b + u) * DECODE_REC + 2 + c) * 4));
      } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) v[b + u] = 0.0f;
      }
    }
    const float m = lane < cnt ? __uint_as_float(ml.x) : -INFINITY;
    const float l = lane < cnt ? __uint_as_float(ml.y) : 0.0f;
    const float Mn = fmaxf(wave_max(m), M);
    if (Mn == -INFINITY) continue;                      // nothing but empty records so far
    const float f = (m == -INFINITY) ? 0.0f : __expf(m - Mn);
    const float keep = (M == -INFINITY) ? 0.0f : __expf(M - Mn);
    L = L * keep + wave_sum(l * f);
    o *= keep;
    M = Mn;
#pragma unroll
    for (int b = 0; b < AT_ONCE; b += 8) {
      if (b < cnt) {
#pragma unroll
        for (int u = 0; u < 8; ++u) o += v[b + u] * lane_bcast(f, b + u);
      }
    }
  }
  out[(size_t)row * D + c] = (uint16_t)f2h(o / L);
}

constexpr int CUS = GEAR_CUS;

// Whether a read goes through the single-launch kernel, if its LDS fits: `slabs` blocks of nwaves waves, against slabs * nblocks blocks of four
// waves and the merge's launch.  The second launch is 3 to 4 us; what the single block costs is that all its waves share one CU's
// vector issue, which a small batch spreads over several.  So the line is drawn at the waves the fullest CU gets beyond the other
// kernel's, times what a wave issues (850 vector instructions at one column, 1750 at four).  Measured, split and merge -> single:
//   32 slabs, 1 column, 512 tokens + 1 chunk 13.5 -> 10.7 us, 900 + 2 13.7 -> 11.0 (4 bits 13.3 -> 12.2), 1400 + 2 13.2 -> 14.5
//   16 slabs, 2 columns, 512 + 5 chunks 13.4 -> 12.3 (4 bits 13.9 -> 13.6), 1400 + 2 13.3 -> 15.6
//   8 slabs, 4 columns, 512 + 1 15.7 -> 14.4, 512 + 5 15.3 -> 16.9; at 256 slabs 30.5 -> 18.3; 8 columns, 512 + 1: equal
// With more than 12 waves a CU holds one block, and its end is not covered by another: it has to have nearly no more waves than
// the other kernel's CU, and few rounds of blocks (1024 slabs, 1400 + 2 tokens: 41.6 -> 49.6; 512 slabs 27.4 -> 27.2).
// Beyond 1024 slabs the split kernel's whole blocks of prefill rows are as good (2048 slabs, 4 bits, 512 + 1: 50.1 -> 52.0), but
// not its nearly empty ones (100 tokens: 39.9 -> 16.8).
static bool single_read(int nwaves, int max_waves, int slabs, int nblocks, int columns) {
  if (nwaves > max_waves || nwaves > GEAR_SINGLE_WAVES) return false;
  if (slabs > 4 * CUS) return nwaves <= 4;
  const int here = nwaves * ((slabs + CUS - 1) / CUS), split = 4 * ((slabs * nblocks + CUS - 1) / CUS);
  if (nwaves > 12 && (slabs > 2 * CUS || here > split + 2)) return false;
  return here - split <= (columns == 1 ? 7 : columns == 2 ? 5 : columns == 4 ? 3 : 1);
}

// What a read consists of, as the choice of its launch sees it.
struct ReadShape {
  int bits, g, columns, slabs;     // columns: query columns of a slab
  int npw, ncw, nbw, nblocks;      // waves of the single-launch read (prefill rows, chunk pieces, buffer rows); blocks of four of the other
  int pp, rk0, rv0, rc, odd_rank;  // pieces per chunk; ranks of the prefill segment, largest rank of a chunk; a rank whose rows are not one read
  int waves() const { return npw + ncw + nbw; }
};
static ReadShape read_shape(const Dims& dm, const SegView& k0, const SegView& v0, const ChunkSet& cs, int n_buf, int n_buf_cap) {
  ReadShape s;
  s.bits = dm.bits;
  s.g = dm.g;
  s.columns = dm.Hq / dm.H;
  s.slabs = dm.B * dm.H;
  s.pp = n_buf_cap > WTOK ? 2 : 1;
  s.npw = (k0.n + WTOK - 1) / WTOK;
  s.ncw = cs.n_chunks * s.pp;
  s.nbw = (n_buf + BUF_WAVE_ROWS - 1) / BUF_WAVE_ROWS;
  s.nblocks = (k0.n + MFMA_TS - 1) / MFMA_TS + (s.ncw + 3) / 4 + 1;
  s.rk0 = k0.rank;
  s.rv0 = v0.rank;
  s.rc = 0;
  // a rank whose rows are not one 4-, 8- or 16-byte read anywhere in the launch
  auto one_read = [](int r) { return r == 0 || r == 2 || r == 4 || r == 8; };
  s.odd_rank = !one_read(k0.rank) || !one_read(v0.rank);
  for (int j = 0; j < cs.n_chunks; ++j) {
    s.rc = cs.rank[j] > s.rc ? cs.rank[j] : s.rc;
    s.odd_rank = s.odd_rank || !one_read(cs.rank[j]);
  }
  return s;
}
template <int GQ>
static size_t single_lds(const ReadShape& s) {
  return (size_t)mfma_layout<GQ>(s.bits, s.g, s.rk0, s.rv0, s.rc, s.odd_rank != 0, s.waves(), s.ncw).total;
}

// How a read is launched: 2^lparts blocks share a slab's query columns, in one launch (single) or by the split kernel and the merge.
struct ReadPlan {
  int lparts;
  bool single;
  size_t lds;   // of the single launch
};
// Fewer columns per wave make the wave's chain of steps shorter and the codes are unpacked once per part, so a small grid is read
// faster by more parts and a large one by fewer.  The times are a model of measured ones, in microseconds: a lone block on a CU
// takes `first`, each further one adds `more` (beyond three blocks of eight columns, which is what a CU holds, a quarter as much
// again); a single-launch read takes `base` and `wave` for each wave of the fullest CU, `least` at the least.  Whole -> parts:
// 5 x 8 heads x 3001 tokens, eight columns 29.9 -> 24.1 us (2 parts); 1 x 8 heads x 3001 21.5 -> 12.4 (4); 16 x 8 heads x 8192 97.7
// -> 90.9 (2); four columns, 1 x 8 heads x 8192 16.2 -> 15.0 (2), 64 x 8 heads x 1700 61.7 against 67.4 (whole).  A part has to
// promise 4 % a step.  The constants are those of rank 4 and 2 % outliers: a read without them is up to a third shorter, one with
// 5 % twice as long, for all choices nearly alike.  Over 1237 sizes drawn at random (1 to 64 batch elements, 60 to 20000 tokens, up to
// 20 chunks, one to eight columns, ranks 0 to 8, at most 5 % outliers; profiles/decode_routes.csv) the choice takes 0.72 of the time of
// whole slabs by the split kernel, geometric mean, and the best one of each size would take 0.67.  26 of them are more than 3 % slower
// than that kernel, at worst 1.24 (44 slabs x 1606 tokens, eight columns, rank 8, 155 buffer rows: 27.5 -> 34.1, the parts' buffer
// blocks one after another); a larger margin loses more on the other sizes than it wins on these.
static ReadPlan read_plan(const ReadShape& s) {
  struct Cost { float first, more, least, base, wave; };
  static const Cost costs[2][4] = {   // one, two, four, eight columns
      {{11.8f, 1.9f, 10.0f, 3.0f, 0.75f}, {12.0f, 3.1f, 10.0f, 4.0f, 1.0f}, {15.6f, 4.75f, 12.0f, 3.0f, 1.7f}, {22.0f, 8.3f, 17.0f, 0.0f, 3.6f}},
      {{12.3f, 2.5f, 10.0f, 2.0f, 1.05f}, {13.6f, 4.3f, 10.5f, 3.0f, 1.4f}, {17.8f, 5.8f, 14.0f, 3.0f, 2.1f}, {25.8f, 10.0f, 21.0f, 0.0f, 4.3f}}};
  float best = 0.0f;
  ReadPlan plan{0, false, 0};
  for (int p = 0; (s.columns >> p) > 0; ++p) {
    const int c = s.columns >> p, lc = c == 8 ? 3 : c >> 1;
    const long long blocks = (long long)s.slabs << p;
    if (p > 0 && blocks > 65535) break;   // a dimension of the grid
    const Cost& t = costs[s.bits == 4 ? 1 : 0][lc];
    bool single = single_read(s.waves(), c == 8 ? SINGLE_WAVES<8> : SINGLE_WAVES<1>, (int)blocks, s.nblocks, c);
    size_t lds = 0;
    if (single) {
      lds = c == 8 ? single_lds<8>(s) : c == 4 ? single_lds<4>(s) : c == 2 ? single_lds<2>(s) : single_lds<1>(s);
      single = lds <= LDS_PER_CU;
    }
    float us;
    if (single) {
      us = t.base + t.wave * (float)(s.waves() * ((blocks + CUS - 1) / CUS));
      us = us < t.least ? t.least : us;
    } else {
      const long long k = (blocks * s.nblocks + CUS - 1) / CUS;
      us = t.first + t.more * (float)(k - 1) + (c == 8 && k > 3 ? 0.25f * t.more * (float)(k - 3) : 0.0f);
      if (c == 8 && (s.odd_rank || (s.g == 32 && s.rk0 > 4))) us *= 1.1f;   // (factor rows through LDS; four groups of factors)
    }
    us *= 1.0f + 0.04f * (float)p;
    if (p == 0 || us < best) {
      best = us;
      plan = ReadPlan{p, single, lds};
    }
  }
  return plan;
}

template <int BITS, int GQ, int LG>
static hipError_t launch_decode_t(const Dims& dm, const SegView& k0, const SegView& v0, const ChunkSet& cs, const ReadShape& s,
                                  const ReadPlan& plan, const uint16_t* q, const uint16_t* Kbuf, const uint16_t* Vbuf, int n_buf,
                                  int n_buf_cap, int q_len, int causal, uint16_t* out, float* partial, hipStream_t st) {
  const int blocks = s.slabs << plan.lparts;          // per 512 tokens: a block for each slab and part of its columns
  if (plan.single) {
    static std::atomic<uint64_t> lds_raised{0};
    const hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(decode_single_kernel<BITS, GQ, LG>), lds_raised, plan.lds, LDS_PER_CU);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((decode_single_kernel<BITS, GQ, LG>), dim3(blocks), dim3(64 * s.waves()), plan.lds, st, dm, k0, v0, cs, q,
                       Kbuf, Vbuf, n_buf, n_buf_cap, s.npw, s.ncw, s.pp, s.rc, s.odd_rank, q_len, causal, plan.lparts, out);
    return hipGetLastError();
  }
  size_t lds = (size_t)mfma_layout<GQ>(BITS, dm.g, k0.rank, v0.rank, s.rc, s.odd_rank != 0).total;
  if (lds < sizeof(TailSmem<GQ>)) lds = sizeof(TailSmem<GQ>);
  static std::atomic<uint64_t> lds_raised{0};
  const hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(decode_split_kernel<BITS, GQ, LG>), lds_raised, lds, LDS_PER_CU);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((decode_split_kernel<BITS, GQ, LG>), dim3(s.nblocks, blocks), dim3(256), lds, st, dm, k0, v0, cs, q, Kbuf, Vbuf,
                     n_buf, n_buf_cap, (k0.n + MFMA_TS - 1) / MFMA_TS, s.pp, s.rc, s.odd_rank, q_len, causal, plan.lparts, partial);
  const dim3 rows(dm.B * dm.Hq);
  if (s.nblocks > GEAR_MERGE_32) hipLaunchKernelGGL(decode_combine_kernel<64>, rows, dim3(128), 0, st, (const float*)partial, s.nblocks, out);
  else if (s.nblocks > GEAR_MERGE_16) hipLaunchKernelGGL(decode_combine_kernel<32>, rows, dim3(128), 0, st, (const float*)partial, s.nblocks, out);
  else hipLaunchKernelGGL(decode_combine_kernel<16>, rows, dim3(128), 0, st, (const float*)partial, s.nblocks, out);
  return hipGetLastError();
}

template <int BITS>
static hipError_t launch_decode_b(const Dims& dm, const SegView& k0, const SegView& v0, const ChunkSet& cs,
                                  const uint16_t* q, const uint16_t* Kbuf, const uint16_t* Vbuf, int n_buf,
                                  int n_buf_cap, int rank_cap, int q_len, int causal, uint16_t* out, float* partial,
                                  hipStream_t st) {
  const ReadShape s = read_shape(dm, k0, v0, cs, n_buf, n_buf_cap);
  if (s.rc > rank_cap) return hipErrorInvalidValue;   // the cache never stores more than its configured rank
  const ReadPlan plan = read_plan(s);
#define GEAR_DECODE_CASE(GQV)                                                                                          \
  case GQV:                                                                                                            \
    if (dm.g == 32) return launch_decode_t<BITS, GQV, 5>(dm, k0, v0, cs, s, plan, q, Kbuf, Vbuf, n_buf, n_buf_cap, q_len, causal, out, partial, st); \
    if (dm.g == 64) return launch_decode_t<BITS, GQV, 6>(dm, k0, v0, cs, s, plan, q, Kbuf, Vbuf, n_buf, n_buf_cap, q_len, causal, out, partial, st); \
    return launch_decode_t<BITS, GQV, 7>(dm, k0, v0, cs, s, plan, q, Kbuf, Vbuf, n_buf, n_buf_cap, q_len, causal, out, partial, st);
  switch (s.columns >> plan.lparts) {
    GEAR_DECODE_CASE(1)
    GEAR_DECODE_CASE(2)
    GEAR_DECODE_CASE(4)
    GEAR_DECODE_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef GEAR_DECODE_CASE
}

// q_len query rows per query head ([B, H_q, q_len, 128]): the rows of the query heads of one KV head lie
// next to each other, so they are run as (H_q / H) * q_len query columns of that KV head.
hipError_t launch_decode(const Dims& dm_in, const SegView& k0, const SegView& v0, const ChunkSet& cs,
                         const uint16_t* q, const uint16_t* Kbuf, const uint16_t* Vbuf, int n_buf,
                         int n_buf_cap, int rank_cap, int q_len, int causal, uint16_t* out, float* partial,
                         hipStream_t st) {
  Dims dm = dm_in;
  dm.Hq = dm_in.Hq * q_len;
  if (dm.bits == 2)
    return launch_decode_b<2>(dm, k0, v0, cs, q, Kbuf, Vbuf, n_buf, n_buf_cap, rank_cap, q_len, causal, out, partial, st);
  return launch_decode_b<4>(dm, k0, v0, cs, q, Kbuf, Vbuf, n_buf, n_buf_cap, rank_cap, q_len, causal, out, partial, st);
}

}  // namespace gear
