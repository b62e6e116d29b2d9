// Attention over the fp16 streaming buffer (the rows not yet compressed, Algorithm 1)
// for one (b, h_kv): a plain-ALU block, one thread per buffer row for the scores, one
// thread per (channel, row parity) for the Value side.  Appended chunk segments do not
// come here: they go through the matrix-core block like the prefill.
#pragma once
#include "gear_internal.h"
#include "gear_launch.h"
#include "decode_mfma.h"

namespace gear {

constexpr int TAIL_ROWS = 256;   // >= the largest buffer (n_buf_cap <= 255)

template <int GQ>
struct TailSmem {
  float q[GQ][D];
  float sc[GQ][TAIL_ROWS];
  float o_half[2][GQ][D];
  float red[GQ][4];
  float stat[GQ][2];   // m, l
};

// View of chunk j: the chunk regions lie `stride` bytes apart and share one layout.
__device__ __forceinline__ SegView chunk_view(const SegView& base, uint64_t stride, int j, int n, int rank) {
  SegView v = base;
  const size_t off = (size_t)stride * j;
  v.codes = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(base.codes) + off);
  v.sz = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(base.sz) + off);
  v.A = reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(base.A) + off);
  v.Bf = reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(base.Bf) + off);
  v.ell = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(base.ell) + off);
  v.sp_table = reinterpret_cast<uint2*>(reinterpret_cast<char*>(base.sp_table) + off);
  v.sp_pool = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(base.sp_pool) + off);
  v.n = n;
  v.rank = rank;
  return v;
}

// Kb, Vb: the slab's buffer rows [n_buf][128] fp16.  Writes the record (m, l, o[128]) of each of
// the GQ query columns; m = -inf, l = 0 when a column sees no buffer row.  A column is one query
// row of one query head: column hq holds query row hq % q_len, and with `causal` that query sees
// the buffer rows 0 .. n_buf - q_len + hq % q_len only (the q_len newest tokens are the buffer's
// last q_len rows); q_len = 1: the single-query read, every column sees all n_buf rows.
template <int GQ>
__device__ __forceinline__ void buffer_block(TailSmem<GQ>& S, const uint16_t* __restrict__ qg, const uint16_t* __restrict__ Kb,
                             const uint16_t* __restrict__ Vb, int n_buf, int q_len, int causal, int row0,
                             float* __restrict__ rec_base, int rec_stride) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const float scale = 0.08838834764831845f;  // 1/sqrt(128)
  // Scores: thread (row16 = tid / 16, piece = tid % 16) takes the 16-byte piece (8 channels) of rows
  // row16, row16 + 16, ...; the 16 lanes of a row add their partial dot products.  The loads that do not
  // depend on the scores are requested before anything waits: q, the pieces of the first two rows, and
  // the first eight Value rows of the thread's (channel, parity) on the Value side.
  const int row16 = tid >> 4, piece = tid & 15;
  auto load_piece = [&](int row) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (row < n_buf) v = reinterpret_cast<const uint4*>(Kb + (size_t)row * D)[piece];
    return v;
  };
  const uint4 kp0 = load_piece(row16), kp1 = load_piece(row16 + 16);
  const int vc = tid & 127, vhalf = tid >> 7;
  uint32_t vr0[4];   // two fp16 values per word
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int k = vhalf + 4 * u;
    uint32_t a = 0, b = 0;
    if (k < n_buf) a = Vb[(size_t)k * D + vc];
    if (k + 2 < n_buf) b = Vb[(size_t)(k + 2) * D + vc];
    vr0[u] = a | (b << 16);
  }
  for (int i = tid; i < GQ * D; i += 256) S.q[i / D][i % D] = h2f(qg[i]);
  block_lds_sync();
  auto row_scores = [&](const uint4& kv, int row) {   // raw scores of `row` into S.sc
    const uint32_t w[4] = {kv.x, kv.y, kv.z, kv.w};
    float kf[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) kf[e] = h2f((w[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu);
#pragma unroll
    for (int hq = 0; hq < GQ; ++hq) {
      const float4 a = *reinterpret_cast<const float4*>(&S.q[hq][piece * 8]);   // q of the thread's 8 channels
      const float4 b = *reinterpret_cast<const float4*>(&S.q[hq][piece * 8 + 4]);
      float p = a.x * kf[0] + a.y * kf[1] + a.z * kf[2] + a.w * kf[3] + b.x * kf[4] + b.y * kf[5] + b.z * kf[6] + b.w * kf[7];
      p = row16_sum(p);
      if (piece == 0 && row < n_buf) S.sc[hq][row] = p;
    }
  };
  row_scores(kp0, row16);
  row_scores(kp1, row16 + 16);
  for (int r0 = 32; r0 < n_buf; r0 += 16) row_scores(load_piece(r0 + row16), r0 + row16);
  block_lds_sync();
  float s[GQ];
#pragma unroll
  for (int hq = 0; hq < GQ; ++hq) s[hq] = tid < n_buf ? S.sc[hq][tid] : 0.0f;
  // ---- softmax over the buffer rows
  float p[GQ];
#pragma unroll
  for (int hq = 0; hq < GQ; ++hq) {
    const int seen = causal ? n_buf - q_len + 1 + ((row0 + hq) & (q_len - 1)) : n_buf;   // q_len is a power of two
    s[hq] = tid < seen ? s[hq] * scale : -INFINITY;
    const float mx = wave_max(s[hq]);
    if (lane == 0) S.red[hq][wave] = mx;
  }
  block_lds_sync();
#pragma unroll
  for (int hq = 0; hq < GQ; ++hq) {
    const float m = fmaxf(fmaxf(S.red[hq][0], S.red[hq][1]), fmaxf(S.red[hq][2], S.red[hq][3]));
    p[hq] = s[hq] > -INFINITY ? __expf(s[hq] - m) : 0.0f;
    S.sc[hq][tid] = p[hq];
    if (tid == 0) S.stat[hq][0] = m;
  }
  block_lds_sync();
#pragma unroll
  for (int hq = 0; hq < GQ; ++hq) {
    const float sum = wave_sum(p[hq]);
    if (lane == 0) S.red[hq][wave] = sum;
  }
  // ---- Value side: thread (channel c, parity) walks rows parity, parity + 2, ...; 8 rows in flight
  // (the first eight were requested at the start)
  {
    const int c = vc, half = vhalf;
    float o[GQ];
#pragma unroll
    for (int hq = 0; hq < GQ; ++hq) o[hq] = 0.0f;
    for (int k0 = half; k0 < n_buf; k0 += 16) {
      uint16_t vr[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int k = k0 + 2 * u;
        vr[u] = 0;
        if (k0 == half) vr[u] = (uint16_t)(vr0[u >> 1] >> ((u & 1) * 16));
        else if (k < n_buf) vr[u] = Vb[(size_t)k * D + c];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int k = k0 + 2 * u;
        if (k < n_buf) {
          const float v = h2f(vr[u]);
#pragma unroll
          for (int hq = 0; hq < GQ; ++hq) o[hq] += S.sc[hq][k] * v;
        }
      }
    }
#pragma unroll
    for (int hq = 0; hq < GQ; ++hq) S.o_half[half][hq][c] = o[hq];
  }
  block_lds_sync();
  for (int i = tid; i < GQ * D; i += 256) {
    const int hq = i / D, c = i % D;
    float* rec = rec_base + (size_t)hq * rec_stride;
    rec[2 + c] = S.o_half[0][hq][c] + S.o_half[1][hq][c];
    if (c == 0) {
      rec[0] = S.stat[hq][0];
      rec[1] = S.red[hq][0] + S.red[hq][1] + S.red[hq][2] + S.red[hq][3];
    }
  }
}

// One wave of the single-launch read: buffer rows [r0, r0 + BUF_WAVE_ROWS), everything it reads requested before it waits.
// Leaves the state like mfma_block<SINGLE>: the output plane in the wave's LDS region, (m, l) in wstat.  Joins the block's one
// barrier in front of the merge's (q in LDS), as every other wave does.
constexpr int BUF_WAVE_ROWS = 32;
template <int GQ>
__device__ __forceinline__ void buffer_wave(unsigned char* smem, const MfmaLayout& L, const uint16_t* __restrict__ qg,
                                            const uint16_t* __restrict__ Kb, const uint16_t* __restrict__ Vb, int n_buf, int r0,
                                            int q_len, int causal, int row0, int wave, int nthreads) {
  const int tid = threadIdx.x, lane = tid & 63, row4 = lane >> 4, piece = lane & 15;
  float* Sq = reinterpret_cast<float*>(smem + L.q);                 // [128][GQ]
  MfmaMisc<GQ, SINGLE_WAVES<GQ>>& M = *reinterpret_cast<MfmaMisc<GQ, SINGLE_WAVES<GQ>>*>(smem + L.misc);
  unsigned char* wbase = smem + L.wave0 + (size_t)wave * L.wave_stride;
  float* Ssc = reinterpret_cast<float*>(wbase + L.sc);              // [32][GQ]
  float* Sosp = reinterpret_cast<float*>(wbase + L.osp);            // [128][GQ]
  const float scale = 0.08838834764831845f;  // 1/sqrt(128)
  uint32_t qreg[GQ];
#pragma unroll
  for (int k = 0; k < GQ; ++k) {   // the block's waves share the staging of q
    const int i = tid + nthreads * k;
    qreg[k] = 0u;
    if (i < GQ * D / 2) qreg[k] = reinterpret_cast<const uint32_t*>(qg)[i];
  }
  // Keys: the 16 lanes of a row take a 16-byte piece each, four rows per request.  Values: the lane takes channels 2 lane and
  // 2 lane + 1 of every row.  Rows past the buffer's last read as 0.
  const int rows = n_buf - r0 < BUF_WAVE_ROWS ? n_buf - r0 : BUF_WAVE_ROWS;
  const GEAR_BUF_T kview = GEAR_BUF_MAKE(Kb + (size_t)r0 * D, rows * D * 2), vview = GEAR_BUF_MAKE(Vb + (size_t)r0 * D, rows * D * 2);
  uint4 kv[BUF_WAVE_ROWS / 4];
  uint32_t vv[BUF_WAVE_ROWS];
#pragma unroll
  for (int i = 0; i < BUF_WAVE_ROWS / 4; ++i) kv[i] = GEAR_BUF_LOAD16(kview, (4 * i + row4) * (D * 2) + piece * 16);
#pragma unroll
  for (int k = 0; k < BUF_WAVE_ROWS; ++k) vv[k] = GEAR_BUF_LOAD4(vview, k * (D * 2) + lane * 4);
#pragma unroll
  for (int k = 0; k < GQ; ++k) {
    const int i = tid + nthreads * k;
    if (i < GQ * D / 2) {   // channels c, c + 1 of query column hq
      const int hq = i / (D / 2), c = 2 * (i % (D / 2));
      Sq[c * GQ + hq] = h2f(qreg[k] & 0xFFFFu);
      Sq[(c + 1) * GQ + hq] = h2f(qreg[k] >> 16);
    }
  }
  block_lds_sync();
  float qf[8 * GQ];   // [channel of the piece][column]
#pragma unroll
  for (int i = 0; i < 8 * GQ; i += 4) {
    const float4 t = *reinterpret_cast<const float4*>(Sq + piece * 8 * GQ + i);
    qf[i] = t.x; qf[i + 1] = t.y; qf[i + 2] = t.z; qf[i + 3] = t.w;
  }
#pragma unroll
  for (int i = 0; i < BUF_WAVE_ROWS / 4; ++i) {
    const uint32_t w[4] = {kv[i].x, kv[i].y, kv[i].z, kv[i].w};
    float p[GQ];
#pragma unroll
    for (int hq = 0; hq < GQ; ++hq) p[hq] = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float kf = h2f((w[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu);
#pragma unroll
      for (int hq = 0; hq < GQ; ++hq) p[hq] += qf[e * GQ + hq] * kf;
    }
#pragma unroll
    for (int hq = 0; hq < GQ; ++hq) p[hq] = row16_sum(p[hq]);
    if (piece == 0) lds_store_f<GQ>(Ssc + (4 * i + row4) * GQ, p);
  }
  wave_lds_sync();
  // softmax over the wave's rows: lane = row
  float s[GQ];
#pragma unroll
  for (int hq = 0; hq < GQ; ++hq) s[hq] = 0.0f;
  if (lane < BUF_WAVE_ROWS) lds_load_f<GQ>(Ssc + lane * GQ, s);
#pragma unroll
  for (int hq = 0; hq < GQ; ++hq) {
    const int seen = causal ? n_buf - q_len + 1 + ((row0 + hq) & (q_len - 1)) : n_buf;   // q_len is a power of two
    const float v = lane < BUF_WAVE_ROWS && r0 + lane < seen ? s[hq] * scale : -INFINITY;
    const float m = wave_max(v);
    s[hq] = __expf(v - (m == -INFINITY ? 0.0f : m));   // (a score of -inf, like a row that is not seen, weighs nothing)
    const float l = wave_sum(s[hq]);
    if (lane == 0) {
      M.wstat[wave][hq][0] = m;   // -inf when the column sees none of the wave's rows
      M.wstat[wave][hq][1] = l;
    }
  }
  if (lane < BUF_WAVE_ROWS) lds_store_f<GQ>(Ssc + lane * GQ, s);
  wave_lds_sync();
  float o0[GQ], o1[GQ];
#pragma unroll
  for (int hq = 0; hq < GQ; ++hq) o0[hq] = o1[hq] = 0.0f;
#pragma unroll
  for (int k = 0; k < BUF_WAVE_ROWS; ++k) {
    const float a = h2f(vv[k] & 0xFFFFu), b = h2f(vv[k] >> 16);
    float p[GQ];
    lds_load_f<GQ>(Ssc + k * GQ, p);
#pragma unroll
    for (int hq = 0; hq < GQ; ++hq) {
      o0[hq] += p[hq] * a;
      o1[hq] += p[hq] * b;
    }
  }
  lds_store_f<GQ>(Sosp + 2 * lane * GQ, o0);
  lds_store_f<GQ>(Sosp + (2 * lane + 1) * GQ, o1);
}

}  // namespace gear
