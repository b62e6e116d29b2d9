// SVDSolver_r (Eq. 6, Algorithm 2): batched power iteration on the per-head
// residual R = X - D - S.  No copy of R exists: every pass re-derives R = (Y - zero) - code * scale, Y = X - S, from
// X and the mask of S (or, in the solvers of short segments and of a single round, from a copy of Y in the workspace)
// and the stored scale (Keys: with the stored codes; Values: with the code recomputed by the quantizer's own operation
// sequence).  That is exact, and a 16-bit copy of R itself flips enough fp16 roundings of the stored factors to fail
// the attention tolerance.
//
//   (the quantization kernel leaves G = R^T R, 128 x 128 per slab, as partial sums: compress_quant.h.  Every round of
//   Algorithm 2 before the last maps B -> R^T (R B) = G B, so those rounds need no pass over R of their own: they become
//   128 x 128 x r products on G.)
//   pi_solve   : B <- G^(L-1) B0 (columns rescaled between the products: the span,
//                hence A B^T, is unchanged), then the QR of B that opens the last round.
//                With L > 1 the last round comes out of G as well: for A = R Q (Q = that
//                orthonormal B), A^T A = Q^T G Q gives the r x r factor C with orth(A) = A C,
//                and the final B = R^T orth(A) = G Q C; the kernel writes B (fp16) and W = Q C.
//   pi_project : A = R W per token, rounded to fp16: the one pass over R of the last round.
//   (L = 1 has no Gram pass; its single round runs as sweep + update + finish below.)
//   pi_update  : B <- start matrix or sum of the sweep partials; column scaling
//                between rounds (the span, hence A B^T, is unchanged); QR of B
//                before the last round; after the last round the r x r factor
//                that orthonormalises A, and the final B = R^T orth(A).
//   pi_sweep   : one pass over a slab's residual: a_t = R_t B (per token), partial
//                B' = sum_t R_t^T a_t, and in the last round a_t itself and the
//                Gram matrix sum_t a_t a_t^T.
//   pi_finish  : A = a C  (C = the r x r factor), rounded to fp16.
//   pi_small   : all of the above for a segment of at most 256 tokens, in one block per slab.
//   pi_tiny    : a segment of at most 64 tokens (a flushed buffer): one block per slab with the residual in LDS.
#include <atomic>
#include "gear_internal.h"
#include "gear_launch.h"

namespace gear {

constexpr int PT = 256;  // tokens per sweep block

// Sum over the block (128 or 256 threads; the same value in every thread).
template <typename T>
__device__ __forceinline__ T block_sum(T v, T* red /* 4 */) {
  v = wave_sum_shfl(v);
  block_lds_sync();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  block_lds_sync();
  T s = red[0] + red[1];
  if (blockDim.x > 128) s += red[2] + red[3];
  return s;
}

// Sum of a double over the 64 lanes, in every lane: lane exchanges inside rows of 16 (one
// data-parallel-primitive move per 32-bit half), then the four row sums through scalar reads.
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = dpp_u<CTRL>((uint32_t)b), hi = dpp_u<CTRL>((uint32_t)(b >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double lane_bcast_d(double v, int lane) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum_d(double v) {
  v += dpp_d<DPP_XOR1>(v);
  v += dpp_d<DPP_XOR2>(v);
  v += dpp_d<DPP_HALF_MIRROR>(v);
  v += dpp_d<DPP_MIRROR>(v);
  return (lane_bcast_d(v, 0) + lane_bcast_d(v, 16)) + (lane_bcast_d(v, 32) + lane_bcast_d(v, 48));
}
// A double's lanes exchanged as GEAR_LANE_SWAP32 and GEAR_LANE_SWAP16 exchange a word's.
__device__ __forceinline__ uint64_t bits_of(double v) { return __builtin_bit_cast(uint64_t, v); }
__device__ __forceinline__ double double_of(uint32_t lo, uint32_t hi) { return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo); }
__device__ __forceinline__ void lane_swap32_d(double& a, double& b) {
  uint32_t al = (uint32_t)bits_of(a), ah = (uint32_t)(bits_of(a) >> 32), bl = (uint32_t)bits_of(b), bh = (uint32_t)(bits_of(b) >> 32);
  GEAR_LANE_SWAP32(al, bl);
  GEAR_LANE_SWAP32(ah, bh);
  a = double_of(al, ah);
  b = double_of(bl, bh);
}
__device__ __forceinline__ void lane_swap16_d(double& a, double& b) {
  uint32_t al = (uint32_t)bits_of(a), ah = (uint32_t)(bits_of(a) >> 32), bl = (uint32_t)bits_of(b), bh = (uint32_t)(bits_of(b) >> 32);
  GEAR_LANE_SWAP16(al, bl);
  GEAR_LANE_SWAP16(ah, bh);
  a = double_of(al, ah);
  b = double_of(bl, bh);
}
__device__ __forceinline__ double row16_sum_d(double v) {
  v += dpp_d<DPP_XOR1>(v);
  v += dpp_d<DPP_XOR2>(v);
  v += dpp_d<DPP_HALF_MIRROR>(v);
  return v + dpp_d<DPP_MIRROR>(v);
}
// The first `count` (a constant once unrolled) of N values, each summed over the 64 lanes, in every lane.  Four sums at a time: the halves and then
// the rows of the wave take one of them each (row r of lanes: value {0, 2, 1, 3}[r]), so that the four cost little more than one.
template <int N>
__device__ __forceinline__ void wave_sums_d(double (&v)[N], int count) {
#pragma unroll
  for (int i = 0; i < N; i += 4) {
    if (i >= count) continue;
    if (i + 1 == count) {
      v[i] = wave_sum_d(v[i]);
      continue;
    }
    double a = v[i], b = v[i + 1], c = i + 2 < count ? v[(i + 2) % N] : 0.0, d = i + 3 < count ? v[(i + 3) % N] : 0.0;
    lane_swap32_d(a, b);
    lane_swap32_d(c, d);
    double e = a + b, f = c + d;
    lane_swap16_d(e, f);
    const double t = row16_sum_d(e + f);
    v[i] = lane_bcast_d(t, 0);
    v[i + 1] = lane_bcast_d(t, 32);
    if (i + 2 < count) v[(i + 2) % N] = lane_bcast_d(t, 16);
    if (i + 3 < count) v[(i + 3) % N] = lane_bcast_d(t, 48);
  }
}
// 1 / sqrt(x) for x > 0 in double: the single-precision estimate, refined by two Newton steps
// (no double-precision square root or division, which are long instruction sequences)
__device__ __forceinline__ double rsqrt_d(double x) {
  // scaled into single-precision range by an even power of two taken from the exponent
  const int ex = (int)((__builtin_bit_cast(uint64_t, x) >> 52) & 0x7FF) - 1023;
  const int h = ex >> 1;                                   // x = m * 4^h, m in [1, 4)
  const double m = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, x) - ((uint64_t)(2 * h) << 52));
  double y = (double)__builtin_amdgcn_rsqf((float)m);
  y = y * (1.5 - 0.5 * m * y * y);
  y = y * (1.5 - 0.5 * m * y * y);
  return __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, y) - ((uint64_t)h << 52));   // y * 2^-h
}
// Gram-Schmidt (applied twice) in coefficient space: given the r x r Gram matrix G = A^T A of the columns of some A (G[i][j] for i <= j), finds
// C (upper triangular) with orth(A) = A C (column j of orth(A) is A * C[:, j]; dependent columns get C[:, j] = 0).  All of it in every lane's
// registers: some hundred multiply-adds, where a sum over lanes for each quadratic form, and its operands through LDS, took 7200 cycles at
// r = 4 and 30600 at r = 8.
// store(a, j, value): C[a][j] from the next column on.  IN_LDS: G and C lie there, and no entry is kept in
// a register from one pass to the next.
template <int R, bool IN_LDS, class Store>
__device__ __forceinline__ void coeff_orth(const double (&G)[R][R], const double (&C)[R][R], Store&& store) {
#pragma unroll
  for (int j = 0; j < R; ++j) {
    double v[R];   // entries 0 .. j; v[j] stays 1 until the end
#pragma unroll
    for (int a = 0; a < j; ++a) v[a] = 0.0;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      double h[R], dot[R];   // G v; q_k^T v = c_k^T G v, all projections of a pass from the same v
#pragma unroll
      for (int a = 0; a < j; ++a) {
        h[a] = G[a][j];
        if (pass > 0) {
#pragma unroll
          for (int b = 0; b < j; ++b) h[a] = __builtin_fma(a <= b ? G[a][b] : G[b][a], v[b], h[a]);
        }
      }
      if constexpr (IN_LDS) wave_lds_sync();
#pragma unroll
      for (int k = 0; k < j; ++k) {
        dot[k] = 0.0;
#pragma unroll
        for (int a = 0; a <= k; ++a) dot[k] = __builtin_fma(C[a][k], h[a], dot[k]);
      }
      if constexpr (IN_LDS) wave_lds_sync();
#pragma unroll
      for (int a = 0; a < j; ++a)
#pragma unroll
        for (int k = a; k < j; ++k) v[a] = __builtin_fma(-dot[k], C[a][k], v[a]);
      if constexpr (IN_LDS) wave_lds_sync();
    }
    double after2 = G[j][j];   // v^T G v
#pragma unroll
    for (int a = 0; a < j; ++a) {
      double h = 2.0 * G[a][j];
#pragma unroll
      for (int b = 0; b < j; ++b) h = __builtin_fma(a <= b ? G[a][b] : G[b][a], v[b], h);
      after2 = __builtin_fma(v[a], h, after2);
    }
    // (the Gram matrix is a sum of fp32 products: what is left of a dependent column is
    // rounding noise of relative size ~1e-7 in after2, so the cut sits above that)
    const bool ok = G[j][j] > 0.0 && after2 > 1e-6 * G[j][j];
    const double inv = ok ? rsqrt_d(after2) : 0.0;
#pragma unroll
    for (int a = 0; a < R; ++a) store(a, j, a < j ? (ok ? v[a] * inv : 0.0) : a == j ? inv : 0.0);
    if constexpr (IN_LDS) wave_lds_sync();
  }
}
// The same with G and C in LDS, by the threads of one wave (c: lane): kernels that hold more next to it.
template <int R>
__device__ __forceinline__ void coeff_orth_lds(const double (&G)[R][R], double (&C)[R][R], int c) {
  coeff_orth<R, true>(G, C, [&](int a, int j, double x) { if (c == 0) C[a][j] = x; });
}

// grid (B*H), block 256: thread c < 128 owns row c of the [128 x R] matrix.
// from_start          : B <- the start matrix (zero-padded to R)
// else                : B <- sum over `npart` partials ([slab][npart][128*R + R*R])
// do_orth : replace B by the Q factor of its QR (twice-applied modified
//           Gram-Schmidt, fp64; dependent columns become 0)
// final   : also sum the Gram partials, build C with orth(A) = A C, write
//           B_out = B C as fp16 into the arena and C into cmat.
template <int R>
struct UpdateSmem {
  double red[4];
  double G[R][R];
  double C[R][R];
};
// The body runs in a block of 256 threads: threads 128.. sum the Gram partials of the final round
// and otherwise only take part in the barriers.
template <int R>
__device__ __forceinline__ void pi_update_body(UpdateSmem<R>& sm, int slab, bool from_start, const StartB& sb, int rank,
                                               const float* __restrict__ partial, int npart, int do_orth,
                                               int final_round, float* __restrict__ Bcur, float* __restrict__ cmat,
                                               const SegView& sv) {
  double (&G)[R][R] = sm.G;
  double (&C)[R][R] = sm.C;
  double* red = sm.red;
  const int c = threadIdx.x;
  const bool act = c < D;
  double q[R];
#pragma unroll
  for (int r = 0; r < R; ++r) q[r] = 0.0;
  if (act) {
    if (from_start) {
#pragma unroll
      for (int r = 0; r < R; ++r) q[r] = r < rank ? (double)start_b(sb, slab, c, rank, r) : 0.0;
    } else {
      const float* p = partial + (size_t)slab * npart * (D * R + R * R);
      int i = 0;
      // long segments (many partials): the loads of eight partials are requested before the first is added
      // (written as a load loop of its own: an add right after its load makes the compiler wait for every load)
      if (npart > 16) {
        for (; i + 8 <= npart; i += 8) {
          float t[8][R];
#pragma unroll
          for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r) t[u][r] = __builtin_nontemporal_load(&p[(size_t)(i + u) * (D * R + R * R) + c * R + r]);
#pragma unroll
          for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r) q[r] += (double)t[u][r];
        }
      }
      for (; i < npart; ++i) {
#pragma unroll
        for (int r = 0; r < R; ++r) q[r] += (double)p[(size_t)i * (D * R + R * R) + c * R + r];
      }
    }
  }

  if (final_round) {
    if (c >= D && c < D + R * R) {   // threads 128..: the r x r Gram partials, while threads 0..127 sum theirs
      const int gi = c - D;
      const float* p = partial + (size_t)slab * npart * (D * R + R * R) + D * R + gi;
      double s = 0.0;
      int i = 0;
      for (; i + 8 <= npart; i += 8) {
        float t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = __builtin_nontemporal_load(&p[(size_t)(i + u) * (D * R + R * R)]);
#pragma unroll
        for (int u = 0; u < 8; ++u) s += (double)t[u];
      }
      for (; i < npart; ++i) s += (double)p[(size_t)i * (D * R + R * R)];
      G[gi / R][gi % R] = s;
    }
    block_lds_sync();
    if (c < 64) coeff_orth_lds<R>(G, C, c);
    block_lds_sync();
    double o[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      double s = 0.0;
#pragma unroll
      for (int r = 0; r < R; ++r) s += q[r] * C[r][j];
      o[j] = s;
    }
    if (act)
      for (int j = 0; j < rank; ++j) sv.Bf[((size_t)slab * D + c) * sv.rank + j] = (uint16_t)f2h((float)o[j]);
    if (c < R * R) cmat[(size_t)slab * R * R + c] = (float)C[c / R][c % R];
    return;
  }

  if (do_orth) {
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const double before2 = block_sum(q[j] * q[j], red);
      if (before2 == 0.0) { q[j] = 0.0; continue; }
      for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
          if (i < j) {
            const double dot = block_sum(q[i] * q[j], red);
            q[j] -= dot * q[i];
          }
        }
      }
      const double after2 = block_sum(q[j] * q[j], red);
      if (!(sqrt(after2) > 1e-12 * sqrt(before2))) q[j] = 0.0;
      else q[j] *= 1.0 / sqrt(after2);
    }
  } else {
    // keep magnitudes in range between rounds
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const double n2 = block_sum(q[j] * q[j], red);
      if (n2 > 0.0) q[j] *= 1.0 / sqrt(n2);
    }
  }
  if (act) {
#pragma unroll
    for (int r = 0; r < R; ++r) Bcur[((size_t)slab * D + c) * R + r] = (float)q[r];
  }
}

// The last round of a single-round call.
template <int R>
__global__ __launch_bounds__(256) void pi_update_kernel(const float* __restrict__ partial, int npart, float* __restrict__ Bcur,
                                                        float* __restrict__ cmat, SegView sv) {
  __shared__ UpdateSmem<R> sm;
  pi_update_body<R>(sm, blockIdx.x, false, StartB{nullptr, 0, 0}, sv.rank, partial, npart, 0, 1, Bcur, cmat, sv);
}

// grid (ceil(n/PT), B*H), block 256; thread (r0 = tid/16, oc = tid%16) owns
// channels 8*oc..+7 of rows pt*PT + r0 + 16*k.  Y = X - S in fp16 (what the quantization
// kernel left); the residual R = Y - D-hat = (Y - zero) - code * scale is re-derived per
// entry, so it is exact and costs 2 bytes per entry.  Keys take the code from the stored
// code rows (16 or 32 bits per row piece); Values, whose codes are stored in blocks of
// tokens, recompute it with the quantizer's own operation sequence.  The (zero, 1/scale,
// scale) of the block's groups are prepared once per block in LDS.
// B' += R_t^T a_t runs on the matrix cores: v_mfma_f32_4x4x1 works on 16 blocks of 4 lanes and
// adds, in register i of lane L, a(lane 4*(L/4) + i) * b(lane L).  With a = the lane's
// residual entry e and b = a_t[r = oc % 4], register i of accumulator e holds
// B'[channel 8*(4*(oc/4) + i) + e][r = oc % 4]: 8 instructions per token row instead of 32
// multiply-adds (the sweeps are bound by vector instruction issue, not by HBM).
// LAST: the final round, which also leaves a_t and the Gram matrix (its extra state costs
// one resident block per CU, so the rounds before it are compiled without).
template <bool IS_K, int R>
struct SweepSmem {
  float red[4][D * R];
  float redg[4][R * R];
  // Keys: [2][groups of the block <= 8][128] (zero, scale); Values: [rows][groups of a row <= 4] (zero, 1/scale, scale, -)
  __attribute__((aligned(16))) float prm[IS_K ? 2 * (PT / 32) * D : PT * 4 * 4];
};
// One block's share of a sweep: rows [pt * PT, pt * PT + PT) of slab `slab`, 256 threads.
template <bool IS_K, int R, bool LAST>
__device__ __forceinline__ void pi_sweep_body(SweepSmem<IS_K, R>& sm, int slab, int pt, const uint16_t* __restrict__ Y,
                                              const uint32_t* __restrict__ sv_sz, const uint32_t* __restrict__ sv_codes,
                                              int sv_n_cap, int sv_ng_cap, int g, int bits, int n, int t_lr,
                                              const float* __restrict__ Bcur, float* __restrict__ partial, int npart,
                                              float* __restrict__ Atmp) {
  float (&red)[4][D * R] = sm.red;
  float (&redg)[4][R * R] = sm.redg;
  float* prm = sm.prm;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int r0 = tid >> 4, oc = tid & 15;
  const uint16_t* Xs = Y + (size_t)slab * n * D;
  const int lg = 31 - __clz(g);   // g is a power of two
  constexpr int GSTR = (PT / 32) * D;   // Keys: floats per parameter plane
  const float qmax = (float)((1 << bits) - 1);
  const uint32_t* crow = sv_codes + (size_t)slab * sv_n_cap * (4 * bits);   // Keys: 128 * bits / 32 words per row

  constexpr int UN = 4;  // rows in flight per thread
  // the rows of an iteration, all requested before the first one is used
  // (buffer views of the slab's rows: a row past the end reads as 0)
  const GEAR_BUF_T xbuf = GEAR_BUF_MAKE(Xs, n * (D * 2));
  const GEAR_BUF_T cbuf = GEAR_BUF_MAKE(crow, IS_K ? n * (16 * bits) : 0);
  const int xoff0 = (pt * PT + r0) * (D * 2) + oc * 16;
  const int coff0 = (pt * PT + r0) * (16 * bits) + oc * (bits == 4 ? 4 : 2);
  auto request = [&](int k0, uint4 (&xv)[UN], uint32_t (&cw)[UN]) {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      xv[u] = GEAR_BUF_LOAD16_NT(xbuf, xoff0 + 16 * (k0 + u) * (D * 2));
      cw[u] = 0u;
      if (IS_K) {
        const int co = coff0 + 16 * (k0 + u) * (16 * bits);
        cw[u] = bits == 4 ? GEAR_BUF_LOAD4(cbuf, co) : GEAR_BUF_LOAD2(cbuf, co);
      }
    }
  };
  uint4 xv_first[UN];
  uint32_t cw_first[UN];   // Keys: the row piece's 8 codes
  request(0, xv_first, cw_first);   // in flight while the parameters are prepared

  if (IS_K) {
    const int ngb = (PT >> lg) > 0 ? (PT >> lg) : 1, grp0 = (pt * PT) >> lg, ng = (n + g - 1) >> lg;
    for (int i = tid; i < ngb * D; i += 256) {
      const int gi = grp0 + (i >> 7);
      GroupQ q;
      q.mn = 0.0f; q.inv = 0.0f; q.delta = 0.0f;
      if (gi < ng) q = load_group(sv_sz[((size_t)slab * sv_ng_cap + gi) * D + (i & 127)]);
      prm[i] = q.mn;
      prm[GSTR + i] = q.delta;
    }
  } else {
    const int ngl = 7 - lg;   // log2 of the groups per row
    for (int i = tid; i < (PT << ngl); i += 256) {
      const int t = pt * PT + (i >> ngl);
      GroupQ q;
      q.mn = 0.0f; q.inv = 0.0f; q.delta = 0.0f;
      if (t < n) q = load_group(sv_sz[(((size_t)slab * sv_n_cap + t) << ngl) + (i & ((1 << ngl) - 1))]);
      *reinterpret_cast<float4*>(&prm[4 * i]) = make_float4(q.mn, q.inv, q.delta, 0.0f);
    }
  }

  float bc[8][R];
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int r = 0; r < R; ++r) bc[e][r] = Bcur[((size_t)slab * D + oc * 8 + e) * R + r];

  constexpr int NB = (R + 3) / 4;   // column blocks of four
  floatx4 acc[8][NB];
  float gacc[R];
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[e][nb] = floatx4{0.f, 0.f, 0.f, 0.f};
  const bool partial_blk = pt * PT + PT > n;   // block-uniform: only such a block has rows past the end
#pragma unroll
  for (int r = 0; r < R; ++r) gacc[r] = 0.0f;
  block_lds_sync();

#pragma unroll   // no copies of the accumulators at a loop's back edge
  for (int k0 = 0; k0 < PT / 16; k0 += UN) {
    if (pt * PT + 16 * k0 >= n) break;  // block-uniform
    uint4 xv[UN];
    uint32_t cw[UN];
    if (k0 == 0) {
#pragma unroll
      for (int u = 0; u < UN; ++u) { xv[u] = xv_first[u]; cw[u] = cw_first[u]; }
    } else {
      request(k0, xv, cw);
    }
    float pmn[8], pdl[8];   // Keys: parameters of my 8 channels in the current group
    int gi_prev = -1;
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int tl = r0 + 16 * (k0 + u), t = pt * PT + tl;
      float vmn = 0.0f, vinv = 0.0f, vdl = 0.0f;   // Values: parameters of my row's channel group
      if (IS_K) {
        const int gi = (16 * (k0 + u)) >> lg;   // group inside the block, block-uniform
        if (gi != gi_prev) {
          const float* pb = &prm[gi * D + oc * 8];
          const float4 a0 = *reinterpret_cast<const float4*>(pb), a1 = *reinterpret_cast<const float4*>(pb + 4);
          const float4 c0 = *reinterpret_cast<const float4*>(pb + GSTR), c1 = *reinterpret_cast<const float4*>(pb + GSTR + 4);
          pmn[0] = a0.x; pmn[1] = a0.y; pmn[2] = a0.z; pmn[3] = a0.w; pmn[4] = a1.x; pmn[5] = a1.y; pmn[6] = a1.z; pmn[7] = a1.w;
          pdl[0] = c0.x; pdl[1] = c0.y; pdl[2] = c0.z; pdl[3] = c0.w; pdl[4] = c1.x; pdl[5] = c1.y; pdl[6] = c1.z; pdl[7] = c1.w;
          gi_prev = gi;
        }
      } else {
        const float4 pv = *reinterpret_cast<const float4*>(&prm[4 * ((tl << (7 - lg)) + ((oc * 8) >> lg))]);
        vmn = pv.x; vinv = pv.y; vdl = pv.z;
      }
      const uint32_t w[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w};
      float cf[8];   // Keys: the stored codes of my 8 channels as floats (one bit-field extract each)
      if (IS_K) {
#pragma unroll
        for (int e = 0; e < 8; ++e) cf[e] = (float)GEAR_UBFE(cw[u], e * bits, bits);
      }
      float res[8];
      float a[R];
#pragma unroll
      for (int r = 0; r < R; ++r) a[r] = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float y = h2f((e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xFFFFu));
        if (IS_K) {   // the stored code
          res[e] = __builtin_fmaf(-cf[e], pdl[e], y - pmn[e]);
        } else {      // the code the quantizer computed
          res[e] = quant_error(y, vmn, vinv, vdl, qmax);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) a[r] += res[e] * bc[e][r];
      }
      // the 16 lanes of a row hold one token: row sums of a[], delivered where the product
      // B' += R^T a wants them, a_t[4 * nb + oc % 4] in lane oc (0 past R)
      float bsel[NB];
      if constexpr (R == 2) {
        const float u = row16_sum2(a[0], a[1], lane);
        bsel[0] = (oc & 2) ? 0.0f : u;
      } else {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) bsel[nb] = row16_sum4(a[4 * nb], a[4 * nb + 1], a[4 * nb + 2], a[4 * nb + 3], lane);
      }
      // Keys: a row past the end has res = -zero-point, not 0; its a_t is dropped instead
      // (Values: the parameters of such rows are 0, so res is)
      // rows before t_lr take no part in the low-rank term (error reduction on the most recent tokens only)
      if ((IS_K && partial_blk && t >= n) || t < t_lr) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) bsel[nb] = 0.0f;
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e][nb] = __builtin_amdgcn_mfma_f32_4x4x1f32(res[e], bsel[nb], acc[e][nb], 0, 0, 0);
      }
      if (LAST) {
        // lane oc < R holds a_t[oc]
        const float mine = (NB > 1 && oc >= 4) ? bsel[NB - 1] : bsel[0];
        if (oc < R && t < n) Atmp[((size_t)slab * n + t) * R + oc] = mine;
        float ar[R];   // the whole a_t in every lane, from the four lanes of the quad
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const float src = bsel[r >> 2];
          ar[r] = (r & 3) == 0 ? dpp_f<0x00>(src) : (r & 3) == 1 ? dpp_f<0x55>(src) : (r & 3) == 2 ? dpp_f<0xAA>(src) : dpp_f<0xFF>(src);
        }
        if (oc < R) {
#pragma unroll
          for (int r = 0; r < R; ++r) gacc[r] += mine * ar[r];
        }
      }
    }
  }

  // reduce over the 16 row-threads that share a channel octet
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float v = acc[e][nb][i];
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        acc[e][nb][i] = v;
      }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    float v = gacc[r];
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    gacc[r] = v;
  }
  if (lane < 16) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 4 * nb + (oc & 3);
          if (r < R) red[wave][(8 * (4 * (oc >> 2) + i) + e) * R + r] = acc[e][nb][i];
        }
    if (oc < R) {
#pragma unroll
      for (int r = 0; r < R; ++r) redg[wave][oc * R + r] = gacc[r];
    }
  }
  block_lds_sync();
  float* out = partial + ((size_t)slab * npart + pt) * (D * R + R * R);
  for (int i = tid; i < D * R; i += 256) out[i] = red[0][i] + red[1][i] + red[2][i] + red[3][i];
  if (tid < R * R) out[D * R + tid] = LAST ? (redg[0][tid] + redg[1][tid] + redg[2][tid] + redg[3][tid]) : 0.0f;
}

template <bool IS_K, int R>
__global__ __launch_bounds__(256, (R <= 2 ? 4 : R <= 4 ? 3 : 2)) void pi_sweep_kernel(const uint16_t* __restrict__ Y, SegView sv, int g,
                                                       int bits, int n, int t_lr, const float* __restrict__ Bcur,
                                                       float* __restrict__ partial, int npart,
                                                       float* __restrict__ Atmp) {
  __shared__ SweepSmem<IS_K, R> sm;
  pi_sweep_body<IS_K, R, true>(sm, blockIdx.y, blockIdx.x, Y, sv.sz, sv.codes, sv.n_cap, sv.ng_cap, g, bits, n, t_lr, Bcur, partial,
                               npart, Atmp);
}

// ------------------------------------------------------------------ the pass of the last round when the Gram matrix exists
// A = R W, with the projection matrix W that pi_solve_kernel leaves, straight into the arena as fp16; from X, whose entries in S are
// left out.  The contraction runs on the matrix cores, 16 tokens x 32 channels x 16 columns at a time (v_mfma_f32_16x16x32_f16): a
// residual goes in as two fp16 numbers, its leading part and what that leaves, W the same way (columns 0 .. 7 its leading parts, 8 .. 15
// the rest), and all four products are formed in fp32.  Both are scaled by powers of two first, R by one per slab that keeps the largest
// residual there can be (the norm of R is the root of G's trace) in range, W by one per column, so that the two parts carry 22 bits
// also where fp16 alone would underflow.
//
// A wave takes 64 tokens, 16 at a time: rows come in as whole 256-byte lines, are turned in LDS (pieces of row r lie at piece ^ r: no bank
// conflicts in either direction), where the entries of S are zeroed by set bit of the mask, and are read as operands: lane (kg = lane /
// 16, m = lane % 16) holds channels 32 kg .. + 31 of row m, eight per instruction.  A Value row's group is then the same for all of a
// lane's channels; of the Keys a lane keeps the parameters of its 32 channels.  A stored Key code is read as an fp16 denormal (an AND
// for two codes; the power of two is part of the scale).
//
// Bound by the bytes (64 x 8 heads x 8192 tokens of rank 4: 2.5 GB in 465 us, 5.4 TB/s) next to vector issue (9 instructions per entry:
// the residual 3 to 5, the split 1.5, the zeroing 1).  With multiply-adds (rank times 1 per entry) and sums over the 16 lanes of a row it took
// 549 us and 15.5 instructions; 32 heads x 32768 tokens of rank 8 182 -> 119, 16 x 32 x 4096 of rank 4 273 -> 232 (all under the profiler).
// The two parts hold 22 of the 24 bits of an fp32 operand, and fewer (18 at the least that G itself resolves) of rows 2^17 and more below the
// largest of their slab.  Of the stored A that is nothing next to the rounding to fp16: of 16500 tensors (257 to 32768 tokens, ranks 2 to 8,
// 2 to 5 rounds, entries of 1e-3, 1 and 50) the error against the same steps in 64 bits is that of multiply-adds in fp32, 2.07e-4,
// to five digits or below it (the solver), and that of the product A B^T 0.9997 to 1.0002 of it in nine of ten of the others.  Three
// rows of 1000 times the rest make no difference either (median 0.1 of the Values' error before, one in a hundred above 1.003).
struct ProjectScale {   // per tensor and slab, left by pi_solve_kernel where its first partial Gram matrix was: the scale of R, its inverse, of each column of W the inverse
  float r, inv_r;
  float inv_w[8];
};
// `gram` as pi_solve_kernel takes it: strip matrices of the tensors' slabs, one after the other
__device__ __forceinline__ const ProjectScale& project_scale(const float* gram, size_t slab, int strips) {
  return *reinterpret_cast<const ProjectScale*>(gram + slab * strips * GRAM_FLOATS);
}
typedef _Float16 project_h8 __attribute__((ext_vector_type(8)));
constexpr int PROJECT_ROWS = 16;   // tokens of a step
constexpr int PROJECT_WAVE = 64;   // tokens of a wave

// Eight floats as the two fp16 parts of a matrix operand: hi, and what it leaves, v - hi (exact in fp32), rounded.  `one` is 1 in a scalar register
// that the compiler does not see through, so that the difference and its rounding are one mixed-precision instruction per entry.  It has to find
// them by itself: of instructions in inline asm it does not know that they write vector registers, and it leaves out wait states before
// a matrix instruction that reads those (it put one of two) and after one whose operands they overwrite.  (hi opaque: otherwise its
// halves are made twice; l0 opaque: otherwise the two halves of lo are rounded together, three instructions instead of two; by
// fours: behind such an asm the compiler leaves a wait state.  2493 vector instructions in the kernel of rank 4 and 2 bits, as with asm; 2635
// with neither, 2981 with a subtraction.)
__device__ __forceinline__ void split8(const float (&v)[8], float one, uint32_t (&hi)[4], uint32_t (&lo)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) hi[j] = pack_h2(v[2 * j], v[2 * j + 1]);
  GEAR_OPAQUE_VGPR4(hi);
  _Float16 l0[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) l0[j] = (_Float16)__builtin_fmaf((float)__builtin_bit_cast(h2_t, hi[j])[0], -one, v[2 * j]);
  GEAR_OPAQUE_VGPR4(l0);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const h2_t l = {l0[j], (_Float16)__builtin_fmaf((float)__builtin_bit_cast(h2_t, hi[j])[1], -one, v[2 * j + 1])};
    lo[j] = __builtin_bit_cast(uint32_t, l);
  }
}

template <bool IS_K, int BITS, int R>
__device__ __forceinline__ void project_wave(uint4 (&rows)[PROJECT_ROWS][D / 8], const uint16_t* __restrict__ X, const uint4* __restrict__ mask,
                                             const SegView& sv, int lg /* log2 of the group size */, int slab, int t0, int n, int t_lr,
                                             const uint16_t* __restrict__ W, const ProjectScale& scale) {
  const int lane = lane_id(), m = lane & 15, kg = lane >> 4;
  const GEAR_BUF_T xbuf = GEAR_BUF_MAKE(X + (size_t)slab * n * D, n * (D * 2));   // rows past the end read as 0
  const GEAR_BUF_T mbuf = GEAR_BUF_MAKE(mask + (size_t)slab * n, mask ? n * 16 : 0);
  const GEAR_BUF_T cbuf = GEAR_BUF_MAKE(sv.codes + (size_t)slab * sv.n_cap * (4 * BITS), IS_K ? n * (16 * BITS) : 0);
  const int ngl = 7 - lg;   // Values: log2 of a row's groups
  const GEAR_BUF_T pbuf = IS_K ? GEAR_BUF_MAKE(sv.sz + (size_t)slab * sv.ng_cap * D, ((n + (1 << lg) - 1) >> lg) * (D * 4))
                               : GEAR_BUF_MAKE(sv.sz + (((size_t)slab * sv.n_cap) << ngl), (n << ngl) * 4);
  constexpr float QMAX = (float)((1 << BITS) - 1);
  constexpr int CW = BITS;   // Keys: words of a lane's 32 codes

  uint4 xn[4];          // the next step's rows
  uint32_t mk, cn[CW];  // their mask (row lane / 4, channels 32 (lane % 4) ..), codes (Keys) or parameters (Values)
  auto request = [&](int t) {
#pragma unroll
    for (int i = 0; i < 4; ++i) xn[i] = GEAR_BUF_LOAD16_NT(xbuf, (t + 4 * i + kg) * (D * 2) + m * 16);
    mk = GEAR_BUF_LOAD4(mbuf, t * 16 + lane * 4);
    if constexpr (!IS_K) {
      cn[0] = GEAR_BUF_LOAD4(pbuf, (((t + m) << ngl) + ((32 * kg) >> lg)) * 4);
    } else if constexpr (BITS == 2) {
      const uint2 c = GEAR_BUF_LOAD8(cbuf, (t + m) * 32 + kg * 8);
      cn[0] = c.x; cn[1] = c.y;
    } else {
      const uint4 c = GEAR_BUF_LOAD16(cbuf, (t + m) * 64 + kg * 16);
      cn[0] = c.x; cn[1] = c.y; cn[2] = c.z; cn[3] = c.w;
    }
  };
  request(t0);
  // columns of W: lane's column m (of the leading parts, of the rest), channels 32 kg + 8 kb ..
  project_h8 wf[4];
  {
    const int r = m & 7;
    const GEAR_BUF_T wbuf = GEAR_BUF_MAKE(W + (size_t)slab * (2 * R * D), 2 * R * D * 2);
    const int at = r < R ? (((m >> 3) * R + r) * D + 32 * kg) * 2 : 2 * R * D * 2;   // columns past R: past the view, 0
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) wf[kb] = __builtin_bit_cast(project_h8, GEAR_BUF_LOAD16(wbuf, at + 16 * kb));
  }
  float one = 1.0f;
  GEAR_PIN_SGPR(one);
  const float rs = scale.r;
  float back[4];   // of columns 4 (kg % 2) + i
#pragma unroll
  for (int i = 0; i < 4; ++i) back[i] = scale.inv_w[4 * (kg & 1) + i] * scale.inv_r;

  float pmn[IS_K ? 32 : 1], pdl[IS_K ? 32 : 1];   // Keys: -zero and scale of the lane's channels, with the scale of R
  uint16_t* half = reinterpret_cast<uint16_t*>(&rows[0][0]);
#pragma unroll   // (rolled, the rows in flight are moved from registers to registers: 64 x 8 heads x 8192 tokens 20 us)
  for (int step = 0; step < PROJECT_WAVE / PROJECT_ROWS; ++step) {
    const int t = t0 + PROJECT_ROWS * step;
    if (t >= n) break;   // wave-uniform
    if constexpr (IS_K) {
      if (step == 0 || (t & ((1 << lg) - 1)) == 0) {   // a new group
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint4 z = GEAR_BUF_LOAD16(pbuf, ((t >> lg) * D + 32 * kg + 4 * i) * 4);
          const uint32_t zw[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int e = (4 * i + j) & 7;   // channel within its eight
            const int bit = BITS == 2 ? (e < 5 ? 2 * e : 2 * (e - 5)) : 4 * (e & 1);   // where its code lies after the AND below
            pmn[4 * i + j] = -(h2f(zw[j] >> 16) * rs);
            pdl[4 * i + j] = h2f(zw[j] & 0xFFFFu) * (rs * (float)(1 << (24 - bit)));
          }
        }
      }
    }
    // this step's rows, turned; the entries of S become 0
    wave_lds_sync();
#pragma unroll
    for (int i = 0; i < 4; ++i) rows[4 * i + kg][m ^ (4 * i + kg)] = xn[i];
    wave_lds_sync();
    uint32_t c[CW];
#pragma unroll
    for (int i = 0; i < (IS_K ? CW : 1); ++i) c[i] = cn[i];
    {
      const int row = lane >> 2, at = row * D + (((4 * (lane & 3)) ^ row) << 3);
      uint32_t w = mk;
      while (w != 0u) {
        const int b = __ffs((int)w) - 1;
        w &= w - 1u;
        half[at ^ b] = 0;   // (piece b / 8 of the four, entry b % 8)
      }
    }
    if (step + 1 < PROJECT_WAVE / PROJECT_ROWS) request(t + PROJECT_ROWS);   // (past n: nothing is fetched)
    wave_lds_sync();
    float mn = 0.0f, inv = 0.0f, dl = 0.0f;   // Values: my row's group
    if constexpr (!IS_K) {
      const GroupQ q = load_group(c[0]);
      const float inv_rs = scale.inv_r;
      mn = -(q.mn * rs);
      dl = q.delta * rs;
      inv = q.inv * inv_rs;
    }
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      const uint4 xv = rows[m][(4 * kg + kb) ^ m];
      const uint32_t x[4] = {xv.x, xv.y, xv.z, xv.w};
      uint32_t cv[8];   // Keys: the code of channel e in half `ch`
      if constexpr (IS_K && BITS == 2) {
        const uint32_t w = c[kb >> 1], w2 = w >> 10;
#pragma unroll
        for (int e = 0; e < 8; ++e) cv[e] = e < 5 ? w & (0x00030003u << (2 * e)) : w2 & (0x00030003u << (2 * (e - 5)));
      } else if constexpr (IS_K) {
        const uint32_t w = c[kb], w2 = w >> 8;
#pragma unroll
        for (int e = 0; e < 4; ++e) cv[e] = (e < 2 ? w : w2) & (0x000F000Fu << (4 * (e & 1)));
      }
      float res[8];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int e = 2 * j + h;
          const float y = h2f(h ? x[j] >> 16 : x[j] & 0xFFFFu);
          if constexpr (IS_K) {
            const int ch = BITS == 2 ? kb & 1 : e >> 2;
            const uint32_t cw = cv[BITS == 2 ? e : e & 3];
            const float code = h2f(ch ? cw >> 16 : cw & 0xFFFFu);   // times 2^(bit - 24)
            res[e] = __builtin_fmaf(-code, pdl[8 * kb + e], __builtin_fmaf(y, rs, pmn[8 * kb + e]));
          } else {
#pragma clang fp contract(off)
            const float ym = __builtin_fmaf(y, rs, mn);   // (y - zero) rs, rounded as y - zero is
            const float k = clamp_f32(rintf(__fmul_rn(ym, inv)), 0.0f, QMAX);
            res[e] = __builtin_fmaf(-k, dl, ym);
          }
        }
      }
      uint32_t hi[4], lo[4];
      split8(res, one, hi, lo);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[kb], __builtin_bit_cast(project_h8, make_uint4(hi[0], hi[1], hi[2], hi[3])), acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[kb], __builtin_bit_cast(project_h8, make_uint4(lo[0], lo[1], lo[2], lo[3])), acc, 0, 0, 0);
    }
    // register i of lane (kg, m): column 4 kg + i of token t + m; the rest of W's share lies 32 lanes further
    float av[4];
    const bool live = t + m >= t_lr;   // rows before t_lr take no part in the low-rank term
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t a = __float_as_uint(acc[i]), b = a;
      GEAR_LANE_SWAP32(a, b);
      av[i] = live ? (__uint_as_float(a) + __uint_as_float(b)) * back[i] : 0.0f;
    }
    const int rank = sv.rank;
    if (t + m < n && 4 * kg < R) {
      uint16_t* out = sv.A + ((size_t)slab * sv.n_cap + t + m) * rank + 4 * kg;
      if (R >= 4 && rank == R) {
        *reinterpret_cast<uint2*>(out) = make_uint2(pack_h2(av[0], av[1]), pack_h2(av[2], av[3]));
      } else if (R == 2 && rank == 2) {
        *reinterpret_cast<uint32_t*>(out) = pack_h2(av[0], av[1]);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (4 * kg + i < rank) out[i] = (uint16_t)f2h(av[i]);
      }
    }
  }
}
// Both tensors in one launch (z = 0: Keys, 1: Values): on a short prompt each is a few blocks' latency (512 tokens of 32
// heads: 9.6 + 9.3 us one after the other).  grid (ceil(n / 256), B*H, 2), block 256.
template <int BITS, int R>
__global__ __launch_bounds__(256, 3) void pi_project_kernel(const uint16_t* __restrict__ XK, const uint16_t* __restrict__ XV,
                                                         const uint4* __restrict__ maskK, const uint4* __restrict__ maskV, SegView ks, SegView vs,
                                                         int lgk, int lgv, int n, int t_lr, const uint16_t* __restrict__ W,
                                                         const float* __restrict__ gram, int nstrips) {
  __shared__ uint4 rows[4][PROJECT_ROWS][D / 8];
  const int wave = GEAR_WAVE_UNIFORM((int)(threadIdx.x >> 6)), t0 = (int)blockIdx.x * (4 * PROJECT_WAVE) + PROJECT_WAVE * wave;
  if (blockIdx.z == 0)
    project_wave<true, BITS, R>(rows[wave], XK, maskK, ks, lgk, blockIdx.y, t0, n, t_lr, W, project_scale(gram, blockIdx.y, nstrips));
  else
    project_wave<false, BITS, R>(rows[wave], XV, maskV, vs, lgv, blockIdx.y, t0, n, t_lr, W + (size_t)gridDim.y * (2 * R * D),
                                 project_scale(gram, (size_t)gridDim.y + blockIdx.y, nstrips));
}

// A = a C for tokens [256 * pt, 256 * pt + 256) of one slab, one token per thread.  Cs: LDS, R * R floats.
template <int R>
__device__ __forceinline__ void pi_finish_body(float* Cs, int slab, int pt, const float* __restrict__ Atmp,
                                               const float* __restrict__ cmat, const SegView& sv, int n) {
  float* C = Cs;
  if (threadIdx.x < R * R) C[threadIdx.x] = cmat[(size_t)slab * R * R + threadIdx.x];
  block_lds_sync();
  const int t = pt * 256 + threadIdx.x;
  if (t >= n) return;
  float a[R];
#pragma unroll
  for (int r = 0; r < R; ++r) a[r] = Atmp[((size_t)slab * n + t) * R + r];
  for (int j = 0; j < sv.rank; ++j) {
    float s = 0.0f;
#pragma unroll
    for (int r = 0; r < R; ++r) s += a[r] * C[r * R + j];
    sv.A[((size_t)slab * sv.n_cap + t) * sv.rank + j] = (uint16_t)f2h(s);
  }
}

// grid (ceil(n/256), B*H), block 256.
template <int R>
__global__ __launch_bounds__(256) void pi_finish_kernel(const float* __restrict__ Atmp,
                                                        const float* __restrict__ cmat, SegView sv, int n) {
  __shared__ float C[R * R];
  pi_finish_body<R>(C, blockIdx.y, blockIdx.x, Atmp, cmat, sv, n);
}

// The whole power iteration of a short segment (n <= PT: a flushed buffer) in one block per
// slab: the same steps as the separate kernels, in the same order and on the same workspace
// arrays, with block barriers where the kernel boundaries were (a slab's steps only depend
// on that slab).  Saves 7 launches of a few microseconds each per tensor.
// grid (B*H), block 256.
template <bool IS_K, int R>
__global__ __launch_bounds__(256, 1) void pi_small_kernel(const uint16_t* __restrict__ Y, SegView sv, int g, int bits,
                                                          int n, int t_lr, int iters, StartB sb,
                                                          float* __restrict__ Bcur, float* __restrict__ partial,
                                                          float* __restrict__ Atmp, float* __restrict__ cmat) {
  __shared__ UpdateSmem<R> um;
  __shared__ SweepSmem<IS_K, R> ss;
  __shared__ float Cs[R * R];
  const int slab = blockIdx.x;
  pi_update_body<R>(um, slab, true, sb, sv.rank, nullptr, 0, iters == 1 ? 1 : 0, 0, Bcur, cmat, sv);
  __syncthreads();   // also orders the block's global writes before its reads
#pragma unroll 1
  for (int l = 0; l < iters; ++l) {
    const int last = (l == iters - 1);
    // the rounds read the same Y, codes and scales: an offset the compiler cannot see through
    // keeps it from hoisting those loads out of the loop (and holding them in registers)
    int off = 0;
    GEAR_PIN_VGPR(off);
    if (last)
      pi_sweep_body<IS_K, R, true>(ss, slab, 0, Y + off, sv.sz + off, sv.codes + off, sv.n_cap, sv.ng_cap, g, bits, n, t_lr, Bcur,
                                   partial, 1, Atmp);
    else
      pi_sweep_body<IS_K, R, false>(ss, slab, 0, Y + off, sv.sz + off, sv.codes + off, sv.n_cap, sv.ng_cap, g, bits, n, t_lr, Bcur,
                                    partial, 1, Atmp);
    __syncthreads();
    pi_update_body<R>(um, slab, false, sb, sv.rank, partial, 1, (l == iters - 2) ? 1 : 0, last, Bcur, cmat, sv);
    __syncthreads();
  }
  pi_finish_body<R>(Cs, slab, 0, Atmp, cmat, sv, n);
}

// Sums a slab's partial Gram matrices into the first of them where there are many (long segments with few slabs): the
// solve kernel, one block per slab, would wait for one after another.  grid (GRAM_TILES, B*H), block 256.
constexpr int GRAM_SUM_MIN = 8;   // fewer than this are summed by the solve kernel: a launch costs as much as four to eight of them
__global__ __launch_bounds__(256) void gram_sum_kernel(float* __restrict__ gram, int nstrips) {
  float* g = gram + (size_t)blockIdx.y * nstrips * GRAM_FLOATS + blockIdx.x * 256 + threadIdx.x;
  float sum = 0.0f;
  for (int s0 = 0; s0 < nstrips; s0 += 16) {
    float t[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      t[u] = 0.0f;
      if (s0 + u < nstrips) t[u] = __builtin_nontemporal_load(g + (size_t)(s0 + u) * GRAM_FLOATS);   // block-uniform
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) sum += t[u];
  }
  *g = sum;
}

// Dynamic LDS of the solve kernel: G as [128][128] floats, entry (row, c) at c ^ solve_swizzle(row); B as [128][R] doubles, and the Gram
// matrix of A = R B.  Two blocks fit a CU.
template <int R>
struct SolveSmem {
  float G[D * D];      // at the end also P = G B, [128][R] doubles
  __attribute__((aligned(16))) double Bs[D * R];   // rows as SolveRows lays them out
  double GA[R][R];
};
// 128 rows of R doubles in LDS.  The pairs of a row are exchanged by a pattern that changes every time the rows have gone once
// through the banks, so that neither neighbouring rows nor every eighth one meet in a bank.
template <int R>
struct SolveRows {
  double* base;
  static __device__ __forceinline__ int turn(int row) { return (row >> (R == 8 ? 2 : R == 4 ? 3 : 4)) & (R / 2 - 1); }
  __device__ __forceinline__ double at(int row, int r) const { return base[row * R + 2 * ((r >> 1) ^ turn(row)) + (r & 1)]; }
  __device__ __forceinline__ void load(int row, double (&v)[R]) const {
#pragma unroll
    for (int p = 0; p < R / 2; ++p) {
      const double2 t = *reinterpret_cast<const double2*>(base + row * R + 2 * (p ^ turn(row)));
      v[2 * p] = t.x;
      v[2 * p + 1] = t.y;
    }
  }
  __device__ __forceinline__ void store(int row, const double (&v)[R]) const {
#pragma unroll
    for (int p = 0; p < R / 2; ++p) *reinterpret_cast<double2*>(base + row * R + 2 * (p ^ turn(row))) = make_double2(v[2 * p], v[2 * p + 1]);
  }
};
// Columns stay together by fours (one 16-byte read).  The eight rows 8 i .. 8 i + 7 that a product reads four at a time lie in both
// halves of the banks, and the tiles' scattered entries spread over 16 places.
__device__ __forceinline__ int solve_swizzle(int row) {
  return ((row & 1) << 5) | (((row >> 3) & 3) << 3) | (((row >> 5) & 1) << 2);
}
// Sums of N per-thread values over the block (256 threads), all in every thread: one pair of
// barriers for the N sums together.
template <int N>
__device__ __forceinline__ void block_sum_vec(double (&v)[N], double* red /* 4 * N */) {
  wave_sums_d<N>(v, N);
  block_lds_sync();
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) red[(threadIdx.x >> 6) * N + i] = v[i];
  }
  block_lds_sync();
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = (red[i] + red[N + i]) + (red[2 * N + i] + red[3 * N + i]);
}
// floor of half the exponent of x > 0, and 2^e: x = m * 4^h with m in [1, 4), so that sqrt(x) lies in [2^h, 2^(h + 1))
__device__ __forceinline__ int half_exponent(double x) {
  return ((int)((__builtin_bit_cast(uint64_t, x) >> 52) & 0x7FF) - 1023) >> 1;
}
__device__ __forceinline__ double pow2_d(int e) { return __builtin_bit_cast(double, (uint64_t)(e + 1023) << 52); }
// QR of the 128 rows of B that a wave holds (a: rows lane, b: rows lane + 64) by Gram-Schmidt applied twice; dependent columns become 0.
// Every inner product is a sum over the lanes, those of a pass together, with no barrier and no LDS traffic.
template <int R>
__device__ __forceinline__ void qr_rows(double (&a)[R], double (&b)[R]) {
  double before2[R];
#pragma unroll
  for (int j = 0; j < R; ++j) before2[j] = a[j] * a[j] + b[j] * b[j];
  wave_sums_d<R>(before2, R);
#pragma unroll
  for (int j = 0; j < R; ++j) {
    double after2 = before2[j];
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      if (j == 0) break;
      double d[R];   // the projections of a pass are taken together (classical Gram-Schmidt, applied twice); the second time the norm as well
#pragma unroll
      for (int i = 0; i < j; ++i) d[i] = a[i] * a[j] + b[i] * b[j];
      d[j] = a[j] * a[j] + b[j] * b[j];
      wave_sums_d<R>(d, pass == 0 ? j : j + 1);
      if (pass == 1) after2 = d[j];
#pragma unroll
      for (int i = 0; i < j; ++i) {
        a[j] -= d[i] * a[i];
        b[j] -= d[i] * b[i];
        // (what the second pass takes away is the rounding of the first: 1e-16 of the column, far below the cut)
        if (pass == 1) after2 -= d[i] * d[i];
      }
    }
    const bool ok = before2[j] > 0.0 && after2 > 1e-24 * before2[j];   // norm after > 1e-12 * norm before
    const double inv = ok ? rsqrt_d(after2) : 0.0;
    a[j] = ok ? a[j] * inv : 0.0;
    b[j] = ok ? b[j] * inv : 0.0;
  }
}
// The same for row c of B in thread c < 128 (q; the other threads of the block hold zeros and keep them).  Called by all 256 threads.
// The rows go through LDS (Bq) once; then each of the two waves that own rows orthonormalises all of them by itself (the same
// numbers in the same order) and keeps its own.
template <int R>
__device__ __forceinline__ void qr_columns(double (&q)[R], double (*Bq)[R] /* LDS [128][R] */) {
  const int c = threadIdx.x & (D - 1);
  const bool owner = threadIdx.x < D;
  block_lds_sync();
  if (owner) {
#pragma unroll
    for (int r = 0; r < R; ++r) Bq[c][r] = q[r];
  }
  block_lds_sync();
  if (!owner) return;   // (whole waves)
  const int lane = c & 63;
  double a[R], b[R];
#pragma unroll
  for (int r = 0; r < R; ++r) { a[r] = Bq[lane][r]; b[r] = Bq[lane + 64][r]; }
  qr_rows<R>(a, b);
#pragma unroll
  for (int r = 0; r < R; ++r) q[r] = c < 64 ? a[r] : b[r];
}
// Row 32 wave + 4 (lane % 8) + 2 (lane / 32) + (lane / 16) % 2 of G B, in fp64 (G symmetric, swizzled; the same in lanes 8 apart).  A lane
// multiplies four rows by every eighth row of B, from one 16-byte read of G and R / 2 of B; the eight lanes of the same rows add up.
template <int R>
__device__ __forceinline__ void gram_product(const float* G, const SolveRows<R>& Bs, int wave, int lane, double (&out)[R]) {
  const int kg = lane >> 3, rows = 32 * wave + 4 * (lane & 7);
  double acc[4][R];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int r = 0; r < R; ++r) acc[x][r] = 0.0;
#pragma unroll 4
  for (int i = 0; i < D / 8; ++i) {
    const int k = 8 * i + kg;
    const float4 g = *reinterpret_cast<const float4*>(G + k * D + (rows ^ solve_swizzle(k)));
    const double gd[4] = {(double)g.x, (double)g.y, (double)g.z, (double)g.w};
    double bk[R];
    Bs.load(k, bk);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int x = 0; x < 4; ++x) acc[x][r] = __builtin_fma(gd[x], bk[r], acc[x][r]);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      lane_swap32_d(acc[x][r], acc[x + 2][r]);
      acc[x][r] += acc[x + 2][r];   // lanes 32 ..: row x + 2
    }
    lane_swap16_d(acc[0][r], acc[1][r]);
    const double t = acc[0][r] + acc[1][r];   // odd rows of 16 lanes: row x + 1
    out[r] = t + dpp_d<DPP_ROR8>(t);
  }
}
// grid (B*H, tensors), block 256.
// A block is a chain of dependent fp64 steps that nothing in it hides, and two blocks fit a CU: Keys (y = 0) and Values (y = 1) of one call go in
// one launch, which up to 256 slabs costs the time of one tensor.  So the chain is kept short: a product G B reads G four rows and B a
// row at a time and adds up in lanes, every wave orthonormalises all 128 rows of B and finds C by itself, and sums over lanes are
// taken four at a time.  Cycles of a lone block (rank 4; rank 8), before (two threads per row of B through LDS, one sum at a time,
// C by one wave from LDS) and now: G 8000 -> 6400, a product 6800 -> 3400 (13000 -> 6800), QR 4600 -> 2600 (17700 -> 8200), B^T P 4000 -> 900
// (5500 -> 1800), C 7200 -> 1500 (30600 -> 7200), W 4200 -> 2200 (10600 -> 4800).  The kernel: 32 slabs of rank 4 22 -> 13 us, of rank 8
// (32768 tokens) 52 -> 27, 280 slabs of rank 4 49 -> 30, 512 slabs 68 -> 46.
template <int R>
__global__ __launch_bounds__(256, 2) void pi_solve_kernel(StartB sb0, StartB sb1, int rank,
                                                       float* __restrict__ gram_partial, int nstrips, int stride, int rounds,
                                                       float* __restrict__ Bcur_all, int last_round, uint16_t* Bf0, uint16_t* Bf1) {
  GEAR_DYN_LDS(smem_raw);
  SolveSmem<R>& sm = *reinterpret_cast<SolveSmem<R>*>(smem_raw);
  const SolveRows<R> Bs{sm.Bs}, Ps{reinterpret_cast<double*>(sm.G)};   // Ps: P = G B, at the end, in the place of G
  const int slab = blockIdx.x, tid = threadIdx.x, c = tid & (D - 1), half = GEAR_WAVE_UNIFORM(tid >> 7);
  const int wave = GEAR_WAVE_UNIFORM(tid >> 6), lane = tid & 63;
  const bool second = blockIdx.y != 0;
  const StartB sb = second ? sb1 : sb0;
  uint16_t* Bf = second ? Bf1 : Bf0;
  float* Bcur = Bcur_all + (size_t)blockIdx.y * gridDim.x * (D * R);
  auto start = [&]() {   // B <- the start matrix
#pragma unroll
    for (int i = 0; i < R / 2; ++i) {
      const int r = 2 * i + half;
      sm.Bs[c * R + 2 * (i ^ SolveRows<R>::turn(c)) + half] = r < rank ? (double)start_b(sb, slab, c, rank, r) : 0.0;
    }
  };
  if (rounds == 0) start();
  else {
    // G = sum of the strips' partial tiles (fixed order): element tid + 256 j is register j % 4... of tile j
    // (stride: strips per slab in memory)
    const float* gp = gram_partial + ((size_t)blockIdx.y * gridDim.x + slab) * stride * GRAM_FLOATS + tid;
    constexpr int AT_ONCE = 3;   // strips in flight
    float s[GRAM_TILES];
#pragma unroll
    for (int j = 0; j < GRAM_TILES; ++j) s[j] = 0.0f;
    for (int st = 0; st < nstrips; st += AT_ONCE) {
      float t[AT_ONCE][GRAM_TILES];   // a loop of their own for the loads: added into the sums directly, each would be waited for in turn
#pragma unroll
      for (int u = 0; u < AT_ONCE; ++u) {
        if (u > 0 && st + u >= nstrips) break;   // block-uniform
#pragma unroll
        for (int j = 0; j < GRAM_TILES; ++j) t[u][j] = __builtin_nontemporal_load(gp + (size_t)(st + u) * GRAM_FLOATS + 256 * j);
      }
      if (st == 0) start();   // (while the first ones are on their way)
#pragma unroll
      for (int u = 0; u < AT_ONCE; ++u) {
        if (u > 0 && st + u >= nstrips) break;
#pragma unroll
        for (int j = 0; j < GRAM_TILES; ++j) s[j] += t[u][j];
      }
    }
    // element tid of tile (e, f): register i = tid / 64 of lane l = tid % 64, i.e. G[8*(4*(l/16)+i) + e][8*(l%16) + f]
    const int row0 = 8 * (4 * (lane >> 4) + wave), col0 = 8 * (lane & 15);
    int j = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int f = e; f < 8; ++f) {
        sm.G[(row0 + e) * D + ((col0 + f) ^ solve_swizzle(row0 + e))] = s[j];
        // (a diagonal tile holds both (row, col) and (col, row) itself)
        if (e != f) sm.G[(col0 + f) * D + ((row0 + e) ^ solve_swizzle(col0 + f))] = s[j];
        ++j;
      }
  }
  block_lds_sync();
  const int row = 32 * wave + 4 * (lane & 7) + 2 * (lane >> 5) + ((lane >> 4) & 1);   // of a product (gram_product)
  const bool writes = (lane & 8) == 0;
  for (int l = 0; l < rounds; ++l) {
    double y[R], n2[R];
    gram_product<R>(sm.G, Bs, wave, lane, y);
    // keep magnitudes in range between rounds: the columns of B are scaled to norm 1 before the product, which is to say its result is
    // (after the last product the QR below rescales anyway)
    if (l > 0) {   // block-uniform
      double a[R], b[R];
      Bs.load(lane, a);
      Bs.load(lane + 64, b);
#pragma unroll
      for (int r = 0; r < R; ++r) n2[r] = a[r] * a[r] + b[r] * b[r];
      wave_sums_d<R>(n2, R);
#pragma unroll
      for (int r = 0; r < R; ++r) y[r] = n2[r] > 0.0 ? y[r] * rsqrt_d(n2[r]) : 0.0;
    }
    block_lds_sync();
    if (writes) Bs.store(row, y);
    block_lds_sync();
  }
  {
    double qa[R], qb[R];   // rows lane, lane + 64 of B
    Bs.load(lane, qa);
    Bs.load(lane + 64, qb);
    qr_rows<R>(qa, qb);
    block_lds_sync();
    if (wave == 0) {
      Bs.store(lane, qa);
      Bs.store(lane + 64, qb);
    }
    block_lds_sync();
  }
  if (!last_round) {
    if (tid < D) {
#pragma unroll
      for (int r = 0; r < R; ++r) Bcur[((size_t)slab * D + c) * R + r] = (float)Bs.at(c, r);
    }
    return;
  }
  // The last round of Algorithm 2 without another pass over R for B: with A = R B (B orthonormal now),
  // orth(A) = A C and the round's result B' = R^T orth(A) = (R^T R) B C = G B C, while the r x r Gram matrix
  // that gives C is A^T A = B^T G B.  What is left for the pass over R is A itself: orth(A) = R (B C), so
  // the projection matrix W = B C goes to Bcur and B' to the arena.
  double trace = 0.0;
  {
    double y[R];
    gram_product<R>(sm.G, Bs, wave, lane, y);
    if (wave == 3) trace = wave_sum_d((double)sm.G[lane * D + (lane ^ solve_swizzle(lane))] +
                                      (double)sm.G[(lane + 64) * D + ((lane + 64) ^ solve_swizzle(lane + 64))]);
    block_lds_sync();
    if (writes) Ps.store(row, y);
    block_lds_sync();
  }
#pragma unroll
  for (int p0 = 0; p0 < R * R; p0 += 16) {   // entry (i, j) of B^T P: 16 lanes each
    const int p = p0 + (tid >> 4), i = (p / R) % R, j = p % R, k0 = tid & 15;
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < D / 16; ++u) s = __builtin_fma(Bs.at(k0 + 16 * u, i), Ps.at(k0 + 16 * u, j), s);
    s = row16_sum_d(s);
    if (k0 == 0 && p < R * R) sm.GA[i][j] = s;
  }
  block_lds_sync();
  double C[R][R];
  {
    double ga[R][R];   // symmetric up to rounding
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int j = i; j < R; ++j) ga[i][j] = 0.5 * (sm.GA[i][j] + sm.GA[j][i]);
    coeff_orth<R, false>(ga, C, [&](int a, int j, double x) { C[a][j] = x; });
  }
  // W for the pass over R (pi_project_kernel), column by column: scaled to a norm of 256 .. 512, which is the norm of C's column as B is
  // orthonormal, and split into two fp16 parts.  The halves of the block take half of the columns each.
  uint16_t* W = reinterpret_cast<uint16_t*>(Bcur) + (size_t)slab * (2 * R * D);
  // (into the first partial matrix of this slab, which this block alone has read)
  ProjectScale* sc = reinterpret_cast<ProjectScale*>(gram_partial + ((size_t)blockIdx.y * gridDim.x + slab) * stride * GRAM_FLOATS);
  double q[R], pr[R];
  Bs.load(c, q);
  Ps.load(c, pr);
#pragma unroll
  for (int j = 0; j < R; ++j) {
    if ((j < R / 2) != (half == 0)) continue;   // wave-uniform
    double w = 0.0, bo = 0.0, n2 = 0.0;
#pragma unroll
    for (int r = 0; r <= j; ++r) {
      w += q[r] * C[r][j];
      bo += pr[r] * C[r][j];
      n2 += C[r][j] * C[r][j];
    }
    const int ex = n2 > 0.0 ? half_exponent(n2) : 0;   // norm in [2^ex, 2^(ex + 1))
    const double ws = w * pow2_d(8 - ex);
    const uint32_t hi = f2h((float)ws);
    W[j * D + c] = (uint16_t)hi;
    W[(R + j) * D + c] = (uint16_t)f2h((float)(ws - (double)h2f(hi)));
    if (c == 0) sc->inv_w[j] = (float)pow2_d(ex - 8);
    if (j < rank) Bf[((size_t)slab * D + c) * rank + j] = (uint16_t)f2h((float)bo);
  }
  if (tid == 192) {   // no residual of the rows that count is larger than the norm of R, which then is below 2^15
    const int ex = trace > 0.0 ? half_exponent(trace) : 0;
    sc->r = (float)pow2_d(14 - ex);
    sc->inv_r = (float)pow2_d(ex - 14);
#pragma unroll
    for (int j = R; j < 8; ++j) sc->inv_w[j] = 0.0f;
  }
}

// ------------------------------------------------------------------ segments of at most 64 tokens
// A flushed streaming buffer (n_b = 20 .. 64 tokens in the paper's settings) is small enough for one
// block to keep its residual in LDS: the rows are read and the residual derived once, and every round
// of Algorithm 2 runs out of LDS with a handful of block barriers; nothing goes through the workspace.
// Same steps and the same precision choices as the kernels above: A = R B and B' = R^T A accumulate in
// fp32, column scaling, the QR of B and the coefficient-space orth(A) in fp64.
// grid (B*H, 2): Keys (y = 0) and Values (y = 1) in one launch, block 256 (a block is one long chain of steps: a
// flushed buffer of 128 slabs took 12 us, the two launches one after the other 13 + 11).  Sums over rows keep eight reads or 16 lanes at
// work: one row after the other, a call on 32 slabs x 20 tokens took 21.1 us and not 19.2, on 2048 x 33 of rank 4 157 and not 139.
// Thread (r0 = tid/16, oc = tid%16) derives channels 8*oc..+7 of rows
// r0 + 16 k and later forms their share of A; thread (half = tid/128, c = tid%128) sums rows
// 8 half .. + 7 of every 16 of B'[c][:], thread (0, c) owns row c of B.
constexpr int TINY_ROWS = PI_TINY_ROWS;
constexpr int TINY_PITCH = D + 4;   // floats per residual row in LDS (16-byte aligned pieces)
template <int R>
struct TinySmem {
  __attribute__((aligned(16))) float Rs[TINY_ROWS][TINY_PITCH];   // rows >= n are 0
  __attribute__((aligned(16))) float Bs[D][R];
  float As[TINY_ROWS][R];
  float part[D][R];
  double Bq[D][R];      // the rows of B for its QR
  double red[4 * (R + 1)];
  double GA[R][R];
  double C[R][R];
};
template <int R>
__global__ __launch_bounds__(256, 3) void pi_tiny_kernel(const uint16_t* __restrict__ YK, const uint16_t* __restrict__ YV, SegView ks,
                                                      SegView vs, int gk, int gv, int bits, int n, int t_lr, int iters, StartB sbk,
                                                      StartB sbv) {
  __shared__ TinySmem<R> sm;
  const bool is_k = blockIdx.y == 0;
  const SegView sv = is_k ? ks : vs;
  const StartB sb = is_k ? sbk : sbv;
  const uint16_t* Y = is_k ? YK : YV;
  const int g = is_k ? gk : gv;
  const int slab = blockIdx.x, tid = threadIdx.x;
  const int r0 = tid >> 4, oc = tid & 15;
  const int c = tid & (D - 1), half = tid >> 7;
  const bool owner = half == 0;
  const int rank = sv.rank;
  // ---- the residual, once: R = (Y - zero) - code * scale (Keys: stored codes; Values: the quantizer's sequence)
  {
    const int lg = 31 - __clz(g), ngl = 7 - lg;   // (Keys with per-vector groups pass g = 32768: one group)
    const float qmax = (float)((1 << bits) - 1);
    const GEAR_BUF_T xbuf = GEAR_BUF_MAKE(Y + (size_t)slab * n * D, n * (D * 2));
    const GEAR_BUF_T cbuf = GEAR_BUF_MAKE(sv.codes + (size_t)slab * sv.n_cap * (4 * bits), is_k ? n * (16 * bits) : 0);
    const GEAR_BUF_T pbuf = is_k ? GEAR_BUF_MAKE(sv.sz + (size_t)slab * sv.ng_cap * D, ((n + g - 1) >> lg) * (D * 4))
                                 : GEAR_BUF_MAKE(sv.sz + (((size_t)slab * sv.n_cap) << ngl), (n << ngl) * 4);
    uint4 xv[4], pz[2][2];
    uint32_t cw[4], pv[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {   // every load is requested before the first one is used
      const int t = r0 + 16 * k;
      xv[k] = GEAR_BUF_LOAD16_NT(xbuf, t * (D * 2) + oc * 16);   // rows past the end read as 0
      // (Values: a view of no codes; Keys: a word that is not used)
      const int co = t * (16 * bits) + oc * (bits == 4 ? 4 : 2);
      cw[k] = bits == 4 ? GEAR_BUF_LOAD4(cbuf, co) : GEAR_BUF_LOAD2(cbuf, co);
      pv[k] = GEAR_BUF_LOAD4(pbuf, is_k ? 0 : ((t << ngl) + ((oc * 8) >> lg)) * 4);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {   // Keys: 64 rows lie in at most two groups (g >= 32)
      pz[j][0] = make_uint4(0, 0, 0, 0);
      pz[j][1] = make_uint4(0, 0, 0, 0);
      if (is_k) {
        pz[j][0] = GEAR_BUF_LOAD16(pbuf, (j * D + oc * 8) * 4);
        pz[j][1] = GEAR_BUF_LOAD16(pbuf, (j * D + oc * 8) * 4 + 16);
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int t = r0 + 16 * k;
      const uint32_t w[4] = {xv[k].x, xv[k].y, xv[k].z, xv[k].w};
      float res[8];
      if (is_k) {
        const bool second = (t >> lg) != 0;
        const uint4 z0 = second ? pz[1][0] : pz[0][0], z1 = second ? pz[1][1] : pz[0][1];
        const uint32_t z[8] = {z0.x, z0.y, z0.z, z0.w, z1.x, z1.y, z1.z, z1.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float y = h2f((e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xFFFFu));
          res[e] = __builtin_fmaf(-(float)GEAR_UBFE(cw[k], e * bits, bits), h2f(z[e] & 0xFFFFu), y - h2f(z[e] >> 16));
        }
      } else {
        const GroupQ q = load_group(pv[k]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float y = h2f((e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xFFFFu));
          res[e] = quant_error(y, q.mn, q.inv, q.delta, qmax);
        }
      }
      if (t >= n || t < t_lr) {   // no such row / a row that takes no part in the low-rank term
#pragma unroll
        for (int e = 0; e < 8; ++e) res[e] = 0.0f;
      }
      *reinterpret_cast<float4*>(&sm.Rs[t][oc * 8]) = make_float4(res[0], res[1], res[2], res[3]);
      *reinterpret_cast<float4*>(&sm.Rs[t][oc * 8 + 4]) = make_float4(res[4], res[5], res[6], res[7]);
    }
  }
  double q[R];
#pragma unroll
  for (int r = 0; r < R; ++r) q[r] = (owner && r < rank) ? (double)start_b(sb, slab, c, rank, r) : 0.0;
  if (iters == 1) qr_columns<R>(q, sm.Bq);   // the only round is also the last: B is orthonormalised first
#pragma unroll 1
  for (int l = 0; l < iters; ++l) {
    const bool last = l == iters - 1;
    block_lds_sync();
    if (owner) {
#pragma unroll
      for (int r = 0; r < R; ++r) sm.Bs[c][r] = (float)q[r];
    }
    block_lds_sync();
    // A = R B: the 16 lanes of a row of lanes hold one token
    {
      float bc[8][R];
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int r = 0; r < R; ++r) bc[e][r] = sm.Bs[oc * 8 + e][r];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (16 * k >= n) break;   // block-uniform
        const int t = r0 + 16 * k;
        const float4 x0 = *reinterpret_cast<const float4*>(&sm.Rs[t][oc * 8]);
        const float4 x1 = *reinterpret_cast<const float4*>(&sm.Rs[t][oc * 8 + 4]);
        const float res[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
        for (int r = 0; r < R; ++r) {
          float a = 0.0f;
#pragma unroll
          for (int e = 0; e < 8; ++e) a += res[e] * bc[e][r];
          a = row16_sum(a);
          if (oc == 0) sm.As[t][r] = a;
        }
      }
    }
    block_lds_sync();
    // B' = R^T A
    float p[R];
#pragma unroll
    for (int r = 0; r < R; ++r) p[r] = 0.0f;
    for (int t0 = 8 * half; t0 < n; t0 += 16) {   // (rows n .. of the last 16 are 0; eight reads in flight: one by one, each costs its latency)
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float rv = sm.Rs[t0 + u][c];
#pragma unroll
        for (int r = 0; r < R; ++r) p[r] += rv * sm.As[t0 + u][r];
      }
    }
    if (!owner) {
#pragma unroll
      for (int r = 0; r < R; ++r) sm.part[c][r] = p[r];
    }
    block_lds_sync();
    double qn[R];
#pragma unroll
    for (int r = 0; r < R; ++r) qn[r] = owner ? (double)p[r] + (double)sm.part[c][r] : 0.0;
    if (!last) {
      // keep magnitudes in range between rounds (the span, hence A B^T, is unchanged)
      double n2[R];
#pragma unroll
      for (int r = 0; r < R; ++r) n2[r] = qn[r] * qn[r];
      block_sum_vec<R>(n2, sm.red);
#pragma unroll
      for (int r = 0; r < R; ++r) q[r] = n2[r] > 0.0 ? qn[r] * rsqrt_d(n2[r]) : 0.0;
      if (l == iters - 2) qr_columns<R>(q, sm.Bq);   // the QR of B that opens the last round
      continue;
    }
    // last round: orth(A) = A C from the r x r Gram matrix of A; B = R^T orth(A) = B' C
#pragma unroll
    for (int p0 = 0; p0 < R * R; p0 += 16) {   // an entry by 16 lanes
      const int e = p0 + (tid >> 4), i = (e / R) % R, j = e % R;
      double s = 0.0;
#pragma unroll
      for (int t = 0; t < TINY_ROWS; t += 16)
        if (t + oc < n) s += (double)sm.As[t + oc][i] * (double)sm.As[t + oc][j];
      s = row16_sum_d(s);
      if (oc == 0 && e < R * R) sm.GA[i][j] = s;
    }
    block_lds_sync();
    if (tid < 64) coeff_orth_lds<R>(sm.GA, sm.C, tid);
    block_lds_sync();
    if (owner) {
      for (int j = 0; j < rank; ++j) {
        double bo = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) bo += qn[r] * sm.C[r][j];
        sv.Bf[((size_t)slab * D + c) * rank + j] = (uint16_t)f2h((float)bo);
      }
    }
    for (int i = tid; i < n * rank; i += 256) {
      const int t = i / rank, j = i - t * rank;
      float a = 0.0f;
#pragma unroll
      for (int r = 0; r < R; ++r) a += sm.As[t][r] * (float)sm.C[r][j];
      sv.A[((size_t)slab * sv.n_cap + t) * rank + j] = (uint16_t)f2h(a);
    }
  }
}

// ------------------------------------------------------------------ host side
template <int R>
static hipError_t raise_solve_lds() {
  static std::atomic<uint64_t> lds_raised{0};
  return raise_dynamic_lds(reinterpret_cast<const void*>(pi_solve_kernel<R>), lds_raised, sizeof(SolveSmem<R>), sizeof(SolveSmem<R>));
}

// Keys' per-vector grouping: one group per segment
static int key_group_size(const Dims& dm) { return dm.kcvt ? 32768 : dm.g; }
static int log2_group(int g) { return 31 - __builtin_clz((unsigned)g); }

template <int R>
static hipError_t run_pi_pair(const PiTensor& k, const PiTensor& v, const Dims& dm, int n, int t_lr, int iters, float* Bcur,
                              float* gram, int nstrips, hipStream_t st) {
  const int slabs = dm.B * dm.H, rank = k.sv.rank;
  if (n <= TINY_ROWS) {   // (a flushed buffer of the paper's sizes) with its residual resident in LDS
    hipLaunchKernelGGL(pi_tiny_kernel<R>, dim3(slabs, 2), dim3(256), 0, st, k.Y, v.Y, k.sv, v.sv, key_group_size(dm), dm.g, dm.bits, n,
                       t_lr, iters, k.sb, v.sb);
    return hipGetLastError();
  }
  const hipError_t e = raise_solve_lds<R>();
  if (e != hipSuccess) return e;
  // rounds 1 .. L-1: B <- (R^T R)^(L-1) B0 on the Gram matrix; then QR(B), the last round's B and the factor of orth(A)
  const bool summed = nstrips >= GRAM_SUM_MIN;
  if (summed) hipLaunchKernelGGL(gram_sum_kernel, dim3(GRAM_TILES, 2 * slabs), dim3(256), 0, st, gram, nstrips);
  hipLaunchKernelGGL(pi_solve_kernel<R>, dim3(slabs, 2), dim3(256), sizeof(SolveSmem<R>), st, k.sb, v.sb, rank, gram,
                     summed ? 1 : nstrips, nstrips, iters - 1, Bcur, 1, k.sv.Bf, v.sv.Bf);
  // one light pass writes A
  const dim3 grid((n + 4 * PROJECT_WAVE - 1) / (4 * PROJECT_WAVE), slabs, 2);
  const uint16_t* W = reinterpret_cast<const uint16_t*>(Bcur);
  const int lgk = log2_group(key_group_size(dm)), lgv = log2_group(dm.g);
  if (dm.bits == 2)
    hipLaunchKernelGGL((pi_project_kernel<2, R>), grid, dim3(256), 0, st, k.X, v.X, k.mask, v.mask, k.sv, v.sv, lgk, lgv, n, t_lr, W,
                       (const float*)gram, nstrips);
  else
    hipLaunchKernelGGL((pi_project_kernel<4, R>), grid, dim3(256), 0, st, k.X, v.X, k.mask, v.mask, k.sv, v.sv, lgk, lgv, n, t_lr, W,
                       (const float*)gram, nstrips);
  return hipGetLastError();
}

template <int R>
static hipError_t run_pi(bool is_k, const PiTensor& x, const Dims& dm, int n, int t_lr, int iters, float* Bcur, float* partial,
                         float* Atmp, float* cmat, hipStream_t st) {
  const int slabs = dm.B * dm.H;
  const int npart = (n + PT - 1) / PT;
  const int g = is_k ? key_group_size(dm) : dm.g;
  if (npart == 1) {   // a short segment: everything in one block per slab
    if (is_k)
      hipLaunchKernelGGL((pi_small_kernel<true, R>), dim3(slabs), dim3(256), 0, st, x.Y, x.sv, g, dm.bits, n, t_lr, iters, x.sb, Bcur, partial, Atmp, cmat);
    else
      hipLaunchKernelGGL((pi_small_kernel<false, R>), dim3(slabs), dim3(256), 0, st, x.Y, x.sv, g, dm.bits, n, t_lr, iters, x.sb, Bcur, partial, Atmp, cmat);
    return hipGetLastError();
  }
  // a single round (no Gram pass): A = R B, orth(A) through its r x r Gram matrix, B = R^T A
  const hipError_t e = raise_solve_lds<R>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(pi_solve_kernel<R>, dim3(slabs), dim3(256), sizeof(SolveSmem<R>), st, x.sb, x.sb, x.sv.rank, (float*)nullptr,
                     0, 0, 0, Bcur, 0, x.sv.Bf, x.sv.Bf);
  const dim3 grid(npart, slabs);
  if (is_k)
    hipLaunchKernelGGL((pi_sweep_kernel<true, R>), grid, dim3(256), 0, st, x.Y, x.sv, g, dm.bits, n, t_lr, (const float*)Bcur, partial, npart, Atmp);
  else
    hipLaunchKernelGGL((pi_sweep_kernel<false, R>), grid, dim3(256), 0, st, x.Y, x.sv, g, dm.bits, n, t_lr, (const float*)Bcur, partial, npart, Atmp);
  hipLaunchKernelGGL(pi_update_kernel<R>, dim3(slabs), dim3(256), 0, st, (const float*)partial, npart, Bcur, cmat, x.sv);
  hipLaunchKernelGGL(pi_finish_kernel<R>, dim3((n + 255) / 256, slabs), dim3(256), 0, st, (const float*)Atmp,
                     (const float*)cmat, x.sv, n);
  return hipGetLastError();
}

int pi_padded_rank(int rank) { return rank <= 2 ? 2 : rank <= 4 ? 4 : 8; }

hipError_t launch_power_iteration_pair(const PiTensor& k, const PiTensor& v, const Dims& dm, int n, int t_lr, int iters, float* Bcur,
                                       float* gram, int nstrips, hipStream_t st) {
  switch (pi_padded_rank(k.sv.rank)) {
    case 2: return run_pi_pair<2>(k, v, dm, n, t_lr, iters, Bcur, gram, nstrips, st);
    case 4: return run_pi_pair<4>(k, v, dm, n, t_lr, iters, Bcur, gram, nstrips, st);
    default: return run_pi_pair<8>(k, v, dm, n, t_lr, iters, Bcur, gram, nstrips, st);
  }
}

hipError_t launch_power_iteration(bool is_k, const PiTensor& x, const Dims& dm, int n, int t_lr, int iters, float* Bcur, float* partial,
                                  float* Atmp, float* cmat, hipStream_t st) {
  switch (pi_padded_rank(x.sv.rank)) {
    case 2: return run_pi<2>(is_k, x, dm, n, t_lr, iters, Bcur, partial, Atmp, cmat, st);
    case 4: return run_pi<4>(is_k, x, dm, n, t_lr, iters, Bcur, partial, Atmp, cmat, st);
    default: return run_pi<8>(is_k, x, dm, n, t_lr, iters, Bcur, partial, Atmp, cmat, st);
  }
}

}  // namespace gear
