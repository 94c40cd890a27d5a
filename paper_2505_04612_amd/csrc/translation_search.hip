// Relative-translation grid search (FastMap, arXiv 2505.04612, appendix on
// global translation, "Relative Translation"): for every pair, with the
// relative rotation R_ij = R_j R_i^T of the global rotations, the unit vector
// among the candidates with the lowest mean squared algebraic epipolar error
// t^T A_n t / |Q_n|, A_n = B^T W_n B, B[:, k] = flatten([e_k]_x R_ij); the
// winner keeps the sign of the pair's prior estimate.
//
// k_ts_search: a workgroup takes one to kTsBatches batches of kTsPairs pairs.  Lanes of its
// first wavefront form A_n, one pair each, for all of them (a dependent chain
// of about 750 instructions that the other wavefronts wait for, so it is paid
// once per workgroup); every wavefront then holds a batch's form entries in
// scalar registers
// (five of six; the sixth in a vector register, as eight pairs' six entries
// would not leave room for the addresses).  Each lane visits candidates
// thread, thread + kTsBlock, ..., forms the candidate's six monomials once and
// evaluates them against the eight forms: eight independent chains of one
// product and five FMAs with a scalar operand, and no LDS reads.  The minima
// (value, then index, so the lowest candidate index wins among equal errors)
// are combined by a reduce-scatter over the lanes and through LDS over the
// wavefronts.  Bound by float64 VALU issue, 9 to 10 instructions per
// evaluation.  Per call with 4,096 candidates, against k_ts_search_few, which
// reads the monomials from LDS: 4.8k pairs 15.6 us and 22.9 (issued back to back,
// the host's share of a call is 11 to 14 us), 29.5k pairs 57.2 and 72.6, 187k
// pairs 319 and 366.
#include "fm_internal.h"

#include <cmath>

namespace {

constexpr int kTsBlock = 256;   // threads per workgroup
constexpr int kTsWaves = kTsBlock / 64;
constexpr int kTsPairs = 8;     // pairs evaluated together
constexpr int kTsBatches = 8;   // batches per workgroup, at most (64 pairs: one per lane of a wavefront)

// A = B^T W B from the compact Gram (W_{(ab),(cd)} = W36[6 q(a,c) + q(b,d)])
// and R = R_ij, as its six distinct entries (A00, A11, A22, A01, A02, A12).
__device__ inline void pair_form(const double* __restrict__ w36, const double R[3][3], double A6[6]) {
  // B_k as 3x3: rows of [e_k]_x R
  double B[3][3][3];
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    B[0][0][b] = 0.0;      B[0][1][b] = -R[2][b]; B[0][2][b] = R[1][b];
    B[1][0][b] = R[2][b];  B[1][1][b] = 0.0;      B[1][2][b] = -R[0][b];
    B[2][0][b] = -R[1][b]; B[2][1][b] = R[0][b];  B[2][2][b] = 0.0;
  }
  // WB_l[(ab)] = sum_(cd) W[(ab),(cd)] B_l[c][d]
  double A[3][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      double wb[3] = {0.0, 0.0, 0.0};
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const double w = w36[6 * mono_q(a, c) + mono_q(b, d)];
#pragma unroll
          for (int l = 0; l < 3; ++l) wb[l] += w * B[l][c][d];
        }
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int l = 0; l < 3; ++l) A[k][l] += B[k][a][b] * wb[l];
    }
  A6[0] = A[0][0];
  A6[1] = A[1][1];
  A6[2] = A[2][2];
  A6[3] = A[0][1] + A[1][0];
  A6[4] = A[0][2] + A[2][0];
  A6[5] = A[1][2] + A[2][1];
}

// A minimum and the candidate it belongs to; take() keeps the lower value,
// then the lower index.
struct TsMin {
  double v;
  int i;
  __device__ void take(double ov, int oi) {
    const bool t = (ov < v) | ((ov == v) & (oi < i));
    v = t ? ov : v;
    i = t ? oi : i;
  }
};

template <int BIT>
__device__ inline TsMin ts_partner(const TsMin& m) {
  if constexpr (BIT >= 4) {
    return TsMin{__shfl_xor(m.v, 1 << BIT), __shfl_xor(m.i, 1 << BIT)};
  } else {
    // row_mirror, row_half_mirror, quad_perm xor 2 and xor 1 (the partner has
    // the opposite value of bit BIT and the same value of the higher ones
    // already reduced)
    constexpr int kCtrl = BIT == 3 ? 0x140 : (BIT == 2 ? 0x141 : (BIT == 1 ? 0x4E : 0xB1));
    return TsMin{dpp_mov_d<kCtrl>(m.v), __builtin_amdgcn_update_dpp(0, m.i, kCtrl, 0xF, 0xF, false)};
  }
}

// Reduce-scatter stage over lane bit BIT: lanes keep the lower or upper half
// of 2H minima, combined with the partner's.
template <int BIT, int H>
__device__ inline void ts_stage(TsMin (&m)[kTsPairs], int lane) {
  const bool up = (lane >> BIT) & 1;
#pragma unroll
  for (int k = 0; k < H; ++k) {
    const TsMin lo = m[k], hi = m[k + H];
    const TsMin send = {up ? lo.v : hi.v, up ? lo.i : hi.i};
    const TsMin got = ts_partner<BIT>(send);
    m[k] = TsMin{up ? hi.v : lo.v, up ? hi.i : lo.i};
    m[k].take(got.v, got.i);
  }
}

__device__ inline double uniform_d(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readfirstlane((int)b), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__global__ __launch_bounds__(kTsBlock) void k_ts_search(const double* __restrict__ W36, const float* __restrict__ params,
                                                      const int32_t* __restrict__ cams,
                                                      const int64_t* __restrict__ offsets,
                                                      const double* __restrict__ cand, int32_t C,
                                                      const float* __restrict__ t_prior, int64_t P, int batches,
                                                      float* __restrict__ t_out, int32_t* __restrict__ best_out,
                                                      double* __restrict__ err_out) {
  __shared__ double form[kTsPairs * kTsBatches][6];
  __shared__ double red_v[2][kTsWaves][kTsPairs];
  __shared__ int red_i[2][kTsWaves][kTsPairs];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = kTsPairs * batches;
  const int64_t n_first = (int64_t)blockIdx.x * per;
  if (tid < per) {
    const int64_t n = n_first + tid;
    double A6[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (n < P) {
      double a1[3], a2[3], t[3], Ri[3][3], Rj[3][3], R[3][3];
      load_pose(params, cams[2 * n], a1, a2, t);
      gs_matrix(gs_forward(a1, a2), Ri);
      load_pose(params, cams[2 * n + 1], a1, a2, t);
      gs_matrix(gs_forward(a1, a2), Rj);
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) R[a][b] = Rj[a][0] * Ri[b][0] + Rj[a][1] * Ri[b][1] + Rj[a][2] * Ri[b][2];
      pair_form(W36 + 36 * n, R, A6);
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) form[tid][k] = A6[k];
  }
  __syncthreads();
  // the minima's LDS rows alternate, so that one barrier a batch suffices
  for (int bt = 0; bt < batches; ++bt) {
    const int64_t n0 = n_first + bt * kTsPairs;
    if (n0 >= P) break;   // the whole workgroup
    const double(*f)[6] = form + bt * kTsPairs;
    double A[kTsPairs][6];
    TsMin m[kTsPairs];
#pragma unroll
    for (int p = 0; p < kTsPairs; ++p) {
#pragma unroll
      for (int k = 0; k < 5; ++k) A[p][k] = uniform_d(f[p][k]);
      A[p][5] = f[p][5];
      m[p] = TsMin{INFINITY, 0x7fffffff};
    }
    // the next candidate is loaded while this one is evaluated (past the end,
    // the last one again)
    int64_t next = 3 * (int64_t)(tid < C ? tid : C - 1);
    double nx = cand[next], ny = cand[next + 1], nz = cand[next + 2];
    for (int c = tid; c < C; c += kTsBlock) {
      const double x = nx, y = ny, z = nz;
      next = 3 * (int64_t)(c < C - kTsBlock ? c + kTsBlock : C - 1);
      nx = cand[next];
      ny = cand[next + 1];
      nz = cand[next + 2];
      const double xx = x * x, yy = y * y, zz = z * z, xy = x * y, xz = x * z, yz = y * z;
#pragma unroll
      for (int p = 0; p < kTsPairs; ++p) {
        double q = A[p][1] * yy;
        q = fma(A[p][0], xx, q);
        q = fma(A[p][2], zz, q);
        q = fma(A[p][3], xy, q);
        q = fma(A[p][4], xz, q);
        q = fma(A[p][5], yz, q);
        if (q < m[p].v) {
          m[p].v = q;
          m[p].i = c;
        }
      }
    }
    // eight minima over the lanes: 8 -> 4 -> 2 -> 1 over bits 3, 2, 1, then the
    // kept one over bits 0, 4 and 5
    ts_stage<3, 4>(m, lane);
    ts_stage<2, 2>(m, lane);
    ts_stage<1, 1>(m, lane);
    TsMin o = ts_partner<0>(m[0]);
    m[0].take(o.v, o.i);
    o = ts_partner<4>(m[0]);
    m[0].take(o.v, o.i);
    o = ts_partner<5>(m[0]);
    m[0].take(o.v, o.i);
    if (lane < 16 && (lane & 1) == 0) {
      const int p = 4 * (lane >> 3 & 1) + 2 * (lane >> 2 & 1) + (lane >> 1 & 1);
      red_v[bt & 1][wave][p] = m[0].v;
      red_i[bt & 1][wave][p] = m[0].i;
    }
    __syncthreads();
    const int64_t n = n0 + tid;
    if (tid >= kTsPairs || n >= P) continue;
    TsMin best = {red_v[bt & 1][0][tid], red_i[bt & 1][0][tid]};
#pragma unroll
    for (int w = 1; w < kTsWaves; ++w) best.take(red_v[bt & 1][w][tid], red_i[bt & 1][w][tid]);
    const int64_t cnt = offsets[n + 1] - offsets[n];
    double tp[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) tp[k] = (double)t_prior[3 * n + k];
    if (cnt == 0 || best.i >= C) {
#pragma unroll
      for (int k = 0; k < 3; ++k) t_out[3 * n + k] = (float)tp[k];
      if (best_out) best_out[n] = -1;
      if (err_out) err_out[n] = 0.0;
      continue;
    }
    double tb[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) tb[k] = cand[3 * (int64_t)best.i + k];
    const double sgn = (tb[0] * tp[0] + tb[1] * tp[1] + tb[2] * tp[2]) < 0.0 ? -1.0 : 1.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) t_out[3 * n + k] = (float)(sgn * tb[k]);
    if (best_out) best_out[n] = best.i;
    if (err_out) err_out[n] = best.v / (double)cnt;
  }
}

constexpr int kTsTile = 1024;   // candidates per LDS tile: six monomials each (48 KB of float64)

// The same search with one lane per (pair, slice of the candidates): S lanes
// share a pair and visit candidates slice, slice + S, ...; the candidates are
// staged in LDS tiles and read as broadcasts, which bounds it (48 bytes per
// evaluation); the S lanes combine their minima (value, then index) with a
// butterfly, so the lowest candidate index wins among equal errors whatever S
// is.  Every lane forms its own pair's A_n, so the forms' chain is paid once by
// a whole launch: what few candidates on a large graph need (ts_few_shape).
// The evaluations round as k_ts_search's, so the results are the same to the bit.
__global__ __launch_bounds__(kTsBlock) void k_ts_search_few(const double* __restrict__ W36, const float* __restrict__ params,
                                                      const int32_t* __restrict__ cams,
                                                      const int64_t* __restrict__ offsets,
                                                      const double* __restrict__ cand, int32_t C,
                                                      const float* __restrict__ t_prior, int64_t P, int S,
                                                      float* __restrict__ t_out, int32_t* __restrict__ best_out,
                                                      double* __restrict__ err_out) {
  __shared__ double tile[kTsTile * 6];
  const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n = gtid / S;
  const int slice = (int)(gtid % S);
  const bool live = n < P;
  double A6[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  int64_t cnt = 0;
  if (live) {
    cnt = offsets[n + 1] - offsets[n];
    double a1[3], a2[3], t[3], Ri[3][3], Rj[3][3], R[3][3];
    load_pose(params, cams[2 * n], a1, a2, t);
    gs_matrix(gs_forward(a1, a2), Ri);
    load_pose(params, cams[2 * n + 1], a1, a2, t);
    gs_matrix(gs_forward(a1, a2), Rj);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) R[a][b] = Rj[a][0] * Ri[b][0] + Rj[a][1] * Ri[b][1] + Rj[a][2] * Ri[b][2];
    pair_form(W36 + 36 * n, R, A6);
  }
  double best_v = INFINITY;
  int best_i = 0x7fffffff;
  for (int base = 0; base < C; base += kTsTile) {
    const int len = C - base < kTsTile ? C - base : kTsTile;
    __syncthreads();
    // each candidate's monomials (x^2, y^2, z^2, xy, xz, yz), once per tile
    for (int k = threadIdx.x; k < len; k += blockDim.x) {
      const double x = cand[3 * (int64_t)(base + k)], y = cand[3 * (int64_t)(base + k) + 1],
                   z = cand[3 * (int64_t)(base + k) + 2];
      double* m = tile + 6 * k;
      m[0] = x * x;
      m[1] = y * y;
      m[2] = z * z;
      m[3] = x * y;
      m[4] = x * z;
      m[5] = y * z;
    }
    __syncthreads();
    if (live) {
      // four of this lane's candidates per step: their forms are independent
      // chains, evaluated as one expression each (the same rounding as one
      // at a time) and compared in candidate order (the same ties)
      int c = slice;
      for (; c + 3 * S < len; c += 4 * S) {
        double q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double* m = tile + 6 * (c + u * S);
          q[u] = A6[0] * m[0] + A6[1] * m[1] + A6[2] * m[2] + A6[3] * m[3] + A6[4] * m[4] + A6[5] * m[5];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (q[u] < best_v) {
            best_v = q[u];
            best_i = base + c + u * S;
          }
      }
      for (; c < len; c += S) {
        const double* m = tile + 6 * c;
        const double q = A6[0] * m[0] + A6[1] * m[1] + A6[2] * m[2] + A6[3] * m[3] + A6[4] * m[4] + A6[5] * m[5];
        if (q < best_v) {
          best_v = q;
          best_i = base + c;
        }
      }
    }
  }
  // combine the S lanes of a pair: lower value, then lower index
  for (int sh = 1; sh < S; sh <<= 1) {
    const double ov = __shfl_xor(best_v, sh);
    const int oi = __shfl_xor(best_i, sh);
    if (ov < best_v || (ov == best_v && oi < best_i)) {
      best_v = ov;
      best_i = oi;
    }
  }
  if (!live || slice != 0) return;
  double tp[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) tp[k] = (double)t_prior[3 * n + k];
  if (cnt == 0 || best_i >= C) {
#pragma unroll
    for (int k = 0; k < 3; ++k) t_out[3 * n + k] = (float)tp[k];
    if (best_out) best_out[n] = -1;
    if (err_out) err_out[n] = 0.0;
    return;
  }
  double tb[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) tb[k] = cand[3 * (int64_t)best_i + k];
  const double sgn = (tb[0] * tp[0] + tb[1] * tp[1] + tb[2] * tp[2]) < 0.0 ? -1.0 : 1.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) t_out[3 * n + k] = (float)(sgn * tb[k]);
  if (best_out) best_out[n] = best_i;
  if (err_out) err_out[n] = best_v / (double)cnt;
}

// Launch shape of one of the two kernels: workgroups, lanes per pair (few) or
// batches per workgroup (many), and its estimated time.
struct TsShape {
  int64_t blocks;
  int split;
  double us;
};

// The estimates are the work of the fullest CU and what a call takes beside it,
// fitted to 13 numbers of candidates from 1 to 6,000 on 11 graphs of 4.8k to
// 187k pairs, within a tenth near the line.  us per call, few against many, with
// 64, 1,000, 2,000 and 4,096 candidates: 15k pairs 11.7 / 11.7, 17.2 / 16.8, 25.7 /
// 22.7, 44.1 / 33.5; 45k 12.0 / 23.9, 28.9 / 37.7, 51.7 / 55.8, 98.7 / 90.4; 99k
// 13.1 / 45.4, 64.7 / 77.9, 122 / 116, 242 / 192; 187k 17.8 / 74.2, 98.4 / 129, 186 /
// 192, 366 / 319; below 11k pairs many is never slower.

// Lanes per pair: enough (pair, slice) lanes for about two wavefronts per SIMD,
// at most 64.
inline TsShape ts_few_shape(int64_t P, int32_t C, int num_cu) {
  int S = 1;
  while (S < 64 && P * S < (int64_t)num_cu * 4 * 2 * 64 && S < C) S <<= 1;
  const int64_t blocks = (P * S + kTsBlock - 1) / kTsBlock, full = (blocks + num_cu - 1) / num_cu;
  return TsShape{blocks, S, 8.0 + 0.0295 * (double)C * (double)full / S};
}

// One batch per workgroup until the launch has four workgroups per CU (the
// co-resident limit by registers), then more, so that the forms' latency is
// paid less often (186k pairs, 4,096 candidates: 337 us with one batch, 318
// with eight).
inline TsShape ts_many_shape(int64_t P, int32_t C, int num_cu) {
  const int64_t fit = P / ((int64_t)kTsPairs * 4 * num_cu), b = fit < 1 ? 1 : (fit > kTsBatches ? kTsBatches : fit);
  const int64_t blocks = (P + kTsPairs * b - 1) / (kTsPairs * b), full = b * ((blocks + num_cu - 1) / num_cu);
  return TsShape{blocks, (int)b, 4.0 + (double)full * (0.75 + 6.5e-4 * (double)C)};
}

}  // namespace

extern "C" fm_status fm_translation_search(fm_ctx* ctx, fm_scene* s, const double* W36, const float* params,
                                           const double* cand, int32_t C, const float* t_prior, float* t_out,
                                           int32_t* best, double* err_min, fm_stream stream) {
  if (!ctx) return FM_EINVAL;
  if (!s) return fm_fail(ctx, FM_EINVAL, "fm_translation_search: scene is NULL");
  if (s->ctx != ctx) return fm_fail(ctx, FM_EINVAL, "fm_translation_search: scene belongs to another context");
  if (C < 1) return fm_fail(ctx, FM_EINVAL, "fm_translation_search: no candidates");
  if (s->P == 0) return FM_OK;
  if (!W36 || !params || !cand || !t_prior || !t_out)
    return fm_fail(ctx, FM_EINVAL, "fm_translation_search: NULL argument");
  FM_HIP_TRY(ctx, hipSetDevice(ctx->device));
  fm_timed timer(ctx, FM_K_TS_SEARCH, (hipStream_t)stream);
  const TsShape few = ts_few_shape(s->P, C, ctx->num_cu), many = ts_many_shape(s->P, C, ctx->num_cu);
  if (few.us < many.us)
    hipLaunchKernelGGL(k_ts_search_few, dim3((unsigned)few.blocks), dim3(kTsBlock), 0, (hipStream_t)stream, W36, params,
                       s->pair_cams, s->offsets, cand, C, t_prior, s->P, few.split, t_out, best, err_min);
  else
    hipLaunchKernelGGL(k_ts_search, dim3((unsigned)many.blocks), dim3(kTsBlock), 0, (hipStream_t)stream, W36, params,
                       s->pair_cams, s->offsets, cand, C, t_prior, s->P, many.split, t_out, best, err_min);
  FM_CHECK_LAUNCH(ctx);
  return FM_OK;
}
