// Loss, hand-written adjoint and Adam for epipolar adjustment: eq.
// (epipolar-objective-l2) evaluated per image pair from the compact Grams,
// its gradient with respect to the 6D rotation parameters and translations,
// and the fused persistent loop (Sec. 3.4's kernel fusion, re-designed as one
// cooperative kernel that also applies the Adam update).
//
// One iteration has two phases:
//   pair phase    one thread per image pair: E_n and W_n e_n in float64, the
//                 pair's loss, and the adjoint back to dL/dR and dL/dt of its
//                 two cameras (two 6-float records per pair);
//   camera phase  one 16-lane row of a wavefront per camera (four cameras
//                 per wavefront): the records of the camera's pairs are summed
//                 in a fixed order (lanes stride the camera's incidence list,
//                 then a fixed DPP tree inside the row), the Gram-Schmidt
//                 adjoint gives dL/d(a1, a2), and lanes 0..8 of the row apply
//                 Adam to one parameter each.
// The float64 quadratic form matters: near a minimum e^T W e is many orders
// of magnitude below |W| |e|^2, so float32 would cancel most of its digits.
#include <type_traits>

#include "fm_internal.h"

// Compact Gram of one pair held in registers (indexed like a pointer to it).
template <typename WT>
struct GramRegs {
  WT v[36];
  __device__ const WT& operator[](int k) const { return v[k]; }
};

template <typename WT>
__device__ inline void load_gram(const WT* __restrict__ w, GramRegs<WT>& g) {
#pragma unroll
  for (int k = 0; k < 36; ++k) g.v[k] = w[k];
}

// Loss term of pair n and what its adjoint needs: E_n at the current poses
// (`rot`, optional, holds each camera's rotation from Gram-Schmidt of the
// current parameters, so pairs need not repeat it) and g = W_n e_n, in
// float64.
struct PairEval {
  double Ri[3][3], Rj[3][3], Rij[3][3], th[3], ti[3], g[3][3];
  double ns, loss;
};

// From the poses in e.Ri, e.ti, e.Rj and tj.
template <typename W>
__device__ inline void pair_terms(PairEval& e, const double tj[3], const W& w) {
  double E[3][3];
  e.ns = pair_essential(e.Ri, e.ti, e.Rj, tj, e.Rij, e.th, E);
  // g = W e with W_{(ab),(cd)} = W36[6 q(a,c) + q(b,d)]: walk the index
  // pairs (a, c) and read only the 6-entry row q(a,c) of the compact Gram
  // for each, so few Gram values are live at once
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) e.g[a][b] = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      double row[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) row[k] = (double)w[6 * mono_q(a, c) + k];
#pragma unroll
      for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int d = 0; d < 3; ++d) e.g[a][b] = fma(row[mono_q(b, d)], E[c][d], e.g[a][b]);
    }
  e.loss = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) e.loss = fma(E[a][b], e.g[a][b], e.loss);
}

template <typename W>
__device__ inline PairEval pair_eval(const float* __restrict__ params, const double* __restrict__ rot, int ci, int cj,
                                     const W& w) {
  PairEval e;
  double a1[3], a2[3], tj[3];
  if (rot) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      e.ti[k] = (double)params[(int64_t)ci * 9 + 6 + k];
      tj[k] = (double)params[(int64_t)cj * 9 + 6 + k];
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      e.Ri[k / 3][k % 3] = rot[(int64_t)ci * 9 + k];
      e.Rj[k / 3][k % 3] = rot[(int64_t)cj * 9 + k];
    }
  } else {
    load_pose(params, ci, a1, a2, e.ti);
    gs_matrix(gs_forward(a1, a2), e.Ri);
    load_pose(params, cj, a1, a2, tj);
    gs_matrix(gs_forward(a1, a2), e.Rj);
  }
  pair_terms(e, tj, w);
  return e;
}

// Loss term of an evaluated pair and its adjoint in compact form
// (essential_adjoint_omega): om, dL/dt_i, dL/dt_j (all 0 for a degenerate
// pair).
__device__ inline double pair_adjoint(const PairEval& e, double two_inv_Z, double om[3], double dti[3],
                                      double dtj[3]) {
  double G[3][3], o[3], di[3], dj[3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) G[a][b] = two_inv_Z * e.g[a][b];
  essential_adjoint_omega(G, e.th, e.ns, e.Rij, e.Ri, e.ti, o, di, dj);
  // degenerate pairs by selection: with the stores under a branch the arrays
  // went to scratch memory
  const bool ok = e.ns > 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    om[k] = ok ? o[k] : 0.0;
    dti[k] = ok ? di[k] : 0.0;
    dtj[k] = ok ? dj[k] : 0.0;
  }
  return ok ? e.loss : 0.0;
}

template <typename W>
__device__ inline double pair_loss_omega(const float* __restrict__ params, const double* __restrict__ rot, int ci,
                                         int cj, const W& w, double two_inv_Z, double om[3], double dti[3],
                                         double dtj[3]) {
  return pair_adjoint(pair_eval(params, rot, ci, cj, w), two_inv_Z, om, dti, dtj);
}

// Camera-major record layout: the 6 numbers of item q of the
// incidence lists (a pair's side for one camera: its body-frame rotation
// gradient, -om for camera i and om for camera j, then dL/dt of that camera)
// at contrib + 6 q, so a camera's records are one contiguous run: float32 in
// the fused loop, float64 in the standalone gradient (V: a vector of two).
template <typename V>
__device__ inline void store_sides(float* __restrict__ contrib, int qi, int qj, const double om[3],
                                   const double dti[3], const double dtj[3]) {
  using T = decltype(V::x);
  V* di = reinterpret_cast<V*>(contrib) + (int64_t)qi * 3;
  V* dj = reinterpret_cast<V*>(contrib) + (int64_t)qj * 3;
  di[0] = V{(T)-om[0], (T)-om[1]};
  di[1] = V{(T)-om[2], (T)dti[0]};
  di[2] = V{(T)dti[1], (T)dti[2]};
  dj[0] = V{(T)om[0], (T)om[1]};
  dj[1] = V{(T)om[2], (T)dtj[0]};
  dj[2] = V{(T)dtj[1], (T)dtj[2]};
}

// Pair phase of the fused pair loop over pairs [first, P) with stride
// `stride`: each side written to its slot; returns this thread's loss sum
// (float64, in pair order).  The cameras and slots of the first two pairs
// come in registers (ci0, cj0 and ci1, cj1, qi0, qj0 and qi1, qj1), read once
// per solve; with kHold the first pair's Gram too (w0).
template <bool kHold, typename WT>
__device__ inline double pair_phase_slots(const float* params, const double* rot, const int32_t* cams,
                                          const int32_t* pair_slot, const WT* W36, int64_t P, double two_inv_Z,
                                          float* contrib, int64_t first, int64_t stride, int ci0, int cj0, int ci1,
                                          int cj1, int qi0, int qj0, int qi1, int qj1, const GramRegs<WT>& w0) {
  double sum = 0.0, om[3], dti[3], dtj[3];
  if constexpr (kHold) {
    if (first < P) {
      sum += pair_loss_omega(params, rot, ci0, cj0, w0, two_inv_Z, om, dti, dtj);
      store_sides<float2>(contrib, qi0, qj0, om, dti, dtj);
    }
  }
  for (int64_t n = kHold ? first + stride : first; n < P; n += stride) {
    const bool held0 = !kHold && n == first, held1 = n == first + stride;
    const int ci = held0 ? ci0 : (held1 ? ci1 : cams[2 * n]), cj = held0 ? cj0 : (held1 ? cj1 : cams[2 * n + 1]);
    const int qi = held0 ? qi0 : (held1 ? qi1 : pair_slot[2 * n]);
    const int qj = held0 ? qj0 : (held1 ? qj1 : pair_slot[2 * n + 1]);
    sum += pair_loss_omega(params, rot, ci, cj, W36 + n * 36, two_inv_Z, om, dti, dtj);
    store_sides<float2>(contrib, qi, qj, om, dti, dtj);
  }
  return sum;
}

// Record slots per lane that the camera rows load in one round:
// 6 x 16 covers cameras of up to 96 pairs (slots past them are read in
// further rounds).
constexpr int kRowItems = 6;

// Summed records of one camera in every lane of its row, from the
// camera-major layout (slots lo..hi-1, 6 numbers each; a row is LANES lanes):
// lane l takes slots lo + l + LANES j; the first NE of them are all loaded before any is added
// (without lane conditions, under which each load is waited for on its own:
// slots past the end load the last one's record, or a camera without pairs
// its predecessor's, and count as 0), then added in slot order, then the rest.
// The pair loop on the 5,000-camera street graph (74 pairs per camera) takes
// 0.5 us less per iteration than with conditional loads.  acc = (om, dL/dt) of the camera.
template <int NE, typename V, int LANES = 16>
__device__ inline void row_camera_sums_slots(int lo, int hi, const float* __restrict__ contrib, int lane,
                                             double (&acc)[6]) {
  const V* c = reinterpret_cast<const V*>(contrib);
  const int l = lane & (LANES - 1);
  const int last = max(hi - 1, 0);
  V r[NE][3];
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    const int q = min(lo + l + LANES * j, last);
#pragma unroll
    for (int k = 0; k < 3; ++k) r[j][k] = c[(int64_t)q * 3 + k];
  }
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    const bool live = lo + l + LANES * j < hi;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      r[j][k].x = live ? r[j][k].x : 0;
      r[j][k].y = live ? r[j][k].y : 0;
    }
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) acc[k] = 0.0;
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    acc[0] += r[j][0].x; acc[1] += r[j][0].y; acc[2] += r[j][1].x;
    acc[3] += r[j][1].y; acc[4] += r[j][2].x; acc[5] += r[j][2].y;
  }
  for (int q = lo + LANES * NE + l; q < hi; q += LANES) {
    const V a0 = c[(int64_t)q * 3], a1 = c[(int64_t)q * 3 + 1], a2 = c[(int64_t)q * 3 + 2];
    acc[0] += a0.x; acc[1] += a0.y; acc[2] += a1.x;
    acc[3] += a1.y; acc[4] += a2.x; acc[5] += a2.y;
  }
  if constexpr (LANES == 16) {
    row_sum6(acc, lane);
  } else {
    double v = row_partial6(acc, lane);
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
#pragma unroll
    for (int k = 0; k < 6; ++k) acc[k] = __shfl(v, 8 * (k / 3) + 2 * (k % 3));
  }
}

// ------------------------------------------------------------------ standalone loss + gradient

// One thread per pair: loss term and both sides' records.
template <typename WT>
__global__ __launch_bounds__(kBlock) void k_pair_phase(const float* __restrict__ params,
                                                       const int32_t* __restrict__ cams,
                                                       const int32_t* __restrict__ pair_slot,
                                                       const WT* __restrict__ W36, int64_t P, double inv_Z,
                                                       const int64_t* __restrict__ Z_dev, float* __restrict__ contrib,
                                                       double* __restrict__ loss_part) {
  __shared__ double lds[kBlock / 64];
  const double iz = Z_dev ? 1.0 / (double)(*Z_dev > 0 ? *Z_dev : 1) : inv_Z;
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double v = 0.0;
  if (n < P) {
    double om[3], dti[3], dtj[3];
    v = pair_loss_omega(params, nullptr, cams[2 * n], cams[2 * n + 1], W36 + n * 36, 2.0 * iz, om, dti, dtj);
    store_sides<double2>(contrib, pair_slot[2 * n], pair_slot[2 * n + 1], om, dti, dtj);
  }
  const double t = block_sum(v, lds);
  if (threadIdx.x == 0) loss_part[blockIdx.x] = t;
}

// One row of LANES lanes per camera: its records summed in a fixed order, the
// Gram-Schmidt adjoint (rows of 16: the same lanes for four cameras, whose
// float64 chains are what the kernel issues; of 64 where a camera has more than
// kWideCamera pairs, which 16 lanes take too long to add: 2,500 cameras, one of
// 2,499 pairs, 42.6 us a call by rows of 16, 26.6 by wavefronts when the choice
// was made).  The last workgroup, one more than the cameras
// take, sums the loss partials instead.  The records are float64: rounded to
// float32, the gradient was on average 3.5e-8 from 64 bits (relative, 24 graphs
// of 20 to 3,000 cameras; 2.5e-8 now, the rounding of the result), further
// than the 3.4e-8 of 24-float records.  The whole call on the 186k-pair street
// graph: 20.4 us (16.1 with float32 records), against 57.9 with the partials
// added by one thread, a wavefront per camera and 24-float records; at 1,000
// cameras 11.8 against 23.5, 12 against 14 to 15 up to 200 cameras, where the
// launches bound them.
constexpr int kWideCamera = 1024;

template <int LANES>
__global__ __launch_bounds__(kLanes) void k_camera_grad(const float* __restrict__ params,
                                                        const int32_t* __restrict__ cam_ptr,
                                                        const float* __restrict__ contrib, int32_t N,
                                                        const double* __restrict__ loss_part, int64_t n_part,
                                                        double inv_Z, const int64_t* __restrict__ Z_dev,
                                                        float* __restrict__ grad, double* __restrict__ loss,
                                                        unsigned cam_blocks) {
  if (blockIdx.x == cam_blocks) {
    double v = 0.0;
#pragma unroll 4
    for (int64_t k = threadIdx.x; k < n_part; k += kLanes) v += loss_part[k];
#pragma unroll
    for (int sh = 32; sh >= 1; sh >>= 1) v += __shfl_xor(v, sh);
    if (threadIdx.x == 0) *loss = v * (Z_dev ? 1.0 / (double)(*Z_dev > 0 ? *Z_dev : 1) : inv_Z);
    return;
  }
  const int lane = threadIdx.x & 63, l = lane & (LANES - 1);
  const int64_t c = ((int64_t)blockIdx.x * kLanes + threadIdx.x) / LANES;
  if (c >= N) return;   // whole rows leave together: the row exchanges stay within live rows
  double a1[3], a2[3], t[3], acc6[6], acc[12], g[9];
  load_pose(params, (int)c, a1, a2, t);
  const Gs f = gs_forward(a1, a2);
  row_camera_sums_slots<kRowItems, double2, LANES>(cam_ptr[c], cam_ptr[c + 1], contrib, lane, acc6);
  omega_grad(f, acc6, acc6 + 3, acc);
  gs_adjoint(acc, f, a2, g);
  if (l < 9) grad[c * 9 + l] = (float)pick9(g, l);
}

static fm_status check_w(fm_ctx* ctx, const char* fn, const void* W36, fm_dtype wdt, int64_t P) {
  if (!W36 && P > 0) return fm_fail(ctx, FM_EINVAL, "%s: W36 is NULL", fn);
  if (wdt != FM_F64 && wdt != FM_F32) return fm_fail(ctx, FM_EDTYPE, "%s: W36 must be FM_F64 or FM_F32", fn);
  return FM_OK;
}

extern "C" fm_status fm_epipolar_loss_grad(fm_ctx* ctx, fm_scene* s, const void* W36, fm_dtype wdt,
                                           const float* params, double inv_Z, const int64_t* Z_dev, double* loss,
                                           float* grad, fm_stream stream) {
  if (!ctx) return FM_EINVAL;
  if (!s) return fm_fail(ctx, FM_EINVAL, "fm_epipolar_loss_grad: scene is NULL");
  if (s->ctx != ctx) return fm_fail(ctx, FM_EINVAL, "fm_epipolar_loss_grad: scene belongs to another context");
  fm_status rc = check_w(ctx, "fm_epipolar_loss_grad", W36, wdt, s->P);
  if (rc != FM_OK) return rc;
  if (!params && s->N > 0) return fm_fail(ctx, FM_EINVAL, "fm_epipolar_loss_grad: params is NULL");
  if (!Z_dev && !(inv_Z >= 0.0)) return fm_fail(ctx, FM_EINVAL, "fm_epipolar_loss_grad: inv_Z must be >= 0");
  FM_HIP_TRY(ctx, hipSetDevice(ctx->device));
  hipStream_t st = (hipStream_t)stream;
  const unsigned gp = grid_for(s->P > 0 ? s->P : 1, kBlock);
  {
  fm_timed timer(ctx, FM_K_PAIR, st);
  if (wdt == FM_F64)
    hipLaunchKernelGGL(k_pair_phase<double>, dim3(gp), dim3(kBlock), 0, st, params, s->pair_cams,
                       s->pair_slot, (const double*)W36, s->P, inv_Z, Z_dev, s->contrib, s->loss_part);
  else
    hipLaunchKernelGGL(k_pair_phase<float>, dim3(gp), dim3(kBlock), 0, st, params, s->pair_cams,
                       s->pair_slot, (const float*)W36, s->P, inv_Z, Z_dev, s->contrib, s->loss_part);
  }
  FM_CHECK_LAUNCH(ctx);
  const bool wide = s->max_pairs > kWideCamera;
  const unsigned cam_blocks = grad ? grid_for((int64_t)s->N * (wide ? 64 : 16), kLanes) : 0u,
                 gc = cam_blocks + (loss ? 1u : 0u);
  if (gc > 0) {
  fm_timed timer(ctx, FM_K_CAMERA, st);
  hipLaunchKernelGGL(wide ? k_camera_grad<64> : k_camera_grad<16>, dim3(gc), dim3(kLanes), 0, st, params, s->cam_ptr, s->contrib, s->N,
                     s->loss_part, (int64_t)gp, inv_Z, Z_dev, grad, loss, cam_blocks);
  }
  FM_CHECK_LAUNCH(ctx);
  if (ctx->check) {
    // degenerate pairs and non-finite parameters at the input poses, then
    // the outputs themselves
    if ((rc = fm_launch_essentials(s, params, st)) != FM_OK) return rc;
    if ((rc = fm_check_finite(ctx, st, loss, 1, true, FM_CHECK_LOSS)) != FM_OK) return rc;
    if ((rc = fm_check_finite(ctx, st, grad, (int64_t)s->N * 9, false, FM_CHECK_LOSS)) != FM_OK) return rc;
  }
  return FM_OK;
}

// ------------------------------------------------------------------ Adam

__global__ void k_adam(int64_t n, float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, const float* __restrict__ lr, int lr_stride, double b1, double b2,
                       double eps, double bc1, double bc2) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  float mk = m[k], vk = v[k];
  p[k] = adam_update(p[k], g[k], mk, vk, (double)lr[lr_stride ? k : 0], b1, b2, eps, bc1, bc2);
  m[k] = mk;
  v[k] = vk;
}

extern "C" fm_status fm_adam_step(fm_ctx* ctx, int64_t n, float* p, const float* g, float* m, float* v,
                                  int64_t step, const float* lr, int lr_stride, float beta1, float beta2, float eps,
                                  fm_stream stream) {
  if (!ctx) return FM_EINVAL;
  if (n < 0) return fm_fail(ctx, FM_ESHAPE, "fm_adam_step: n < 0");
  if (n > 0 && (!p || !g || !m || !v || !lr)) return fm_fail(ctx, FM_EINVAL, "fm_adam_step: NULL argument");
  if (step < 1) return fm_fail(ctx, FM_EINVAL, "fm_adam_step: step is 1-based");
  if (lr_stride != 0 && lr_stride != 1) return fm_fail(ctx, FM_EINVAL, "fm_adam_step: lr_stride must be 0 or 1");
  if (!(beta1 >= 0.0f && beta1 < 1.0f && beta2 >= 0.0f && beta2 < 1.0f && eps >= 0.0f))
    return fm_fail(ctx, FM_EINVAL, "fm_adam_step: bad beta/eps");
  if (n == 0) return FM_OK;
  FM_HIP_TRY(ctx, hipSetDevice(ctx->device));
  const double bc1 = 1.0 - pow((double)beta1, (double)step), bc2 = 1.0 - pow((double)beta2, (double)step);
  hipLaunchKernelGGL(k_adam, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, (hipStream_t)stream, n, p, g, m, v, lr,
                     lr_stride, (double)beta1, (double)beta2, (double)eps, bc1, bc2);
  FM_CHECK_LAUNCH(ctx);
  return FM_OK;
}

// ------------------------------------------------------------------ fused persistent solve

// Re-arms the barriers before a launch: counts, generations and XCD
// registrations start at 0, and the launch's failure flag is cleared (a
// launch that ended on a failed barrier leaves it set).
__device__ inline void bar_clear(unsigned* __restrict__ bar) {
  if (threadIdx.x == 0) {
    bar[0] = 0u;
    bar[32] = 0u;
    bar[64] = 0u;
    bar[kBarTop] = 0u;
  }
  // grid_sync's per-XCD arrival counts, generations and workgroup
  // registrations
  if (threadIdx.x < kMaxXcd) {
    bar[kBarXcdCount + 32 * threadIdx.x] = 0u;
    bar[kBarXcdGen + 32 * threadIdx.x] = 0u;
    bar[kBarXcdReg + 32 * threadIdx.x] = 0u;
  }
}

__global__ void k_bar_reset(unsigned* __restrict__ bar) { bar_clear(bar); }

hipError_t fm_bar_reset(unsigned* bar, hipStream_t st) {
  hipLaunchKernelGGL(k_bar_reset, dim3(1), dim3(64), 0, st, bar);
  return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_mail_reset(unsigned* __restrict__ bar, MailWord* __restrict__ mail,
                                                       int64_t words) {
  if (blockIdx.x == 0) bar_clear(bar);
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < words) mail[k] = 0;
}

hipError_t fm_mail_reset(unsigned* bar, MailWord* mail, int64_t words, hipStream_t st) {
  hipLaunchKernelGGL(k_mail_reset, dim3(grid_for(words > 0 ? words : 1, kBlock)), dim3(kBlock), 0, st, bar, mail,
                     words);
  return hipGetLastError();
}

struct SolveArgs {
  float* params;
  float* m;
  float* v;
  const int32_t* cams;
  const void* W36;
  const int32_t* cam_ptr;
  const int32_t* cam_items;
  float* contrib;
  double* loss_part;
  double* rot;
  double* loss_trace;
  unsigned* bar;
  const int64_t* Z_dev;
  double inv_Z;
  int64_t P;
  int32_t N;
  int32_t K;
  double lr_rot, lr_t, log_frac;
  double b1, b2, eps;
  int64_t lr_step0, lr_total, adam_step0;
  const int32_t* pair_slot;
};

// Grid barrier of the pair loop: per-XCD (grid_sync) or flat (grid_barrier);
// `early` loads what no workgroup writes, during the wait where that can be.
template <bool XS, typename F>
__device__ inline void loop_sync(GridBar& gb, XcdSync& xs, F&& early) {
  if constexpr (XS) {
    grid_sync(gb.bar, xs, early);
  } else {
    grid_barrier(gb);
    early();
  }
}

template <typename WT, bool XS>
__global__ __launch_bounds__(kSolveBlock) void k_solve(SolveArgs a) {
  __shared__ double lds[kSolveBlock / 64];
  const double iz = a.Z_dev ? 1.0 / (double)(*a.Z_dev > 0 ? *a.Z_dev : 1) : a.inv_Z;
  const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t gsize = (int64_t)gridDim.x * blockDim.x;
  const int lane = threadIdx.x & 63;
  const int64_t gwave = gtid >> 6, nwaves = gsize >> 6;
  const WT* W36 = reinterpret_cast<const WT*>(a.W36);
  // static data of this thread's first two pairs (cameras and record slots)
  // and this row's first camera (its slot range), read once instead of once
  // per iteration
  const int ci0 = gtid < a.P ? a.cams[2 * gtid] : 0, cj0 = gtid < a.P ? a.cams[2 * gtid + 1] : 0;
  const int qi0 = gtid < a.P ? a.pair_slot[2 * gtid] : 0, qj0 = gtid < a.P ? a.pair_slot[2 * gtid + 1] : 0;
  const int64_t g1 = gtid + gsize;
  const int ci1 = g1 < a.P ? a.cams[2 * g1] : 0, cj1 = g1 < a.P ? a.cams[2 * g1 + 1] : 0;
  const int qi1 = g1 < a.P ? a.pair_slot[2 * g1] : 0, qj1 = g1 < a.P ? a.pair_slot[2 * g1 + 1] : 0;
  // the float32 Gram of the thread's first pair is loaded ahead of its pair
  // phase, in the wait of the barrier before it (186k pairs: 19.2 us an
  // iteration, 19.8 without; held through the launch it spills, 19.5; a
  // float64 Gram does not fit the registers)
  constexpr bool kHold = sizeof(WT) == 4;
  GramRegs<WT> w0{};
  auto load_first = [&] {
    if constexpr (kHold)
      if (gtid < a.P) load_gram(W36 + gtid * 36, w0);
  };
  load_first();
  // cameras 4 gwave + row, then strided by 4 nwaves
  const int row = lane >> 4, l16 = lane & 15, base = lane & ~15;
  const int64_t c_first = 4 * gwave + row, c_stride = 4 * nwaves;
  const int lo0 = c_first < a.N ? a.cam_ptr[c_first] : 0, hi0 = c_first < a.N ? a.cam_ptr[c_first + 1] : 0;
  GridBar gb = grid_bar(a.bar);
  XcdSync xs = {};
  if constexpr (XS) xs = xcd_register(gb);
  StepSched sch(a.log_frac, a.lr_step0, a.lr_total, a.adam_step0, a.b1, a.b2);
  for (int k = 0; k < a.K; ++k) {
    // iteration 0 runs Gram-Schmidt per pair; later iterations read the
    // rotations the camera phase stored with the updated parameters
    const double v = pair_phase_slots<kHold, WT>(a.params, k > 0 ? a.rot : nullptr, a.cams, a.pair_slot, W36, a.P,
                                                2.0 * iz, a.contrib, gtid, gsize, ci0, cj0, ci1, cj1, qi0, qj0, qi1,
                                                qj1, w0);
    if (a.loss_trace) {
      const double t = block_sum(v, lds);
      if (threadIdx.x == 0) trace_row(a.loss_part, gridDim.x, k)[blockIdx.x] = t;
    }
    loop_sync<XS>(gb, xs, [] {});
    if (a.loss_trace) trace_batch(a.loss_part, gridDim.x, k, a.K, iz, a.loss_trace, gwave, nwaves, lane);
    const double frac = sch.frac;
    const double bc1 = 1.0 - sch.p1, bc2 = 1.0 - sch.p2;
    sch.next();
    // the loop bound is uniform over the wavefront (rows past N idle), so
    // the row exchanges below always run with every lane present
    for (int64_t c0 = 4 * gwave; c0 < a.N; c0 += c_stride) {
      const int64_t c = c0 + row;
      const bool live = c < a.N;
      // parameters and moments first (they do not depend on the records),
      // so their loads overlap the record loads
      float p0 = 0.0f, mq = 0.0f, vq = 0.0f;
      // (m, v: only this lane reads and writes them during the launch)
      if (live && l16 < 9) {
        p0 = a.params[c * 9 + l16];
        mq = a.m[c * 9 + l16];
        vq = a.v[c * 9 + l16];
      }
      double acc6[6], acc[12];
      const bool first = c0 == 4 * gwave;
      const int lo = first ? lo0 : (live ? a.cam_ptr[c] : 0), hi = first ? hi0 : (live ? a.cam_ptr[c + 1] : 0);
      // Gram-Schmidt of the camera's own parameters ahead of the record
      // gather (it overlaps the record loads); a row without a camera has
      // zero parameters: keep its Gram-Schmidt away from 0/0 (its results
      // are not stored)
      double a1[3], a2[3], g[9];
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        a1[j] = (double)__shfl(p0, base + j);
        a2[j] = (double)__shfl(p0, base + 3 + j);
      }
      if (!live) a1[0] = a2[1] = 1.0;
      const Gs f = gs_forward(a1, a2);
      row_camera_sums_slots<kRowItems, float2>(lo, hi, a.contrib, lane, acc6);
      omega_grad(f, acc6, acc6 + 3, acc);
      gs_adjoint(acc, f, a2, g);
      // lanes 0..8 of the row update one parameter each
      float pq = 0.0f;
      if (live && l16 < 9) {
        const double lr = (l16 < 6 ? a.lr_rot : a.lr_t) * frac;
        pq = adam_update(p0, (float)pick9(g, l16), mq, vq, lr, a.b1, a.b2, a.eps, bc1, bc2);
        a.params[c * 9 + l16] = pq;
        a.m[c * 9 + l16] = mq;
        a.v[c * 9 + l16] = vq;
      }
      // rotation of the updated parameters for the next pair phase
      double n1[3], n2[3], R[3][3];
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        n1[j] = (double)__shfl(pq, base + j);
        n2[j] = (double)__shfl(pq, base + 3 + j);
      }
      if (!live) n1[0] = n2[1] = 1.0;
      gs_matrix(gs_forward(n1, n2), R);
      if (live && l16 < 9) {
        double rv = R[0][0];
#pragma unroll
        for (int j = 1; j < 9; ++j) rv = (l16 == j) ? R[j / 3][j % 3] : rv;
        a.rot[c * 9 + l16] = rv;
      }
    }
    loop_sync<XS>(gb, xs, load_first);
  }
}

// Camera-centric variant of the fused loop: one wavefront per camera; each
// lane evaluates one of the camera's pairs (its loss and the adjoint for the
// camera's own side, so every pair is evaluated twice, once from each end),
// the wavefront sums them in a fixed order and lanes 0..8 take the Adam
// step.  The parameters of the other cameras come from their mailboxes
// (mail_take), so an iteration has no grid barrier and leaves the caches
// alone: 100 iterations at 200 cameras 361 us, 527 with parameters and
// rotations exchanged through a grid barrier.  What is left is one
// wavefront's chain of float64 arithmetic (about 2.4 us an iteration) and the
// way of a store to another XCD's load.
struct CamSolveArgs {
  float* params;
  float* m;
  float* v;
  const int32_t* cams;
  const void* W36;
  const int32_t* cam_ptr;
  const int32_t* cam_items;
  MailWord* mail;      // [2, N, kMailWords]
  double* loss_part;   // [2 kTraceBatch, min(N, wavefronts)]
  double* loss_trace;
  unsigned* bar;
  const int64_t* Z_dev;
  double inv_Z;
  int64_t P;
  int32_t N;
  int32_t K;
  double lr_rot, lr_t, log_frac;
  double b1, b2, eps;
  int64_t lr_step0, lr_total, adam_step0;
};

// Gram-Schmidt of the parameters p0 held by lanes 0..5 of the wavefront (a2
// receives the second column's parameters).
__device__ inline Gs cam_gs(float p0, double a2[3]) {
  double a1[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    a1[j] = (double)__shfl(p0, j);
    a2[j] = (double)__shfl(p0, 3 + j);
  }
  return gs_forward(a1, a2);
}

// Incidence entry lo + q0 + lane of camera c and the camera's slot range; in
// lanes past the end (`live` false) the last entry, and for a camera without
// pairs or past N entry 0, so that what they point at can be read.
struct CamSlot {
  int lo, hi, item, other;
  bool live;
};

__device__ inline CamSlot cam_slot(const CamSolveArgs& a, int64_t c, int q0, int lane) {
  CamSlot s{0, 0, 0, 0, false};
  if (c < a.N) {
    s.lo = a.cam_ptr[c];
    s.hi = a.cam_ptr[c + 1];
    if (s.lo < s.hi) {
      const int q = s.lo + q0 + lane;
      s.live = q < s.hi;
      s.item = a.cam_items[s.live ? q : s.hi - 1];
      s.other = a.cams[(int64_t)s.item ^ 1];
    }
  }
  return s;
}

template <typename WT>
__global__ __launch_bounds__(kCamBlock) void k_solve_cam(CamSolveArgs a) {
  const double iz = a.Z_dev ? 1.0 / (double)(*a.Z_dev > 0 ? *a.Z_dev : 1) : a.inv_Z;
  const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t gsize = (int64_t)gridDim.x * blockDim.x;
  const int lane = threadIdx.x & 63;
  const int64_t gwave = gtid >> 6, nwaves = gsize >> 6;
  const int kq = lane < 9 ? lane : 8;
  const WT* W36 = reinterpret_cast<const WT*>(a.W36);
  const int64_t NM = (int64_t)a.N * kMailWords;
  constexpr unsigned kRecord = kMailWords * sizeof(MailWord);
  const unsigned mail_bytes = (unsigned)a.N * kRecord;
  const int64_t slots = nwaves < a.N ? nwaves : a.N;   // wavefronts with a camera
  // first records (buffer 0, tag 1)
  for (int64_t c = gwave; c < a.N; c += nwaves) {
    const float p0 = a.params[c * 9 + kq];
    if (lane < 9) mail_put(a.mail + c * kMailWords + lane, p0, 1u);
  }
  // static data, read once: this lane's first two incidence entries of the
  // wavefront's first camera and the Gram of the first of them, the lane's
  // first entry of the wavefront's second camera, both cameras' slot ranges
  const CamSlot s0 = cam_slot(a, gwave, 0, lane), s1 = cam_slot(a, gwave, 64, lane),
                n0 = cam_slot(a, gwave + nwaves, 0, lane);
  GramRegs<WT> w0{};
  if (s0.live) load_gram(W36 + (int64_t)(s0.item >> 1) * 36, w0);
  // the wavefront's first camera stays in registers for the launch: its
  // parameters, Adam moments and their Gram-Schmidt, carried from one
  // iteration's update to the next
  const bool own = gwave < a.N;
  float p_own = 0.0f, m_own = 0.0f, v_own = 0.0f;
  double a2_own[3] = {0.0, 1.0, 0.0};
  Gs f_own{};
  if (own) {
    p_own = a.params[gwave * 9 + kq];
    m_own = a.m[gwave * 9 + kq];
    v_own = a.v[gwave * 9 + kq];
    f_own = cam_gs(p_own, a2_own);
  }
  GridBar gb = grid_bar(a.bar);
  // a wait expired: the wavefront does no more than take part in its
  // workgroup's barriers, of which an untraced launch has none
  bool dead = false;
  StepSched sch(a.log_frac, a.lr_step0, a.lr_total, a.adam_step0, a.b1, a.b2);
  for (int k = 0; k < a.K; ++k) {
    MailWord* in = a.mail + (k & 1) * NM;
    MailWord* out = a.mail + ((k & 1) ^ 1) * NM;
    const unsigned tag = (unsigned)k + 1u;
    // the step's scalars before the wait (pinned there: sunk to their use
    // they would follow it)
    double lr = (lane < 6 ? a.lr_rot : a.lr_t) * sch.frac, ib1 = 1.0 / (1.0 - sch.p1), ib2 = 1.0 / (1.0 - sch.p2);
    sch.next();
    asm volatile("" : "+v"(lr), "+v"(ib1), "+v"(ib2));
    double lwave = 0.0;   // in lane kLossLane: the wavefront's loss
    // one camera: its parameters and moments
    // (lanes 9..63 hold entry 8; no other wavefront reads or writes them in
    // memory) and their Gram-Schmidt f.  All 64 lanes take part.
    auto camera = [&](auto first_cam, int64_t c, const CamSlot& held, float& p0, float& mq, float& vq,
                      const double (&a2)[3], const Gs& f) {
      double g[9], R[3][3], t[3];
      gs_matrix(f, R);
#pragma unroll
      for (int j = 0; j < 3; ++j) t[j] = (double)__shfl(p0, 6 + j);
      // this camera's side of each of its pairs: body-frame rotation
      // gradient (om for camera j, -om for camera i) and dL/dt
      double acc6[6], acc[12], lsum = 0.0;
#pragma unroll
      for (int j = 0; j < 6; ++j) acc6[j] = 0.0;
      auto add_pair = [&](int side, const float (&po)[9], const auto& w) {
        const double o1[3] = {(double)po[0], (double)po[1], (double)po[2]};
        const double o2[3] = {(double)po[3], (double)po[4], (double)po[5]};
        double Ro[3][3], tj[3], om[3], dti[3], dtj[3];
        gs_matrix(gs_forward(o1, o2), Ro);
        PairEval e;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          const double to = (double)po[6 + j];
          e.ti[j] = side ? to : t[j];
          tj[j] = side ? t[j] : to;
#pragma unroll
          for (int i = 0; i < 3; ++i) {
            e.Ri[j][i] = side ? Ro[j][i] : R[j][i];
            e.Rj[j][i] = side ? R[j][i] : Ro[j][i];
          }
        }
        pair_terms(e, tj, w);
        const double l = pair_adjoint(e, 2.0 * iz, om, dti, dtj);
        if (side == 0) lsum += l;   // each pair's loss once, from its first camera
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          acc6[j] += (double)(float)(side ? om[j] : -om[j]);
          acc6[3 + j] += (double)(float)(side ? dtj[j] : dti[j]);
        }
      };
      float po[9];
      if (first_cam.value && s0.lo < s0.hi) {
        mail_take(a.bar, in, mail_bytes, (unsigned)s0.other * kRecord, tag, s0.live, po, dead);
        if (s0.live) add_pair(s0.item & 1, po, w0);
      }
      // entries from memory, the first of these passes' held in `held`; the
      // Grams are on their way during the wait
      for (int q0 = first_cam.value ? 64 : 0; held.lo + q0 < held.hi; q0 += 64) {
        const CamSlot e = q0 == (first_cam.value ? 64 : 0) ? held : cam_slot(a, c, q0, lane);
        GramRegs<WT> w;
        load_gram(W36 + (int64_t)(e.item >> 1) * 36, w);
        mail_take(a.bar, in, mail_bytes, (unsigned)e.other * kRecord, tag, e.live, po, dead);
        if (e.live) add_pair(e.item & 1, po, w);
      }
      lwave += wave_sum6_loss(acc6, lsum, lane);
      omega_grad(f, acc6, acc6 + 3, acc);
      gs_adjoint(acc, f, a2, g);
      p0 = adam_update_inv(p0, (float)pick9(g, kq), mq, vq, lr, a.b1, a.b2, a.eps, ib1, ib2);
      if (lane < 9) mail_put(out + c * kMailWords + lane, p0, tag + 1u);
    };
    if (own && !dead) {
      camera(std::true_type{}, gwave, s1, p_own, m_own, v_own, a2_own, f_own);
      f_own = cam_gs(p_own, a2_own);
    }
    for (int64_t c = gwave + nwaves; c < a.N && !dead; c += nwaves) {
      float p0 = a.params[c * 9 + kq], mq = a.m[c * 9 + kq], vq = a.v[c * 9 + kq];
      double a2[3];
      const Gs f = cam_gs(p0, a2);
      camera(std::false_type{}, c, c == gwave + nwaves ? n0 : cam_slot(a, c, 0, lane), p0, mq, vq, a2, f);
      if (lane < 9) {
        a.params[c * 9 + lane] = p0;
        a.m[c * 9 + lane] = mq;
        a.v[c * 9 + lane] = vq;
      }
    }
    if (a.loss_trace) {
      if (lane == kLossLane && gwave < slots) store_wt(trace_row(a.loss_part, slots, k) + gwave, lwave);
      if (trace_due(k, a.K)) {
        grid_barrier_wt(gb);
        trace_batch(a.loss_part, slots, k, a.K, iz, a.loss_trace, gwave, nwaves, lane);
      }
    } else if (dead) {
      break;
    }
  }
  // the first camera's values, kept in registers during the launch
  if (own && lane < 9) {
    a.params[gwave * 9 + lane] = p_own;
    a.m[gwave * 9 + lane] = m_own;
    a.v[gwave * 9 + lane] = v_own;
  }
}

// Check mode after a fused solve: the final parameters and the loss trace
// finite, and no degenerate pair at the final poses.
static fm_status solve_checks(fm_ctx* ctx, fm_scene* s, const float* params, const double* loss_trace, int32_t K,
                              hipStream_t st) {
  if (!ctx->check) return FM_OK;
  fm_status rc = fm_check_finite(ctx, st, params, (int64_t)s->N * 9, false, FM_CHECK_PARAMS);
  if (rc == FM_OK) rc = fm_check_finite(ctx, st, loss_trace, K, true, FM_CHECK_LOSS);
  if (rc == FM_OK) rc = fm_launch_essentials(s, params, st);
  return rc;
}

// Co-resident workgroups of the fused loops: the smallest occupancy over
// every instantiation, times the CU count.
template <typename K>
static bool occ_min(K kernel, int block, int& per_cu) {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, block, 0) != hipSuccess) return false;
  if (n < per_cu) per_cu = n;
  return true;
}

int fm_solve_coop_blocks(fm_ctx* ctx, bool cam) {
  int per_cu = 1 << 20;
  const bool ok = cam ? occ_min(k_solve_cam<double>, kCamBlock, per_cu) && occ_min(k_solve_cam<float>, kCamBlock, per_cu)
                      : occ_min(k_solve<double, false>, kSolveBlock, per_cu) &&
                            occ_min(k_solve<float, false>, kSolveBlock, per_cu) &&
                            occ_min(k_solve<double, true>, kSolveBlock, per_cu) &&
                            occ_min(k_solve<float, true>, kSolveBlock, per_cu);
  return ok ? per_cu * ctx->num_cu : 0;
}

// Instantiation of the pair loop for the Gram dtype and the barrier kind
// (per-XCD from kXcdSyncMinBlocks workgroups on).
static const void* pair_loop_kernel(fm_dtype wdt, int64_t blocks) {
  const bool xs = blocks >= kXcdSyncMinBlocks;
  if (wdt == FM_F64) return xs ? (const void*)k_solve<double, true> : (const void*)k_solve<double, false>;
  return xs ? (const void*)k_solve<float, true> : (const void*)k_solve<float, false>;
}

extern "C" fm_status fm_epipolar_solve(fm_ctx* ctx, fm_scene* s, const void* W36, fm_dtype wdt, float* params,
                                       float* m, float* v, int32_t K, const fm_adam_cfg* cfg, double inv_Z,
                                       const int64_t* Z_dev, double* loss_trace, fm_stream stream) {
  if (!ctx) return FM_EINVAL;
  if (!s) return fm_fail(ctx, FM_EINVAL, "fm_epipolar_solve: scene is NULL");
  if (s->ctx != ctx) return fm_fail(ctx, FM_EINVAL, "fm_epipolar_solve: scene belongs to another context");
  fm_status rc = check_w(ctx, "fm_epipolar_solve", W36, wdt, s->P);
  if (rc != FM_OK) return rc;
  if (!cfg || (s->N > 0 && (!params || !m || !v)))
    return fm_fail(ctx, FM_EINVAL, "fm_epipolar_solve: NULL argument");
  if (K < 0) return fm_fail(ctx, FM_EINVAL, "fm_epipolar_solve: K < 0");
  if (cfg->lr_total_steps <= 0 || cfg->lr_step0 < 0 || cfg->adam_step0 < 0 || !(cfg->lr_final_frac > 0.0f) ||
      !(cfg->beta1 >= 0.0f && cfg->beta1 < 1.0f && cfg->beta2 >= 0.0f && cfg->beta2 < 1.0f && cfg->eps >= 0.0f))
    return fm_fail(ctx, FM_EINVAL, "fm_epipolar_solve: bad Adam configuration");
  if (!Z_dev && !(inv_Z >= 0.0)) return fm_fail(ctx, FM_EINVAL, "fm_epipolar_solve: inv_Z must be >= 0");
  if (K == 0) return FM_OK;
  FM_HIP_TRY(ctx, hipSetDevice(ctx->device));
  // about one pair per thread and one 16-lane row per camera, capped at 192
  // workgroups (each adds about 0.02 us to each of the two grid barriers per
  // iteration, measured, so past this size a second round of pairs per thread
  // or of cameras per row is cheaper than more workgroups), and at the
  // co-resident limit; at least as many as synchronise per XCD.  The graphs
  // that come here by themselves have 131k pairs, or over 1,024 cameras that
  // cost more camera by camera (cam_loop_wins): 4,000 cameras / 24k pairs 12.3
  // us per iteration at 128 workgroups, 15.3 at 125 (flat barrier), 37 at 16;
  // 20,000 / 40k 23.4 at 192, 25.4 at 128
  int64_t want = grid_for(s->P, kSolveBlock);
  const int64_t want_c = grid_for((int64_t)s->N * 16, kSolveBlock);
  if (want_c > want) want = want_c;
  if (want < kXcdSyncMinBlocks) want = kXcdSyncMinBlocks;
  if (want > 192) want = 192;
  if (cfg->blocks > 0) want = cfg->blocks;
  if (want < 1) want = 1;
  if (want > s->coop_blocks) want = s->coop_blocks;
  if (2 * kTraceBatch * want > s->loss_part_cap)
    return fm_fail(ctx, FM_ECOOP, "fm_epipolar_solve: loss workspace too small");
  SolveArgs a;
  a.params = params; a.m = m; a.v = v;
  a.cams = s->pair_cams; a.W36 = W36; a.cam_ptr = s->cam_ptr; a.cam_items = s->cam_items;
  a.contrib = s->contrib; a.loss_part = s->loss_part; a.rot = s->rot; a.loss_trace = loss_trace; a.Z_dev = Z_dev;
  a.bar = s->bar;
  a.inv_Z = inv_Z; a.P = s->P; a.N = s->N; a.K = K;
  a.lr_rot = cfg->lr_rot; a.lr_t = cfg->lr_t; a.log_frac = log((double)cfg->lr_final_frac);
  a.b1 = cfg->beta1; a.b2 = cfg->beta2; a.eps = cfg->eps;
  a.lr_step0 = cfg->lr_step0; a.lr_total = cfg->lr_total_steps; a.adam_step0 = cfg->adam_step0;
  a.pair_slot = s->pair_slot;
  void* args[] = {&a};
  // automatic grid where cam_loop_wins, or cfg->blocks < 0: the
  // camera-centric loop, no barrier in an iteration; a forced workgroup count
  // or any other graph (also one whose records a buffer descriptor does not
  // span) runs the pair loop.
  // Workgroups of two wavefronts while they fit one to a CU: the wavefronts'
  // scattered reads of the mailboxes spread over twice as many CUs (us per
  // iteration, two against four: 200 cameras 3.16 against 3.40, 500 of 73 pairs
  // 5.17 and 5.40, 512 of 180 pairs 9.2 and 9.9); past a workgroup per CU four
  // (600 cameras 3.6 against 6.7, 1,000 4.4 and 6.5).
  const int cam_threads = ((int64_t)s->N + 1) / 2 <= ctx->num_cu ? kCamBlock / 2 : kCamBlock;
  int64_t want_cam = grid_for((int64_t)s->N * 64, cam_threads);
  if (want_cam > s->coop_blocks_cam) want_cam = s->coop_blocks_cam;
  if (want_cam > ctx->num_cu) want_cam = ctx->num_cu;
  if ((cfg->blocks < 0 || (cfg->blocks == 0 && cam_loop_wins(s->N, s->P, s->max_pairs, ctx->num_cu))) &&
      2 * kTraceBatch * want_cam * (cam_threads / 64) <= s->loss_part_cap &&
      (int64_t)s->N * kMailWords * (int64_t)sizeof(MailWord) <= INT32_MAX) {
    CamSolveArgs ca;
    ca.params = params; ca.m = m; ca.v = v;
    ca.cams = s->pair_cams; ca.W36 = W36; ca.cam_ptr = s->cam_ptr; ca.cam_items = s->cam_items;
    ca.mail = s->mail; ca.loss_part = s->loss_part; ca.loss_trace = loss_trace; ca.bar = s->bar; ca.Z_dev = Z_dev;
    ca.inv_Z = inv_Z; ca.P = s->P; ca.N = s->N; ca.K = K;
    ca.lr_rot = a.lr_rot; ca.lr_t = a.lr_t; ca.log_frac = a.log_frac;
    ca.b1 = a.b1; ca.b2 = a.b2; ca.eps = a.eps;
    ca.lr_step0 = a.lr_step0; ca.lr_total = a.lr_total; ca.adam_step0 = a.adam_step0;
    void* cargs[] = {&ca};
    FM_HIP_TRY(ctx, fm_mail_reset(s->bar, s->mail, 2 * (int64_t)s->N * kMailWords, (hipStream_t)stream));
    {
    fm_timed timer(ctx, FM_K_SOLVE, (hipStream_t)stream);
    const void* kernel = wdt == FM_F64 ? (const void*)k_solve_cam<double> : (const void*)k_solve_cam<float>;
    hipError_t e = hipLaunchCooperativeKernel(kernel, dim3((unsigned)want_cam), dim3(cam_threads), cargs, 0,
                                              (hipStream_t)stream);
    if (e != hipSuccess) return fm_fail(ctx, FM_ECOOP, "cooperative launch failed: %s", hipGetErrorString(e));
    }
    return solve_checks(ctx, s, params, loss_trace, K, (hipStream_t)stream);
  }
  FM_HIP_TRY(ctx, fm_bar_reset(s->bar, (hipStream_t)stream));
  {
  fm_timed timer(ctx, FM_K_SOLVE, (hipStream_t)stream);
  hipError_t e = hipLaunchCooperativeKernel(pair_loop_kernel(wdt, want), dim3((unsigned)want), dim3(kSolveBlock),
                                            args, 0, (hipStream_t)stream);
  if (e != hipSuccess) return fm_fail(ctx, FM_ECOOP, "cooperative launch failed: %s", hipGetErrorString(e));
  }
  return solve_checks(ctx, s, params, loss_trace, K, (hipStream_t)stream);
}

extern "C" fm_status fm_solve_barrier_failures(fm_ctx* ctx, fm_scene* s, int64_t* failures) {
  if (!ctx) return FM_EINVAL;
  if (!s || !failures) return fm_fail(ctx, FM_EINVAL, "fm_solve_barrier_failures: NULL argument");
  if (s->ctx != ctx) return fm_fail(ctx, FM_EINVAL, "fm_solve_barrier_failures: scene belongs to another context");
  FM_HIP_TRY(ctx, hipSetDevice(ctx->device));
  FM_HIP_TRY(ctx, hipDeviceSynchronize());
  unsigned f = 0;
  FM_HIP_TRY(ctx, hipMemcpy(&f, s->bar + 96, sizeof(unsigned), hipMemcpyDeviceToHost));
  if (f) FM_HIP_TRY(ctx, hipMemset(s->bar + 96, 0, sizeof(unsigned)));
  *failures = (int64_t)f;
  return FM_OK;
}
