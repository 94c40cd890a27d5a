// Global rotation averaging (FastMap, arXiv 2505.04612, Sec. 3.3 "Global
// Rotation": eq. rotation-objective with the geodesic distance, the 6D
// rotation parameterisation) on a scene's pair graph.
//
// The per-pair records are [P, 24] floats: for each side of the pair dL/dR as
// 3x3 row-major and three unused entries.  Parameters
// are (a1, a2) per camera, [N, 6].
#include <algorithm>

#include "fm_internal.h"

#include <cmath>

namespace {

// One pair's geodesic term and its record, float64.  With Q = R^{i->j},
// M = R_j^T Q R_i, c = (tr M - 1)/2 and d = arccos(c) (c clipped to
// [-1, 1]): dd/dc = -1/sqrt(1 - c^2) (0 where |c| = 1), dc/dR_j = Q R_i / 2
// = R_j M / 2 and dc/dR_i = Q^T R_j / 2 = R_i M^T / 2; both scaled by invP.
// The records keep only the part of these that moves along the rotation
// group (R_j K and -R_i K with K = (M - M^T)/2): the rest is annihilated by
// the Gram-Schmidt adjoint, and it grows like 1/d, so a float32 record of
// the full matrix would lose the O(1) tangent part to rounding when d is
// small.  Returns d.
__device__ inline double ra_pair(const double Ri[3][3], const double Rj[3][3], const float* __restrict__ q,
                                 double invP, float* __restrict__ rec) {
  double Q[3][3], QRi[3][3], M[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) Q[a][b] = (double)q[3 * a + b];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) QRi[a][b] = Q[a][0] * Ri[0][b] + Q[a][1] * Ri[1][b] + Q[a][2] * Ri[2][b];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) M[a][b] = Rj[0][a] * QRi[0][b] + Rj[1][a] * QRi[1][b] + Rj[2][a] * QRi[2][b];
  double c = 0.5 * (M[0][0] + M[1][1] + M[2][2] - 1.0);
  const bool inside = c > -1.0 && c < 1.0;
  c = c > 1.0 ? 1.0 : (c < -1.0 ? -1.0 : c);
  if (rec) {
    const double half_gc = inside ? -0.5 * invP / sqrt(1.0 - c * c) : 0.0;
    double K[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) K[a][b] = 0.5 * (M[a][b] - M[b][a]);
    float gi[12], gj[12];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        gj[3 * a + b] = (float)(half_gc * (Rj[a][0] * K[0][b] + Rj[a][1] * K[1][b] + Rj[a][2] * K[2][b]));
        gi[3 * a + b] = (float)(-half_gc * (Ri[a][0] * K[0][b] + Ri[a][1] * K[1][b] + Ri[a][2] * K[2][b]));
      }
    gi[9] = gi[10] = gi[11] = 0.0f;
    gj[9] = gj[10] = gj[11] = 0.0f;
    float4* dst = reinterpret_cast<float4*>(rec);
    dst[0] = make_float4(gi[0], gi[1], gi[2], gi[3]);
    dst[1] = make_float4(gi[4], gi[5], gi[6], gi[7]);
    dst[2] = make_float4(gi[8], gi[9], gi[10], gi[11]);
    dst[3] = make_float4(gj[0], gj[1], gj[2], gj[3]);
    dst[4] = make_float4(gj[4], gj[5], gj[6], gj[7]);
    dst[5] = make_float4(gj[8], gj[9], gj[10], gj[11]);
  }
  return acos(c);
}

__device__ inline void rot6(const float* __restrict__ p6, int c, double R[3][3]) {
  double a1[3], a2[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    a1[k] = (double)p6[6 * (int64_t)c + k];
    a2[k] = (double)p6[6 * (int64_t)c + 3 + k];
  }
  gs_matrix(gs_forward(a1, a2), R);
}

__device__ inline void load_rot(const double* __restrict__ rot, int c, double R[3][3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) R[a][b] = rot[9 * (int64_t)c + 3 * a + b];
}

// ------------------------------------------------------------------ standalone loss + gradient

__global__ __launch_bounds__(kBlock) void k_ra_pair(const float* __restrict__ params, const int32_t* __restrict__ cams,
                                                    const float* __restrict__ Rrel, int64_t P, double invP,
                                                    float* __restrict__ contrib, double* __restrict__ part) {
  __shared__ double lds[kBlock / 64];
  const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, gsize = (int64_t)gridDim.x * blockDim.x;
  double v = 0.0;
  for (int64_t n = gtid; n < P; n += gsize) {
    double Ri[3][3], Rj[3][3];
    rot6(params, cams[2 * n], Ri);
    rot6(params, cams[2 * n + 1], Rj);
    v += ra_pair(Ri, Rj, Rrel + 9 * n, invP, contrib + 24 * n);
  }
  const double t = block_sum(v, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

__global__ __launch_bounds__(kBlock) void k_ra_camera(const float* __restrict__ params,
                                                      const int32_t* __restrict__ cam_ptr,
                                                      const int32_t* __restrict__ cam_items,
                                                      const float* __restrict__ contrib, int32_t N,
                                                      float* __restrict__ grad) {
  const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t c = gtid >> 4;
  const int lane = threadIdx.x & 63, l16 = lane & 15;
  if (c >= N) return;   // whole rows leave together: the row exchanges stay within live rows
  double acc[12];
  row_camera_sums(row_list(cam_ptr, cam_items, (int)c, l16), cam_items, contrib, lane, acc);
  double a1[3], a2[3], g[9];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    a1[k] = (double)params[6 * c + k];
    a2[k] = (double)params[6 * c + 3 + k];
  }
  gs_adjoint(acc, a1, a2, g);
  if (l16 < 6) grad[6 * c + l16] = (float)pick9(g, l16);
}

__global__ void k_ra_loss_final(const double* __restrict__ part, int64_t nblocks, double invP, double* __restrict__ loss) {
  if (threadIdx.x != 0) return;
  double s = 0.0;
  for (int64_t b = 0; b < nblocks; ++b) s += part[b];
  *loss = s * invP;
}

// ------------------------------------------------------------------ fused persistent loop

struct RaArgs {
  float* params;
  float* m;
  float* v;
  const int32_t* cams;
  const float* Rrel;
  const int32_t* cam_ptr;
  const int32_t* cam_items;
  float* contrib;
  double* rot;
  double* part;
  double* trace;
  unsigned* bar;
  int64_t P;
  int32_t N;
  int32_t K;
  double invP, lr, log_frac, b1, b2, eps;
  int64_t lr_step0, lr_total, adam_step0;
};

// Rotation of camera c from the parameters p0 held by lanes 0..5 of its row,
// stored by lanes 0..8 (written through to memory if WTS).
template <bool WTS = false>
__device__ inline void ra_store_rot(double* __restrict__ rot, int64_t c, float p0, int base, int l16, bool live) {
  double a1[3], a2[3], R[3][3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    a1[j] = (double)__shfl(p0, base + j);
    a2[j] = (double)__shfl(p0, base + 3 + j);
  }
  if (!live) a1[0] = a2[1] = 1.0;   // a row without a camera: keep Gram-Schmidt away from 0/0
  gs_matrix(gs_forward(a1, a2), R);
  if (live && l16 < 9) {
    double rv = R[0][0];
#pragma unroll
    for (int j = 1; j < 9; ++j) rv = (l16 == j) ? R[j / 3][j % 3] : rv;
    if constexpr (WTS)
      store_wt(&rot[c * 9 + l16], rv);
    else
      rot[c * 9 + l16] = rv;
  }
}

__global__ __launch_bounds__(kSolveBlock) void k_ra_solve(RaArgs a) {
  GridBar gb = grid_bar(a.bar);
  __shared__ double lds[kSolveBlock / 64];
  const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t gsize = (int64_t)gridDim.x * blockDim.x;
  const int lane = threadIdx.x & 63;
  const int64_t gwave = gtid >> 6, nwaves = gsize >> 6;
  const int row = lane >> 4, l16 = lane & 15, base = lane & ~15;
  const int64_t c_first = 4 * gwave + row, c_stride = 4 * nwaves;
  // rotations of the initial parameters
  for (int64_t c0 = 4 * gwave; c0 < a.N; c0 += c_stride) {
    const int64_t c = c0 + row;
    const bool live = c < a.N;
    const float p0 = (live && l16 < 6) ? a.params[6 * c + l16] : 0.0f;
    ra_store_rot(a.rot, c, p0, base, l16, live);
  }
  // static data of this thread's first pair and this row's first camera
  int ci0 = 0, cj0 = 0;
  if (gtid < a.P) {
    ci0 = a.cams[2 * gtid];
    cj0 = a.cams[2 * gtid + 1];
  }
  RowList L0 = {0, 0, {-1, -1, -1, -1}};
  if (c_first < a.N) L0 = row_list(a.cam_ptr, a.cam_items, (int)c_first, l16);
  grid_barrier(gb);
  StepSched sch(a.log_frac, a.lr_step0, a.lr_total, a.adam_step0, a.b1, a.b2);
  for (int k = 0; k < a.K; ++k) {
    double v = 0.0;
    for (int64_t n = gtid; n < a.P; n += gsize) {
      double Ri[3][3], Rj[3][3];
      load_rot(a.rot, n == gtid ? ci0 : a.cams[2 * n], Ri);
      load_rot(a.rot, n == gtid ? cj0 : a.cams[2 * n + 1], Rj);
      v += ra_pair(Ri, Rj, a.Rrel + 9 * n, a.invP, a.contrib + 24 * n);
    }
    if (a.trace) {
      const double t = block_sum(v, lds);
      if (threadIdx.x == 0) a.part[blockIdx.x] = t;
    }
    grid_barrier(gb);
    if (a.trace && gtid == 0) {
      double s = 0.0;
      for (int b = 0; b < (int)gridDim.x; ++b) s += a.part[b];
      a.trace[k] = s * a.invP;
    }
    const double lr = a.lr * sch.frac;
    const double bc1 = 1.0 - sch.p1, bc2 = 1.0 - sch.p2;
    sch.next();
    // the loop bound is uniform over the wavefront (rows past N idle), so
    // the row exchanges always run with every lane present
    for (int64_t c0 = 4 * gwave; c0 < a.N; c0 += c_stride) {
      const int64_t c = c0 + row;
      const bool live = c < a.N;
      float p0 = 0.0f, mq = 0.0f, vq = 0.0f;
      if (live && l16 < 6) {
        p0 = a.params[6 * c + l16];
        mq = a.m[6 * c + l16];
        vq = a.v[6 * c + l16];
      }
      double acc[12];
      const RowList L = c0 == 4 * gwave ? L0 : (live ? row_list(a.cam_ptr, a.cam_items, (int)c, l16)
                                                     : RowList{0, 0, {-1, -1, -1, -1}});
      row_camera_sums(L, a.cam_items, a.contrib, lane, acc);
      double a1[3], a2[3], g[9];
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        a1[j] = (double)__shfl(p0, base + j);
        a2[j] = (double)__shfl(p0, base + 3 + j);
      }
      if (!live) a1[0] = a2[1] = 1.0;
      gs_adjoint(acc, a1, a2, g);
      float pq = 0.0f;
      if (live && l16 < 6) {
        pq = adam_update(p0, (float)pick9(g, l16), mq, vq, lr, a.b1, a.b2, a.eps, bc1, bc2);
        a.params[6 * c + l16] = pq;
        a.m[6 * c + l16] = mq;
        a.v[6 * c + l16] = vq;
      }
      ra_store_rot(a.rot, c, pq, base, l16, live);
    }
    grid_barrier(gb);
  }
}

// Camera-by-camera variant of the loop (the automatic choice): one
// wavefront per camera; each lane evaluates one
// of the camera's pairs and keeps its own side of the record (float32, as
// the records are), the wavefront sums them in a fixed order and lanes 0..5
// take the Adam steps.  No records are exchanged, so an iteration needs one
// grid barrier; the parameters and rotations other wavefronts read are
// double-buffered by iteration parity.
struct RaCamArgs {
  float* params;       // buffer 0 [N, 6] (the caller's)
  float* alt;          // buffer 1 [N, 6]
  float* m;
  float* v;
  const int32_t* cams;
  const float* Rrel;
  const int32_t* cam_ptr;
  const int32_t* cam_items;
  double* rot;         // [2, N, 9]
  double* part;        // [2, gridDim.x]
  double* trace;
  unsigned* bar;
  int64_t P;
  int32_t N;
  int32_t K;
  double invP, lr, log_frac, b1, b2, eps;
  int64_t lr_step0, lr_total, adam_step0;
};

// Static data of one incidence entry: the entry (pair << 1 | side), both
// cameras and the pair's relative rotation.
struct RaEntry {
  int item, ci, cj;
  float q[9];
};

__device__ inline RaEntry ra_entry(const RaCamArgs& a, int q) {
  RaEntry e;
  e.item = a.cam_items[q];
  const int64_t n = e.item >> 1;
  e.ci = a.cams[2 * n];
  e.cj = a.cams[2 * n + 1];
#pragma unroll
  for (int k = 0; k < 9; ++k) e.q[k] = a.Rrel[9 * n + k];
  return e;
}

__global__ __launch_bounds__(kSolveBlock) void k_ra_solve_cam(RaCamArgs a) {
  GridBar gb = grid_bar(a.bar);
  __shared__ double lds[kSolveBlock / 64];
  const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t gsize = (int64_t)gridDim.x * blockDim.x;
  const int lane = threadIdx.x & 63;
  const int64_t gwave = gtid >> 6, nwaves = gsize >> 6;
  const int kq = lane < 6 ? lane : 5;
  const int64_t NR = (int64_t)a.N * 9;
  // rotations of the initial parameters (buffer 0)
  for (int64_t c = gwave; c < a.N; c += nwaves) ra_store_rot(a.rot, c, a.params[6 * c + kq], 0, lane, true);
  grid_barrier(gb);
  // static data of the first 64 incidence entries of this wavefront's first
  // camera (one per lane) and its slot range, read once for the launch
  RaEntry e0{};
  int lo0 = 0, hi0 = 0;
  if (gwave < a.N) {
    lo0 = a.cam_ptr[gwave];
    hi0 = a.cam_ptr[gwave + 1];
    if (lo0 + lane < hi0) e0 = ra_entry(a, lo0 + lane);
  }
  StepSched sch(a.log_frac, a.lr_step0, a.lr_total, a.adam_step0, a.b1, a.b2);
  for (int k = 0; k < a.K; ++k) {
    const int rb = k & 1;
    const float* pr = rb ? a.alt : a.params;
    float* pw = rb ? a.params : a.alt;
    const double* rr = a.rot + rb * NR;
    double* rw = a.rot + (rb ^ 1) * NR;
    const double lr = a.lr * sch.frac;
    const double bc1 = 1.0 - sch.p1, bc2 = 1.0 - sch.p2;
    sch.next();
    double lsum = 0.0;
    // the loop bound is uniform over the wavefront, so the wavefront sums
    // run with every lane present
    for (int64_t c = gwave; c < a.N; c += nwaves) {
      const int lo = c == gwave ? lo0 : a.cam_ptr[c], hi = c == gwave ? hi0 : a.cam_ptr[c + 1];
      const float p0 = pr[6 * c + kq];
      float mq = a.m[6 * c + kq], vq = a.v[6 * c + kq];
      double acc[12];
#pragma unroll
      for (int j = 0; j < 12; ++j) acc[j] = 0.0;
      for (int q = lo + lane; q < hi; q += 64) {
        // the lane's first entry of the wavefront's first camera from
        // registers (read once per launch), the others from memory
        RaEntry e;
        if (c == gwave && q == lo + lane)
          e = e0;
        else
          e = ra_entry(a, q);
        const int side = e.item & 1;
        double Ri[3][3], Rj[3][3];
        load_rot(rr, e.ci, Ri);
        load_rot(rr, e.cj, Rj);
        float rec[24];
        const double d = ra_pair(Ri, Rj, e.q, a.invP, rec);
        if (side == 0) lsum += d;   // each pair's term once, from its first camera
#pragma unroll
        for (int j = 0; j < 12; ++j) acc[j] += (double)(side ? rec[12 + j] : rec[j]);
      }
      wave_sum12(acc, lane);
      double a1[3], a2[3], g[9];
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        a1[j] = (double)__shfl(p0, j);
        a2[j] = (double)__shfl(p0, 3 + j);
      }
      gs_adjoint(acc, a1, a2, g);
      const float pq = adam_update(p0, (float)pick9(g, kq), mq, vq, lr, a.b1, a.b2, a.eps, bc1, bc2);
      // parameters, rotations and loss partials are read by other
      // workgroups after the barrier: written through to memory
      if (lane < 6) {
        store_wt(&pw[6 * c + lane], pq);
        a.m[6 * c + lane] = mq;
        a.v[6 * c + lane] = vq;
      }
      ra_store_rot<true>(rw, c, pq, 0, lane, true);
    }
    if (a.trace) {
      const double t = block_sum(lsum, lds);
      if (threadIdx.x == 0) store_wt(&a.part[rb * gridDim.x + blockIdx.x], t);
    }
    grid_barrier_wt(gb);
    if (a.trace && gtid == 0) {
      double t = 0.0;
      for (int b = 0; b < (int)gridDim.x; ++b) t += a.part[rb * gridDim.x + b];
      a.trace[k] = t * a.invP;
    }
  }
  // after an odd number of iterations the latest parameters are in buffer 1
  if (a.K & 1) {
    for (int64_t c = gwave; c < a.N; c += nwaves)
      if (lane < 6) a.params[6 * c + lane] = a.alt[6 * c + lane];
  }
}

// ------------------------------------------------------------------ initialisation (column-wise least squares)

// The quadratic forms of the appendix on rotation initialisation, as an
// operator on stacked 3-vectors v [N,3]:
//   (A v)_c = sum over pairs n = (i, j) containing c of
//             v_j - Q v_i          (c = j),
//             Q^T Q v_i - Q^T v_j  (c = i),
// which is x^T A x = sum_n |x_j - Q x_i|^2; the second-column problem uses
// alpha A + beta diag(u_c u_c^T) with alpha = 1/P, beta = 1/N and u the
// first columns.  The smallest eigenvector comes from Lanczos with full
// reorthogonalisation, the smallest eigenpair of the tridiagonal matrix
// (multisection on the Sturm count, twisted factorisation) and the Ritz
// vector.
//
// A step is a chain of grid-wide reductions, so what bounds it is the number of
// grid barriers and the memory rounds between them.  Each workgroup owns the
// rows of consecutive cameras and keeps its rows of the basis in LDS (what
// does not fit, in memory); it forms its rows of the operator's image and the
// partial dots with its basis rows (one barrier: the dots' partials), then
// updates its rows and their norm (one barrier: the new vector and the norm's
// partials).  Before the dots, the two terms known without a reduction are
// taken off: beta_{k-1} q_{k-1} and, as the diagonal entry varies little from
// step to step, alpha_{k-1} q_k.  One pass of classical Gram-Schmidt then
// leaves the vector orthogonal to rounding unless its norm falls below half
// of what it was (the Daniel-Gragg-Kaufman-Stewart test); only then a second
// pass runs.  (With the image itself, whose q_k part is several times the
// rest, a single pass loses orthogonality by that factor every step.)  Every
// workgroup holds the tridiagonal matrix and finds its eigenpair itself, so
// that needs no barrier.
//
// Both columns, against the form with two unconditional passes, the basis in
// memory, seven barriers a step, and one thread's bisection and pivoted inverse
// iteration every 10 steps: 200 cameras, 4,849 pairs 6.52 -> 1.08 ms
// (0.97 with the exchanges by mailbox, see k_ra_lanczos); 1,000
// cameras 38.3 -> 4.7; 5,000 cameras, 209k pairs 166.5 -> 12.9.

constexpr int kLzBlock = 512;           // threads per workgroup
constexpr int kLzWaves = kLzBlock / 64;
// Workgroups up to which the exchanges go by mailbox: everyone reads everyone's
// dots past the caches, whose cost grows with their square (8 % are left of the
// gain at 63).
constexpr int kLzMailBlocks = 64;
constexpr int kLzMaxBlocks = 160;       // workgroups of the automatic grid, at most
constexpr int kLzMisc = 64 + kLzBlock;  // doubles of small LDS scratch
// Lanczos steps between convergence checks, and the relative residual
// bound |beta_k s_k| / |T| below which the Ritz pair is taken as converged.
constexpr int kLzCheck = 10;
constexpr int kLzMaxSteps = 4096;
constexpr double kLzTol = 1e-11;
// Steps and rows per workgroup up to which a workgroup's vectors and
// tridiagonal matrix stay in LDS (the LDS variant; the other one keeps all of
// them in memory).
constexpr int kLzLdsSteps = 1024;
constexpr int kLzLdsRows = 3072;

struct LzArgs {
  const int32_t* cams;
  const float* Rrel;
  const int32_t* cam_ptr;
  const int32_t* cam_items;
  const double* start;   // [2, n]
  double* V;             // [m + 1 - lv, n] basis rows past the LDS
  double* wbuf;          // [n] the current vector before its scaling
  double* part_h;        // [blocks, lz_hrow(m)] partial dots
  double* part_n;        // [blocks, kLzWaves] partial squared norms
  MailWord* mail;        // the three of them as mailboxes (two words a value)
  double* gws;           // [blocks, lz_work(rows, m)] (the memory variant)
  float* params;         // [N, 6]
  double* info;          // [4] or null: Ritz value and steps of each column
  unsigned* bar;
  int64_t n;
  int32_t N, m;
  int32_t nc;            // cameras per workgroup
  int32_t lv;            // basis vectors held in LDS
  double inv_P, inv_N;
};

// Row of a workgroup's partial dots: whole 128-byte lines, so that workgroups
// on different XCDs never write to the same one.
__host__ __device__ inline int64_t lz_hrow(int64_t m) { return (m + 2 + 15) / 16 * 16; }

// Doubles of one workgroup's vectors and tridiagonal matrix.
__host__ __device__ inline int64_t lz_work(int64_t rows, int64_t m) { return 3 * rows + 5 * m; }

// Reciprocal by two Newton steps on the hardware estimate (about an ulp).
__device__ inline double lz_rcp(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  return fma(r, fma(-d, r, 1.0), r);
}

// The value of lane `src` of every lane (uniform).
__device__ inline double lane_d(double v, int src) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, src), hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Wave-wide reductions, the same in every lane: DPP inside the 16-lane rows,
// then the four rows' values by lane reads (short chains: both are on the
// steps' critical path).
template <typename F>
__device__ inline double wave_reduce_d(double v, F f) {
  v = f(v, dpp_mov_d<0xB1>(v));    // quad_perm xor 1
  v = f(v, dpp_mov_d<0x4E>(v));    // quad_perm xor 2
  v = f(v, dpp_mov_d<0x141>(v));   // row_half_mirror
  v = f(v, dpp_mov_d<0x140>(v));   // row_mirror
  return f(f(lane_d(v, 0), lane_d(v, 16)), f(lane_d(v, 32), lane_d(v, 48)));
}

__device__ inline double wave_min_d(double v) {
  return wave_reduce_d(v, [](double x, double y) { return fmin(x, y); });
}

__device__ inline double wave_sum_d(double v) {
  return wave_reduce_d(v, [](double x, double y) { return x + y; });
}

// Smallest eigenpair of the symmetric tridiagonal matrix with diagonal
// al [m] and off-diagonal be [m - 1], by a whole workgroup: s [m] receives
// the unit eigenvector (its entries' sum made nonnegative), the eigenvalue is
// returned in every thread.  dp, dm [m]: scratch.
//   1. Multisection: four wavefronts evaluate the Sturm sequence of leading
//      principal minors of T - x (a sign change means an eigenvalue below x)
//      at 256 points of the interval, so each pass narrows it 257-fold.  The
//      sequence has no division: one FMA per row on the critical path, both
//      members scaled by a power of two every eight rows.
//   2. Twice: the forward and backward LDL^T factorisations of T - theta (two
//      lanes, one each), the twist with the smallest |gamma|, the eigenvector
//      from their ratios, and the Rayleigh correction gamma_r / |z|^2.
__device__ inline double lz_tridiag(const double* al, const double* be, int m, double* dp, double* dm, double* s,
                                    int* misc) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double lo = INFINITY, hi = INFINITY;   // hi: of the negated upper bounds
  for (int i = lane; i < m; i += 64) {
    const double r = (i > 0 ? fabs(be[i - 1]) : 0.0) + (i + 1 < m ? fabs(be[i]) : 0.0);
    lo = fmin(lo, al[i] - r);
    hi = fmin(hi, -(al[i] + r));
  }
  lo = wave_min_d(lo);
  hi = -wave_min_d(hi);
  // dm: squares of the off-diagonal entries, shifted to the row they enter
  for (int i = threadIdx.x; i < m; i += kLzBlock) dm[i] = i > 0 ? be[i - 1] * be[i - 1] : 0.0;
  __syncthreads();
  constexpr int kPts = 256;
  constexpr double kPart = 1.0 / (kPts + 1);
  for (int it = 0; it < 32 && hi - lo > 1e-15 * fmax(1.0, fabs(lo) + fabs(hi)); ++it) {
    const double w = hi - lo;
    if (wave < kPts / 64) {
      const double x = lo + w * (kPart * (64 * wave + lane + 1));
      int signs = 0;               // sign bit: a change so far
      double p1 = 1.0, p2 = 0.0;   // minors i - 1 and i - 2
      auto row = [&](double ai, double b2) {
        const double p = fma(ai - x, p1, -(b2 * p2));
        signs |= __double2hiint(p) ^ __double2hiint(p1);
        p2 = p1;
        p1 = p;
      };
      int i = 0;
      for (; i + 8 <= m; i += 8) {
        double av[8], bv[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          av[q] = al[i + q];
          bv[q] = dm[i + q];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) row(av[q], bv[q]);
        const int e = -__builtin_amdgcn_frexp_exp(fmax(fabs(p1), fabs(p2)));
        p1 = ldexp(p1, e);
        p2 = ldexp(p2, e);
      }
      for (; i < m; ++i) row(al[i], dm[i]);
      const unsigned long long bal = __ballot(signs < 0);
      if (lane == 0) misc[(it & 1) * 4 + wave] = bal ? 64 * wave + __builtin_ctzll(bal) : kPts;
    }
    __syncthreads();
    int f = kPts;   // the first point above the smallest eigenvalue
#pragma unroll
    for (int q = 0; q < kPts / 64; ++q) f = min(f, misc[(it & 1) * 4 + q]);
    const double nhi = f < kPts ? lo + w * (kPart * (f + 1)) : hi;
    const double nlo = f > 0 ? lo + w * (kPart * f) : lo;
    if (!(nhi - nlo < w)) break;
    lo = nlo;
    hi = nhi;
  }
  double theta = 0.5 * (lo + hi);
  for (int round = 0; round < 2; ++round) {
    __syncthreads();
    if (wave == 0 && lane < 2) {
      // lane 0 forward (rows 0, 1, ...), lane 1 backward (rows m - 1, ...); a
      // pivot of exactly 0 becomes 1e-300
      double* out = lane ? dm + (m - 1) : dp;
      const double* av = lane ? al + (m - 1) : al;
      const double* bv = lane ? be + (m - 2) : be;   // couples row q with row q + 1 in this direction
      const int step = lane ? -1 : 1;
      double d = av[0] - theta + 1e-300;
      out[0] = d;
      int q = 1;
      auto row = [&](double ai, double b) {
        d = fma(-(b * b), lz_rcp(d), ai - theta) + 1e-300;
        return d;
      };
      for (; q + 4 <= m; q += 4) {
        double a4[4], b4[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          a4[t] = av[(q + t) * step];
          b4[t] = bv[(q + t - 1) * step];
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) out[(q + t) * step] = row(a4[t], b4[t]);
      }
      for (; q < m; ++q) out[q * step] = row(av[q * step], bv[(q - 1) * step]);
    }
    __syncthreads();
    // the twist: every wavefront finds it (smallest |gamma|, lowest index)
    double g = INFINITY;
    for (int i = lane; i < m; i += 64) g = fmin(g, fabs(dp[i] + dm[i] - (al[i] - theta)));
    g = wave_min_d(g);
    int r = 0;   // stays 0 if every gamma is NaN
    for (int i0 = 0; i0 < m; i0 += 64) {
      const int i = i0 + lane;
      const unsigned long long at = __ballot(i < m && fabs(dp[i < m ? i : 0] + dm[i < m ? i : 0] - (al[i < m ? i : 0] - theta)) == g);
      if (at) {
        r = i0 + __builtin_ctzll(at);
        break;
      }
    }
    const double gamma = dp[r] + dm[r] - (al[r] - theta);
    __syncthreads();
    for (int i = threadIdx.x; i < m; i += kLzBlock) {
      dp[i] = i + 1 < m ? -be[i] * lz_rcp(dp[i]) : 0.0;
      dm[i] = i > 0 ? -be[i - 1] * lz_rcp(dm[i]) : 0.0;
    }
    __syncthreads();
    if (wave == 0 && lane < 2) {
      const int step = lane ? 1 : -1, count = lane ? m - 1 - r : r;
      const double* ratio = (lane ? dm : dp) + r + step;
      double* out = s + r + step;
      double z = 1.0;
      if (lane == 0) s[r] = 1.0;
      int q = 0;
      for (; q + 8 <= count; q += 8) {
        double t8[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) t8[t] = ratio[(q + t) * step];
#pragma unroll
        for (int t = 0; t < 8; ++t) out[(q + t) * step] = z *= t8[t];
      }
      for (; q < count; ++q) out[q * step] = z *= ratio[q * step];
    }
    __syncthreads();
    double n2 = 0.0;
    for (int i = lane; i < m; i += 64) n2 += s[i] * s[i];
    n2 = wave_sum_d(n2);
    theta += gamma / n2;
  }
  double n2 = 0.0, sum = 0.0;
  for (int i = lane; i < m; i += 64) {
    n2 += s[i] * s[i];
    sum += s[i];
  }
  n2 = wave_sum_d(n2);
  sum = wave_sum_d(sum);
  // (a matrix that is not finite has no eigenvector: its vector is NaN too)
  const double sc = isnan(theta) ? theta : (sum < 0.0 ? -1.0 : 1.0) / sqrt(n2);
  __syncthreads();
  for (int i = threadIdx.x; i < m; i += kLzBlock) s[i] *= sc;
  __syncthreads();
  return theta;
}

// One entry of a camera's incidence list as the operator reads it.
struct LzEntry {
  int other;    // the pair's other camera; -1: none
  int is_j;     // this camera is the pair's second one
  float Q[9];
};

__device__ inline LzEntry lz_entry(const LzArgs& a, int q) {
  LzEntry e;
  const int item = a.cam_items[q];
  const int64_t n = item >> 1;
  e.is_j = item & 1;
  e.other = a.cams[2 * n + (e.is_j ? 0 : 1)];
#pragma unroll
  for (int k = 0; k < 9; ++k) e.Q[k] = a.Rrel[9 * n + k];
  return e;
}

// This entry's term of (A v)_c, v_c = vc, v_other = vo, added to y.
__device__ inline void lz_term(const LzEntry& e, const double vc[3], const double vo[3], double y[3]) {
  double Q[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) Q[k] = (double)e.Q[k];
  if (e.is_j) {
    // v_j - Q v_i
#pragma unroll
    for (int r = 0; r < 3; ++r) y[r] += vc[r] - (Q[3 * r] * vo[0] + Q[3 * r + 1] * vo[1] + Q[3 * r + 2] * vo[2]);
  } else {
    // Q^T (Q v_i - v_j)
    double t[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) t[r] = Q[3 * r] * vc[0] + Q[3 * r + 1] * vc[1] + Q[3 * r + 2] * vc[2] - vo[r];
#pragma unroll
    for (int k = 0; k < 3; ++k) y[k] += Q[k] * t[0] + Q[3 + k] * t[1] + Q[6 + k] * t[2];
  }
}

// MAIL (few workgroups): the vector, the dots and the norms go from workgroup
// to workgroup as tagged mailbox values instead of through memory and a grid
// barrier.  One set of them does: a workgroup publishes an exchange only after
// it has taken the one before from every workgroup, and each of these had by
// then taken what is overwritten (the dots before the norms, the vector before
// the dots).  300 steps at most: 20 cameras 549 -> 473 us, 200 1,190 -> 973, 500 2,330
// -> 1,871, 1,000 (63 workgroups) 4,312 -> 3,979.
template <bool GL, bool MAIL>
__global__ __launch_bounds__(kLzBlock) void k_ra_lanczos(LzArgs a) {
  extern __shared__ double lds[];
  GridBar gb = grid_bar(a.bar);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int B = gridDim.x, m = a.m, lv = GL ? 0 : a.lv;
  const int rows = 3 * a.nc, ld = rows | 1;
  const int64_t c0 = (int64_t)blockIdx.x * a.nc, row0 = 3 * c0;
  const int nc = (int)(c0 >= a.N ? 0 : min((int64_t)a.nc, a.N - c0)), nr = 3 * nc;
  double* hs = lds;                        // [m + 2] dots of the current pass
  double* misc = hs + m + 2;               // [64]
  double* red = misc + 64;                 // [kLzBlock]
  const int64_t hrow = lz_hrow(m);
  // byte offsets of the dots and norms among the mailboxes
  const unsigned mail_h = 16u * (unsigned)((a.n + 15) / 16 * 16), mail_n = mail_h + 16u * (unsigned)(B * hrow),
                 mail_bytes = mail_n + 16u * (unsigned)(B * kLzWaves);
  unsigned tag = 0u;
  bool dead = false;
  // a value for the other workgroups, and the point after which they can
  // be read
  auto put = [&](double* p, unsigned off, double v) {
    if constexpr (MAIL)
      mail_put_d(a.mail + off / 8, v, tag);
    else
      store_wt(p, v);
  };
  auto exchange = [&] {
    if constexpr (MAIL)
      __syncthreads();
    else
      grid_barrier_wt(gb);
  };
  double* ws = GL ? a.gws + blockIdx.x * lz_work(rows, m) : misc + kLzMisc;
  double* w = ws;                          // [rows] the next vector before its scaling
  double* y = w + rows;                    // [rows] the operator's image, orthogonalised in place
  double* u = y + rows;                    // [rows] first columns
  double* al = u + rows;
  double* be = al + m;
  double* dp = be + m;
  double* dm = dp + m;
  double* sv = dm + m;                     // [m] Ritz coefficients
  double* Vl = sv + m;                     // [lv, ld] basis rows (LDS variant)
  auto vg = [&](int j) { return a.V + (int64_t)(j - lv) * a.n + row0; };
  auto v_at = [&](int j, int r) { return j < lv ? Vl[(int64_t)j * ld + r] : vg(j)[r]; };

  // sum_j coef[j] V[j][r], j < cnt, for this workgroup's rows: sixteen lanes
  // per row; out(r, sum) is called in all of them
  const int l16 = tid & 15;
  auto combine = [&](const double* coef, int cnt, auto out) {
    for (int r = tid >> 4; r < nr; r += kLzBlock / 16) {   // whole rows of lanes
      double s0 = 0.0;
      int j = l16;
#pragma unroll 2
      for (; j < min(cnt, lv); j += 16) s0 = fma(coef[j], Vl[(int64_t)j * ld + r], s0);
#pragma unroll 4
      for (; j < cnt; j += 16) s0 = fma(coef[j], vg(j)[r], s0);
      s0 += dpp_mov_d<0xB1>(s0);
      s0 += dpp_mov_d<0x4E>(s0);
      s0 += dpp_mov_d<0x141>(s0);
      s0 += dpp_mov_d<0x140>(s0);
      out(r, s0);
    }
  };
  // a wavefront's share of a squared norm out (its lanes' values v), and the
  // total of all shares
  auto norm_out = [&](double v) {
    v = wave_sum_d(v);
    const int64_t i = (int64_t)blockIdx.x * kLzWaves + wave;
    if (lane == 0) put(&a.part_n[i], mail_n + 16u * (unsigned)i, v);
  };
  auto norm_in = [&]() {
    double t = 0.0;
    if constexpr (MAIL) {
      for (int i0 = 64 * wave; i0 < B * kLzWaves; i0 += kLzBlock) {   // uniform over the wavefront
        const bool need[1] = {i0 + lane < B * kLzWaves};
        const unsigned off[1] = {need[0] ? mail_n + 16u * (unsigned)(i0 + lane) : 0u};
        double v[1];
        mail_take_d(a.bar, a.mail, mail_bytes, off, need, tag, v, dead);
        t += need[0] ? v[0] : 0.0;
      }
    } else {
      for (int i = tid; i < B * kLzWaves; i += kLzBlock) t += a.part_n[i];
    }
    t = wave_sum_d(t);
    if (lane == 0) misc[16 + wave] = t;
    __syncthreads();
    t = 0.0;
#pragma unroll
    for (int q = 0; q < kLzWaves; ++q) t += misc[16 + q];
    return t;
  };

  // static data of the first 64 entries of the wavefront's first camera, and
  // (MAIL) the vector at their other cameras, taken before the norm so that the
  // two waits overlap
  LzEntry e0;
  e0.other = -1;
  if (wave < nc) {
    const int q = a.cam_ptr[c0 + wave] + lane;
    if (q < a.cam_ptr[c0 + wave + 1]) e0 = lz_entry(a, q);
  }
  double v0[3] = {0.0, 0.0, 0.0};
  auto take_first = [&] {
    if constexpr (MAIL) {
      const bool live = e0.other >= 0;
      const unsigned o = live ? 48u * (unsigned)e0.other : 0u;
      const unsigned off[3] = {o, o + 16u, o + 32u};
      const bool need[3] = {live, live, live};
      mail_take_d(a.bar, a.mail, mail_bytes, off, need, tag, v0, dead);
    }
  };

  for (int col = 0; col < 2; ++col) {
    const double op_alpha = col ? a.inv_P : 1.0;
    // q_0 = start / |start|
    double acc = 0.0;
    ++tag;
    for (int r = tid; r < nr; r += kLzBlock) {
      const double x = a.start[col * a.n + row0 + r];
      w[r] = x;
      put(&a.wbuf[row0 + r], 16u * (unsigned)(row0 + r), x);
      acc += x * x;
    }
    norm_out(acc);
    exchange();
    take_first();
    double inv = 1.0 / sqrt(norm_in());
    double alpha = 0.0, b = 0.0, theta = 0.0;
    int used = m;
    bool have_s = false;
    for (int k = 0; k < m; ++k) {
      for (int r = tid; r < nr; r += kLzBlock) {
        const double v = w[r] * inv;
        if (k < lv)
          Vl[(int64_t)k * ld + r] = v;
        else
          vg(k)[r] = v;
      }
      __syncthreads();
      // y = op(q_k) - alpha_{k-1} q_k - beta_{k-1} q_{k-1}
      for (int cl = wave; cl < nc; cl += kLzWaves) {
        const int lo = a.cam_ptr[c0 + cl], hi = a.cam_ptr[c0 + cl + 1];
        double vc[3], t3[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < 3; ++j) vc[j] = w[3 * cl + j] * inv;
        for (int q0 = lo; q0 < hi; q0 += 64) {   // uniform over the wavefront
          const bool live = q0 + lane < hi;
          LzEntry e;
          e.other = 0;
          if (cl == wave && q0 == lo)
            e = e0;
          else if (live)
            e = lz_entry(a, q0 + lane);
          double vo[3];
          if constexpr (MAIL) {
            if (cl == wave && q0 == lo) {
#pragma unroll
              for (int j = 0; j < 3; ++j) vo[j] = v0[j];
            } else {
              const unsigned o = live ? 48u * (unsigned)e.other : 0u;
              const unsigned off[3] = {o, o + 16u, o + 32u};
              const bool need[3] = {live, live, live};
              mail_take_d(a.bar, a.mail, mail_bytes, off, need, tag, vo, dead);
            }
          }
          if (live) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
              if constexpr (!MAIL) vo[j] = a.wbuf[3 * (int64_t)e.other + j];
              vo[j] *= inv;
            }
            lz_term(e, vc, vo, t3);
          }
        }
        // totals in lanes 0, 4 and 8 (entries 0, 1, 2)
        double b2[2], b1[1];
        rs_stage_d<3, 3>(t3, b2, lane);
        rs_stage_d<2, 2>(b2, b1, lane);
        double t = b1[0];
        t += dpp_mov_d<0x4E>(t);
        t += dpp_mov_d<0xB1>(t);
        t += __shfl_xor(t, 16);
        t += __shfl_xor(t, 32);
        if (lane == 0 || lane == 4 || lane == 8) {
          const int r = 3 * cl + (lane >> 2);
          t *= op_alpha;
          if (col) {
            const double d = u[3 * cl] * vc[0] + u[3 * cl + 1] * vc[1] + u[3 * cl + 2] * vc[2];
            t += a.inv_N * u[r] * d;
          }
          t = fma(-alpha, v_at(k, r), t);
          if (k > 0) t = fma(-b, v_at(k - 1, r), t);
          y[r] = t;
        }
      }
      __syncthreads();
      double nrm2 = 0.0;
      for (int pass = 0; pass < 2; ++pass) {
        const double* src = pass ? w : y;
        ++tag;
        // partial dots with q_0 .. q_k and (entry k + 1) with the vector
        // itself: eight lanes each
        for (int j = tid >> 3; j <= k + 1; j += kLzBlock / 8) {
          const int l8 = tid & 7;
          double d = 0.0;
          if (j < lv && j <= k) {
            const double* vj = Vl + (int64_t)j * ld;
            for (int r = l8; r < nr; r += 8) d = fma(vj[r], src[r], d);
          } else {
            const double* vj = j <= k ? vg(j) : src;
#pragma unroll 4
            for (int r = l8; r < nr; r += 8) d = fma(vj[r], src[r], d);
          }
          d += dpp_mov_d<0xB1>(d);
          d += dpp_mov_d<0x4E>(d);
          d += dpp_mov_d<0x141>(d);
          if (l8 == 0) put(&a.part_h[blockIdx.x * hrow + j], mail_h + 16u * (unsigned)(blockIdx.x * hrow + j), d);
        }
        exchange();
        // the dots: threads over the entries and, while these are few, over
        // interleaved parts of the workgroups
        const int width = k + 2 <= 64 ? 64 : (k + 2 <= 128 ? 128 : (k + 2 <= 256 ? 256 : kLzBlock));
        for (int j0 = 0; j0 <= k + 1; j0 += width) {
          const int j = j0 + (tid & (width - 1)), parts = kLzBlock / width;
          double t = 0.0;
          if constexpr (MAIL) {
            for (int q = tid / width; q < B; q += 4 * parts) {   // uniform over the wavefront: width >= 64
              unsigned off[4];
              bool need[4];
              double p[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                need[e] = j <= k + 1 && q + e * parts < B;
                off[e] = need[e] ? mail_h + 16u * (unsigned)((q + e * parts) * hrow + j) : 0u;
              }
              mail_take_d(a.bar, a.mail, mail_bytes, off, need, tag, p, dead);
#pragma unroll
              for (int e = 0; e < 4; ++e) p[e] = need[e] ? p[e] : 0.0;
              t += (p[0] + p[1]) + (p[2] + p[3]);
            }
          } else if (j <= k + 1) {
            const double* ph = a.part_h + j;
            int q = tid / width;
#pragma unroll 1
            for (; q + 3 * parts < B; q += 4 * parts) {
              const double p0 = ph[q * hrow], p1 = ph[(q + parts) * hrow], p2 = ph[(q + 2 * parts) * hrow],
                           p3 = ph[(q + 3 * parts) * hrow];
              t += (p0 + p1) + (p2 + p3);
            }
            double p[3];   // the rest's loads in flight together too
#pragma unroll
            for (int e = 0; e < 3; ++e) p[e] = q + e * parts < B ? ph[(q + e * parts) * hrow] : 0.0;
            t += (p[0] + p[1]) + p[2];
          }
          if (parts > 1) {   // one round: width > k + 1
            red[tid] = t;
            __syncthreads();
            if (tid < width) {
              t = 0.0;
              for (int e = 0; e < parts; ++e) t += red[e * width + tid];
            }
          }
          if (tid < width && j <= k + 1) hs[j] = t;
        }
        __syncthreads();
        acc = 0.0;
        ++tag;
        combine(hs, k + 1, [&](int r, double t) {
          if (l16 != 0) return;
          const double wr = src[r] - t;
          w[r] = wr;
          put(&a.wbuf[row0 + r], 16u * (unsigned)(row0 + r), wr);
          acc = fma(wr, wr, acc);
        });
        norm_out(acc);
        alpha += hs[k];
        const double before = hs[k + 1];
        exchange();
        take_first();
        nrm2 = norm_in();
        if (!(nrm2 < 0.25 * before)) break;
      }
      b = sqrt(nrm2);
      if (tid == 0) {
        al[k] = alpha;
        be[k] = b;
      }
      // an invariant subspace, the last step, or a converged Ritz pair
      // (every workgroup takes the same decision from the same values)
      bool stop = !(b > 1e-12 * fmax(1.0, fabs(alpha))) || k + 1 == m;
      if (!stop && (k + 1) % kLzCheck == 0) {
        __syncthreads();
        theta = lz_tridiag(al, be, k + 1, dp, dm, sv, reinterpret_cast<int*>(misc));
        double tn = INFINITY;
        for (int i = lane; i <= k; i += 64) tn = fmin(tn, -(fabs(al[i]) + 2.0 * fabs(be[i])));
        tn = -wave_min_d(tn);
        stop = have_s = fabs(b * sv[k]) <= kLzTol * fmax(tn, 1e-300);
      }
      if (stop) {
        used = k + 1;
        break;
      }
      inv = 1.0 / b;
    }
    __syncthreads();
    if (!have_s) theta = lz_tridiag(al, be, used, dp, dm, sv, reinterpret_cast<int*>(misc));
    if (a.info && blockIdx.x == 0 && tid == 0) {
      a.info[2 * col] = theta;
      a.info[2 * col + 1] = (double)used;
    }
    // the Ritz vector, then per camera: c1 = x_c / |x_c| (first column); y_c
    // normalised, made orthogonal to c1 and normalised again (second), the
    // parameters being the rotation's first two columns (its third is c1 x c2
    // by the 6D map)
    combine(sv, used, [&](int r, double t) {
      if (l16 == 0) y[r] = t;
    });
    __syncthreads();
    for (int cl = tid; cl < nc; cl += kLzBlock) {
      double v[3], e[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) v[k] = y[3 * cl + k];
      double r = 1.0 / sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
      if (col == 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) u[3 * cl + k] = v[k] * r;
        continue;
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        v[k] *= r;
        e[k] = u[3 * cl + k];
      }
      const double d = v[0] * e[0] + v[1] * e[1] + v[2] * e[2];
#pragma unroll
      for (int k = 0; k < 3; ++k) v[k] -= d * e[k];
      r = 1.0 / sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        a.params[6 * (c0 + cl) + k] = (float)e[k];
        a.params[6 * (c0 + cl) + 3 + k] = (float)(v[k] * r);
      }
    }
    // the second problem overwrites what other workgroups still read
    if (col == 0) grid_barrier_wt(gb);
  }
}

fm_status ra_check(fm_ctx* ctx, fm_scene* s, const char* fn) {
  if (!s) return fm_fail(ctx, FM_EINVAL, "%s: scene is NULL", fn);
  if (s->ctx != ctx) return fm_fail(ctx, FM_EINVAL, "%s: scene belongs to another context", fn);
  return FM_OK;
}

}  // namespace

extern "C" fm_status fm_rotation_loss_grad(fm_ctx* ctx, fm_scene* s, const float* Rrel, const float* params,
                                           double* loss, float* grad, fm_stream stream) {
  if (!ctx) return FM_EINVAL;
  fm_status rc = ra_check(ctx, s, "fm_rotation_loss_grad");
  if (rc != FM_OK) return rc;
  if ((s->P > 0 && !Rrel) || (s->N > 0 && !params)) return fm_fail(ctx, FM_EINVAL, "fm_rotation_loss_grad: NULL argument");
  if (!loss && !grad) return FM_OK;
  FM_HIP_TRY(ctx, hipSetDevice(ctx->device));
  hipStream_t st = (hipStream_t)stream;
  const double invP = s->P > 0 ? 1.0 / (double)s->P : 0.0;
  const unsigned gp = grid_for(s->P > 0 ? s->P : 1, kBlock);
  {
    fm_timed timer(ctx, FM_K_RA_PAIR, st);
    hipLaunchKernelGGL(k_ra_pair, dim3(gp), dim3(kBlock), 0, st, params, s->pair_cams, Rrel, s->P, invP, s->contrib,
                       s->loss_part);
    FM_CHECK_LAUNCH(ctx);
  }
  if (loss) {
    hipLaunchKernelGGL(k_ra_loss_final, dim3(1), dim3(64), 0, st, s->loss_part, (int64_t)gp, invP, loss);
    FM_CHECK_LAUNCH(ctx);
  }
  if (grad && s->N > 0) {
    fm_timed timer(ctx, FM_K_RA_CAMERA, st);
    hipLaunchKernelGGL(k_ra_camera, dim3(grid_for((int64_t)s->N * 16, kBlock)), dim3(kBlock), 0, st, params,
                       s->cam_ptr, s->cam_items, s->contrib, s->N, grad);
    FM_CHECK_LAUNCH(ctx);
  }
  return FM_OK;
}

extern "C" fm_status fm_rotation_solve(fm_ctx* ctx, fm_scene* s, const float* Rrel, float* params, float* m, float* v,
                                       int32_t K, const fm_adam_cfg* cfg, double* loss_trace, fm_stream stream) {
  if (!ctx) return FM_EINVAL;
  fm_status rc = ra_check(ctx, s, "fm_rotation_solve");
  if (rc != FM_OK) return rc;
  if (!cfg || (s->P > 0 && !Rrel) || (s->N > 0 && (!params || !m || !v)))
    return fm_fail(ctx, FM_EINVAL, "fm_rotation_solve: NULL argument");
  if (K < 0) return fm_fail(ctx, FM_EINVAL, "fm_rotation_solve: K < 0");
  if (cfg->lr_total_steps <= 0 || cfg->lr_step0 < 0 || cfg->adam_step0 < 0 || !(cfg->lr_final_frac > 0.0f) ||
      !(cfg->lr_rot >= 0.0f) ||
      !(cfg->beta1 >= 0.0f && cfg->beta1 < 1.0f && cfg->beta2 >= 0.0f && cfg->beta2 < 1.0f && cfg->eps >= 0.0f))
    return fm_fail(ctx, FM_EINVAL, "fm_rotation_solve: bad Adam configuration");
  if (K == 0 || s->N == 0) return FM_OK;
  FM_HIP_TRY(ctx, hipSetDevice(ctx->device));
  hipStream_t st = (hipStream_t)stream;
  if (s->ra_coop_blocks <= 0) {
    int per_cu = 0;
    FM_HIP_TRY(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_ra_solve, kSolveBlock, 0));
    int per_cu_cam = 0;
    FM_HIP_TRY(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_cam, k_ra_solve_cam, kSolveBlock, 0));
    if (per_cu_cam < per_cu) per_cu = per_cu_cam;
    s->ra_coop_blocks = per_cu * ctx->num_cu;
    if (s->ra_coop_blocks <= 0) return fm_fail(ctx, FM_ECOOP, "cannot size the cooperative rotation kernel");
  }
  // sized like the epipolar loop
  int64_t want = grid_for(s->P, kSolveBlock);
  const int64_t want_c = grid_for((int64_t)s->N * 16, kSolveBlock);
  if (want_c > want) want = want_c;
  if (want > (s->P < 32768 ? 16 : 192)) want = s->P < 32768 ? 16 : 192;
  if (cfg->blocks > 0) want = cfg->blocks;
  if (want < 1) want = 1;
  if (want > s->ra_coop_blocks) want = s->ra_coop_blocks;
  if (want > s->loss_part_cap) want = s->loss_part_cap;
  RaArgs a;
  a.params = params; a.m = m; a.v = v;
  a.cams = s->pair_cams; a.Rrel = Rrel; a.cam_ptr = s->cam_ptr; a.cam_items = s->cam_items;
  a.contrib = s->contrib; a.rot = s->rot; a.part = s->loss_part; a.trace = loss_trace; a.bar = s->bar;
  a.P = s->P; a.N = s->N; a.K = K;
  a.invP = s->P > 0 ? 1.0 / (double)s->P : 0.0;
  a.lr = cfg->lr_rot; a.log_frac = log((double)cfg->lr_final_frac);
  a.b1 = cfg->beta1; a.b2 = cfg->beta2; a.eps = cfg->eps;
  a.lr_step0 = cfg->lr_step0; a.lr_total = cfg->lr_total_steps; a.adam_step0 = cfg->adam_step0;
  void* args[] = {&a};
  FM_HIP_TRY(ctx, fm_bar_reset(s->bar, st));
  // automatic grid: the camera loop, one wavefront per camera up to the
  // co-resident limit (faster at every size measured, up to the 5,000-camera
  // street graph with 185k pairs: 26.3 against 36.1 us per iteration)
  const CamGrid cg = cam_grid(s->N, s->ra_coop_blocks, ctx->num_cu);
  const int64_t want_cam = cg.blocks;
  if (cfg->blocks <= 0 && 2 * want_cam <= s->loss_part_cap) {
    RaCamArgs ca;
    ca.params = params; ca.alt = s->params_alt; ca.m = m; ca.v = v;
    ca.cams = s->pair_cams; ca.Rrel = Rrel; ca.cam_ptr = s->cam_ptr; ca.cam_items = s->cam_items;
    ca.rot = s->rot; ca.part = s->loss_part; ca.trace = loss_trace; ca.bar = s->bar;
    ca.P = s->P; ca.N = s->N; ca.K = K;
    ca.invP = a.invP; ca.lr = a.lr; ca.log_frac = a.log_frac; ca.b1 = a.b1; ca.b2 = a.b2; ca.eps = a.eps;
    ca.lr_step0 = a.lr_step0; ca.lr_total = a.lr_total; ca.adam_step0 = a.adam_step0;
    void* cargs[] = {&ca};
    fm_timed timer(ctx, FM_K_RA_SOLVE, st);
    hipError_t e = hipLaunchCooperativeKernel((const void*)k_ra_solve_cam, dim3((unsigned)want_cam),
                                              dim3(cg.threads), cargs, 0, st);
    if (e != hipSuccess) return fm_fail(ctx, FM_ECOOP, "cooperative launch failed: %s", hipGetErrorString(e));
    return FM_OK;
  }
  fm_timed timer(ctx, FM_K_RA_SOLVE, st);
  hipError_t e = hipLaunchCooperativeKernel((const void*)k_ra_solve, dim3((unsigned)want), dim3(kSolveBlock), args, 0, st);
  if (e != hipSuccess) return fm_fail(ctx, FM_ECOOP, "cooperative launch failed: %s", hipGetErrorString(e));
  return FM_OK;
}

extern "C" fm_status fm_rotation_init(fm_ctx* ctx, fm_scene* s, const float* Rrel, const double* start,
                                      int32_t steps, int32_t blocks, float* params, double* info, fm_stream stream) {
  if (!ctx) return FM_EINVAL;
  fm_status rc = ra_check(ctx, s, "fm_rotation_init");
  if (rc != FM_OK) return rc;
  if (s->N == 0) return FM_OK;
  if (!start || !params || (s->P > 0 && !Rrel)) return fm_fail(ctx, FM_EINVAL, "fm_rotation_init: NULL argument");
  if (steps < 1) return fm_fail(ctx, FM_EINVAL, "fm_rotation_init: steps must be >= 1");
  if (blocks < 0) return fm_fail(ctx, FM_EINVAL, "fm_rotation_init: blocks < 0");
  if (s->P == 0) return fm_fail(ctx, FM_ESHAPE, "fm_rotation_init: the pair graph is empty");
  FM_HIP_TRY(ctx, hipSetDevice(ctx->device));
  hipStream_t st = (hipStream_t)stream;
  const int64_t n = 3 * (int64_t)s->N;
  const int32_t m = steps < n ? steps : (int32_t)n;
  if (m > kLzMaxSteps) return fm_fail(ctx, FM_EINVAL, "fm_rotation_init: steps above %d", kLzMaxSteps);
  if (s->lz_coop_blocks <= 0) {
    int lds_max = 0, per_cu = 0;
    FM_HIP_TRY(ctx, hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, ctx->device));
    for (const void* k : {(const void*)k_ra_lanczos<false, false>, (const void*)k_ra_lanczos<false, true>,
                          (const void*)k_ra_lanczos<true, false>})
      FM_HIP_TRY(ctx, hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, lds_max));
    FM_HIP_TRY(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_ra_lanczos<false, false>, kLzBlock, lds_max));
    int per_cu_m = 0;
    FM_HIP_TRY(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_m, k_ra_lanczos<false, true>, kLzBlock, lds_max));
    if (per_cu_m < per_cu) per_cu = per_cu_m;
    int per_cu_g = 0;
    FM_HIP_TRY(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(
                        &per_cu_g, k_ra_lanczos<true, false>, kLzBlock, sizeof(double) * (kLzMaxSteps + 2 + kLzMisc)));
    if (per_cu_g < per_cu) per_cu = per_cu_g;
    s->lz_coop_blocks = per_cu * ctx->num_cu;
    s->lz_lds = lds_max;
    if (s->lz_coop_blocks <= 0) return fm_fail(ctx, FM_ECOOP, "cannot size the cooperative Lanczos kernel");
  }
  // cameras per workgroup: one per wavefront on small graphs, else 16, 32 or a
  // higher multiple of 16, so that a workgroup's rows are whole 128-byte lines
  // (more workgroups make the barriers and the sums of partials dearer, fewer
  // the operator and the basis products: with
  // grid barriers: 200 cameras 25 workgroups 1.08 ms, 13
  // 1.23, 50 1.16; 1,000 cameras 63 workgroups 4.7 ms, 32 and 125 5.4; 5,000
  // cameras 157 workgroups 12.9 ms, 105 14.7, 209 13.3)
  int64_t nc = kLzWaves;
  if (s->N > 64 * nc) nc = 16;
  if (s->N > 64 * nc) nc = 32;
  if (s->N > kLzMaxBlocks * nc) nc = ((int64_t)s->N + 16 * kLzMaxBlocks - 1) / (16 * kLzMaxBlocks) * 16;
  // (a given count is raised to one workgroup per 256 cameras: with a few
  // workgroups their own rows are the chain, 1,000 cameras at 100 steps 73 ms on
  // one, 37 on two)
  int64_t want = blocks > 0 ? std::max<int64_t>(blocks, (s->N + 255) / 256) : (s->N + nc - 1) / nc;
  if (want > s->lz_coop_blocks) want = s->lz_coop_blocks;
  if (want > s->N) want = s->N;
  // a workgroup's vectors fit the LDS variant from this many workgroups on
  const int64_t fit = (n + kLzLdsRows - 1) / kLzLdsRows;
  if (want < fit && fit <= s->lz_coop_blocks) want = fit;
  if (blocks > 0 || want * nc < s->N) nc = ((int64_t)s->N + want - 1) / want;
  const int64_t rows = 3 * nc;
  const int64_t head = m + 2 + kLzMisc;
  const int64_t lds_doubles = s->lz_lds / (int64_t)sizeof(double);
  const bool in_lds = m <= kLzLdsSteps && rows <= kLzLdsRows && head + lz_work(rows, m) <= lds_doubles;
  int64_t lv = in_lds ? (lds_doubles - head - lz_work(rows, m)) / (rows | 1) : 0;
  if (lv > m) lv = m;
  const size_t lds_bytes = sizeof(double) * (head + (in_lds ? lz_work(rows, m) + lv * (rows | 1) : 0));
  // workspace: V [(m - lv) n] | wbuf [n] | part_h [want lz_hrow(m)] | part_n [want kLzWaves] | gws,
  // wbuf and part_h at whole 128-byte lines; as mailboxes twice the size
  const bool mail = in_lds && want <= kLzMailBlocks;
  const int64_t vpad = ((m - lv) * n + 15) / 16 * 16, wpad = (n + 15) / 16 * 16;
  const int64_t shared = wpad + want * (lz_hrow(m) + kLzWaves);
  const int64_t need = vpad + (mail ? 2 : 1) * shared + (in_lds ? 0 : want * lz_work(rows, m));
  if (need > s->lz_cap) {
    FM_HIP_TRY(ctx, hipDeviceSynchronize());
    (void)hipFree(s->lz);
    s->lz = nullptr;
    s->lz_cap = 0;
    if (hipMalloc(&s->lz, sizeof(double) * need) != hipSuccess) {
      (void)hipGetLastError();
      return fm_fail(ctx, FM_ENOMEM, "fm_rotation_init: workspace of %lld doubles", (long long)need);
    }
    s->lz_cap = need;
  }
  LzArgs a;
  a.cams = s->pair_cams; a.Rrel = Rrel; a.cam_ptr = s->cam_ptr; a.cam_items = s->cam_items;
  a.start = start; a.params = params; a.info = info; a.bar = s->bar;
  a.V = s->lz;
  a.wbuf = a.V + vpad;
  a.part_h = a.wbuf + wpad;
  a.part_n = a.part_h + want * lz_hrow(m);
  a.gws = a.part_n + want * kLzWaves;
  a.mail = reinterpret_cast<MailWord*>(a.wbuf);
  a.n = n; a.N = s->N; a.m = m; a.nc = (int32_t)nc; a.lv = (int32_t)lv;
  a.inv_P = 1.0 / (double)s->P; a.inv_N = 1.0 / (double)s->N;
  fm_timed timer(ctx, FM_K_RA_INIT, st);
  void* args[] = {&a};
  FM_HIP_TRY(ctx, mail ? fm_mail_reset(s->bar, a.mail, 2 * shared, st) : fm_bar_reset(s->bar, st));
  const void* kernel = mail ? (const void*)k_ra_lanczos<false, true>
                            : (in_lds ? (const void*)k_ra_lanczos<false, false> : (const void*)k_ra_lanczos<true, false>);
  hipError_t e = hipLaunchCooperativeKernel(kernel, dim3((unsigned)want), dim3(kLzBlock), args, lds_bytes, st);
  if (e != hipSuccess) return fm_fail(ctx, FM_ECOOP, "cooperative launch failed: %s", hipGetErrorString(e));
  return FM_OK;
}
