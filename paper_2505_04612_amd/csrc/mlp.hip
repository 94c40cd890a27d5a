// Learned per-match weights: feature extraction and a 3 -> 64 -> 64 -> 1 MLP
// (ReLU, ReLU, sigmoid) whose 64x64 layer runs on MFMA (float16 operands,
// float32 accumulation), forward and backward.
//
// MFMA layouts (one wavefront, lane l, r = l % 16, q = l / 16), all with
// the 16x16 float32 result D[4q + j][r] in four registers:
//   v_mfma_f32_16x16x32_f16 (gfx950): operand A (16 x 32, M x K) holds
//     A[r][8q + j] in its 8 halves, operand B (32 x 16) holds B[8q + j][r];
//     used where the contraction runs over the hidden units (the forward's
//     second and third layers, the backward's dh1 = dh2 W2);
//   v_mfma_f32_16x16x16_f16: A[r][4q + j], B[4q + j][r]; used for the
//     backward's dW2, whose contraction runs over a 16-match tile;
//   v_mfma_f32_16x16x4_f32: A[r][q], B[q][r]; used for the forward's first
//     layer, whose contraction runs over the three features.  It is exactly
//     the chain of float32 FMAs over k = 0..3 from the start value.
// A tile is 16 matches; lanes r = 0..15 of each quarter q address one match
// (operand B) or one output unit (operand A).
#include <mutex>

#include "fm_internal.h"

typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f4a __attribute__((ext_vector_type(4), aligned(4)));   // in the caller's arrays: any float alignment

constexpr int kHid = 64;
// gradient entries: W2 (64x64), b2, W3, b3, W1 (64x3), b1
constexpr int kG_W2 = 0, kG_b2 = 4096, kG_W3 = 4160, kG_b3 = 4224, kG_W1 = 4225, kG_b1 = 4417, kG_N = 4481;

struct MlpPtrs {
  const float *W1, *b1, *W2, *b2, *W3, *b3, *mean, *std;
};

__device__ inline f4 mfma16(h4 a, h4 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0); }
__device__ inline f4 mfma32(h8 a, h8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }

__device__ inline f4 mfma4(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

constexpr float kLog2e = 1.4426950408889634f;

// What the backward reads of the weights, besides W2.
struct MlpLds {
  float W3[kHid], mean[3], rstd[3], b3;
};

__device__ inline void load_lds(const MlpPtrs& w, MlpLds& s) {
  for (int k = threadIdx.x; k < kHid; k += blockDim.x) s.W3[k] = w.W3[k];
  if (threadIdx.x < 3) {
    s.mean[threadIdx.x] = w.mean[threadIdx.x];
    s.rstd[threadIdx.x] = 1.0f / w.std[threadIdx.x];
  }
  if (threadIdx.x == 0) s.b3 = w.b3[0];
  __syncthreads();
}

__device__ inline void load_x(const float* feats, int64_t m, const MlpLds& s, float x[3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) x[c] = (feats[m * 3 + c] - s.mean[c]) * s.rstd[c];
}

// ReLU and rounding to float16 of four float32 values (rounding first: the
// same values, half the instructions).
__device__ inline h4 relu_h4(f4 c) {
  h4 h = {(_Float16)c[0], (_Float16)c[1], (_Float16)c[2], (_Float16)c[3]};
  return __builtin_elementwise_max(h, h4{});
}

__device__ inline h8 join(h4 a, h4 b) { return h8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]}; }

constexpr int kFwdWaves = 4;      // wavefronts per workgroup of the forward
constexpr int kFwdMatches = 64;   // matches per wavefront and step: four tiles
constexpr int kFwdPair = 2;       // tiles evaluated together

// Each wavefront takes 64 matches (four tiles) per step; the sigmoid and the
// output are one match per lane.
//
// All three layers run on MFMA, each one's result being the next one's operand
// B as it stands.  The first layer's float32 MFMA has the features as k = 2, 1,
// 0 (k = 3: zeros) and the bias as start value, the FMA chain of a plain
// evaluation; its operand A is so ordered that lane (q, r) receives units
// 8q .. 8q + 7 of each half of the layer.  The last layer has W3's float16 high
// and low parts in rows 4i and 4i + 1 of operand A, so that every quarter of
// the lanes holds the tile's z3 and lane l can take match l's.
//
// Bound by issue: per 64 matches 56 MFMAs take 1,150 cycles of a SIMD and some
// 260 VALU instructions 1,100 more (a VALU instruction of another wavefront
// delays running MFMAs by its own cycles, measured; 16 bytes per match move).
// 2.94M matches, per call: 78 us with the first layer on the VALU and one tile
// at a time, 47 one tile at a time, 44 with two tiles together (four: 49).
// KEEP: also store each match's 128 FP16 activations to act (what the
// backward reads back); the plain forward is instantiated without that code.
template <bool KEEP>
__global__ __launch_bounds__(64 * kFwdWaves, 3) void k_mlp_forward(int64_t M, const float* __restrict__ feats,
                                                                   MlpPtrs w, float out_scale,
                                                                   float* __restrict__ out,
                                                                   _Float16* __restrict__ act) {
  // layer 2's operand A in lane order, [kk][nt][lane]
  __shared__ h8 W2s[2][4][64];
  // per-wavefront staging of the kept activations: rows padded by 16 bytes,
  // so that the 16 rows a store instruction touches start in different banks
  constexpr int kTstRow = 2 * kHid + 8;
  __shared__ __attribute__((aligned(16))) _Float16 Tst[KEEP ? kFwdWaves : 1][16][kTstRow];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, q = lane >> 4;
  for (int k = threadIdx.x; k < kHid * kHid / 4; k += 64 * kFwdWaves) {
    const int o = k >> 4, i = 4 * (k & 15);   // unit i = 32 kk + 8 q + j
    const f4 v = *reinterpret_cast<const f4a*>(w.W2 + o * kHid + i);
    h4* dst = reinterpret_cast<h4*>(&W2s[i >> 5][o >> 4][16 * (i >> 3 & 3) + (o & 15)]) + (i >> 2 & 1);
    *dst = h4{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
  }
  // layer 1, MFMA (kk, h): row 4i + j is unit 32 kk + 8 i + 4 h + j, k is
  // feature 2 - k
  float A1[2][2];
  f4 C1[2][2], b2[4];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      A1[kk][h] = q < 3 ? w.W1[3 * (32 * kk + 8 * (r >> 2) + 4 * h + (r & 3)) + 2 - q] : 0.0f;
      C1[kk][h] = *reinterpret_cast<const f4a*>(w.b1 + 32 * kk + 8 * q + 4 * h);
    }
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) b2[nt] = *reinterpret_cast<const f4a*>(w.b2 + 16 * nt + 4 * q);
  // row r: W3's high part (r % 4 = 0), low part (r % 4 = 1) or zero; entry (q, j)
  // of half kk is unit 16 (2 kk + j / 4) + 4 q + j % 4, as layer 2 leaves them
  h8 A3[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float w3 = w.W3[16 * (2 * kk + (j >> 2)) + 4 * q + (j & 3)];
      const _Float16 hi = (_Float16)w3, lo = (_Float16)(w3 - (float)hi);
      A3[kk][j] = (r & 3) == 0 ? hi : ((r & 3) == 1 ? lo : (_Float16)0.0f);
    }
  const float b3 = w.b3[0];
  const int fc = q < 3 ? 2 - q : 0;   // this lane's feature (k = 3 takes zeros)
  const float mean = w.mean[fc], rstd = 1.0f / w.std[fc];
  __syncthreads();
  h8 A2[2][4];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) A2[kk][nt] = W2s[kk][nt][lane];
  const int64_t groups = (M + kFwdMatches - 1) / kFwdMatches, stride = (int64_t)gridDim.x * kFwdWaves;
  // the step's features, one per lane and tile, from one address (only the
  // last step checks the end: past it, match M - 1's)
  float fv[4];
  auto load = [&](int64_t g, float (&f)[4]) {
    const float* p = feats + (g * kFwdMatches + r) * 3 + fc;
    if ((g + 1) * kFwdMatches <= M) {
#pragma unroll
      for (int t = 0; t < 4; ++t) f[t] = p[48 * t];
    } else {
      const int left = (int)(M - 1 - g * kFwdMatches) - r;   // < 64
#pragma unroll
      for (int t = 0; t < 4; ++t) f[t] = p[3 * min(16 * t, left)];
    }
  };
  int64_t g = (int64_t)blockIdx.x * kFwdWaves + wave;
  if (g >= groups) return;   // no workgroup barrier below
  load(g, fv);
  for (; g < groups; g += stride) {
    const int64_t m0 = g * kFwdMatches;
    const int left = (int)min(M - m0, (int64_t)kFwdMatches);   // matches of this step
    _Float16* ap = KEEP ? act + (m0 + q) * 128 + 8 * r : nullptr;
    float fn[4];
    load(g + stride < groups ? g + stride : g, fn);   // the next step's, ahead
    float z = 0.0f;   // this lane's match: tile q
    // two tiles together, layer by layer: one's MFMAs run while the other's
    // results are rounded
#pragma unroll
    for (int t0 = 0; t0 < 4; t0 += kFwdPair) {
      h8 H1[kFwdPair][2], H2[kFwdPair][2];
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        f4 c[kFwdPair][2];
#pragma unroll
        for (int p = 0; p < kFwdPair; ++p) {
          const float x = q < 3 ? (fv[t0 + p] - mean) * rstd : 0.0f;
#pragma unroll
          for (int h = 0; h < 2; ++h) c[p][h] = mfma4(A1[kk][h], x, C1[kk][h]);
        }
#pragma unroll
        for (int p = 0; p < kFwdPair; ++p) H1[p][kk] = join(relu_h4(c[p][0]), relu_h4(c[p][1]));
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {   // units 32 kk .. 32 kk + 31
        f4 c[2][kFwdPair];
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
          for (int p = 0; p < kFwdPair; ++p) c[n][p] = mfma32(A2[0][2 * kk + n], H1[p][0], f4{0.0f, 0.0f, 0.0f, 0.0f});
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
          for (int p = 0; p < kFwdPair; ++p) c[n][p] = mfma32(A2[1][2 * kk + n], H1[p][1], c[n][p]);
#pragma unroll
        for (int p = 0; p < kFwdPair; ++p)
          H2[p][kk] = join(relu_h4(c[0][p] + b2[2 * kk]), relu_h4(c[1][p] + b2[2 * kk + 1]));
      }
#pragma unroll
      for (int p = 0; p < kFwdPair; ++p) {
        const f4 Z = mfma32(A3[1], H2[p][1], mfma32(A3[0], H2[p][0], f4{0.0f, 0.0f, 0.0f, 0.0f}));
        z = q == t0 + p ? Z[0] + Z[1] : z;
      }
      // a tile's activations (16 rows of 128 halves: one contiguous 4 KB
      // block of act) through this wavefront's LDS rows, then written with
      // consecutive 16-byte stores; LDS operations of a wavefront complete in
      // order, the fences keep the compiler from reordering them
      if constexpr (KEEP) {
#pragma unroll
        for (int p = 0; p < kFwdPair; ++p) {
          _Float16* T = &Tst[wave][0][0];
#pragma unroll
          for (int kk = 0; kk < 2; ++kk) {
            *reinterpret_cast<h8*>(T + r * kTstRow + 32 * kk + 8 * q) = H1[p][kk];
            const h8 v = H2[p][kk];
            *reinterpret_cast<h4*>(T + r * kTstRow + kHid + 32 * kk + 4 * q) = h4{v[0], v[1], v[2], v[3]};
            *reinterpret_cast<h4*>(T + r * kTstRow + kHid + 32 * kk + 16 + 4 * q) = h4{v[4], v[5], v[6], v[7]};
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int row = 4 * i + q, t = t0 + p;
            if (row < left - 16 * t)
              *reinterpret_cast<h8*>(ap + (16 * t + 4 * i) * 128) =
                  *reinterpret_cast<const h8*>(T + row * kTstRow + 8 * r);
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
      }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) fv[t] = fn[t];
    // the sigmoid on the hardware 2^x and reciprocal (~1 ulp each)
    const float e = __builtin_amdgcn_exp2f(-(z + b3) * kLog2e);
    if (lane < left) out[m0 + lane] = out_scale * __builtin_amdgcn_rcpf(1.0f + e);
  }
}

template <int CTRL>
__device__ inline float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Backward of sum_m dout[m] * sigmoid(z3[m]) from the stored activations.
// Each wavefront accumulates its gradient contributions in registers; the
// workgroup adds its four wavefronts' in a fixed order and writes them to its
// slot of `part` [workgroups, kG_N]; k_mlp_reduce adds the slots in a fixed
// order.  (With a slot per wavefront, 36.7 MB of them, and each row's inputs
// waited for on their own, 65,536 matches took 20.8 us and the reduction 18.1;
// now 18.0 and 4.1.  A training step of 1M matches 241 us, now 163, of which the
// activations written and read back take 100.)
__global__ __launch_bounds__(256) void k_mlp_backward(int64_t M, const float* __restrict__ feats, MlpPtrs w,
                                                      const _Float16* __restrict__ act,
                                                      const float* __restrict__ dout, float* __restrict__ part) {
  __shared__ MlpLds s;
  struct Stage {
    _Float16 T[4][16][kHid + 4];   // per-wave transpose of dh2
    // per-wave copy of the tile's activations (16 matches x 128, rows padded
    // so that the four row groups a read instruction touches use different
    // banks): read from global memory in 16-byte pieces, then per unit
    _Float16 Ast[4][16][2 * kHid + 8];
  };
  __shared__ union {
    Stage st;
    float sum[2][kG_N];   // two wavefronts' gradients, after the last tile
  } u;
  auto& T = u.st.T;
  auto& Ast = u.st.Ast;
  load_lds(w, s);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, q = lane >> 4;
  // operand B of dh1 = dh2 W2: B[k = o][n = i] = W2[o][i], k-tiles of 32
  h8 B2[2][4];
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int it = 0; it < 4; ++it)
#pragma unroll
      for (int j = 0; j < 8; ++j) B2[kt][it][j] = (_Float16)w.W2[(32 * kt + 8 * q + j) * kHid + 16 * it + r];
  f4 gW2[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) gW2[a][b] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  float gW3[4] = {0, 0, 0, 0}, gb2[4] = {0, 0, 0, 0}, gb1[4] = {0, 0, 0, 0}, gb3 = 0.0f;
  float gW1[4][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
  // The staging rows are the wavefront's own: its LDS operations complete in
  // order, and the fences keep the compiler from reordering them.  All loads
  // of a tile are issued together, from clamped rows (under a lane condition
  // each is waited for on its own); rows past M count as zeros.
  const int64_t ntiles = (M + 15) / 16;
  for (int64_t tile = (int64_t)blockIdx.x * 4 + wave; tile < ntiles; tile += (int64_t)gridDim.x * 4) {
    const int64_t m0 = tile * 16;
    const int left = M - m0 < 16 ? (int)(M - m0) : 16;
    // the tile's 16 x 128 activations (4 KB, 256 pieces of 16 bytes)
    h8 av[4];
    float dv[4], x[4][3];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int row = 4 * t + q;
      av[t] = *reinterpret_cast<const h8*>(act + (m0 + min(row, left - 1)) * 128 + 8 * r);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t m = m0 + min(4 * q + j, left - 1);
      dv[j] = dout[m];
      load_x(feats, m, s, x[j]);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int row = 4 * t + q;
#pragma unroll
      for (int j = 0; j < 8; ++j) av[t][j] = row < left ? av[t][j] : (_Float16)0.0f;
      *reinterpret_cast<h8*>(&Ast[wave][row][8 * r]) = av[t];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // this lane's result-layout rows 4q + j
    float h2[4][4], h1[4][4], d3[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool ok = 4 * q + j < left;
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        h2[j][nt] = (float)Ast[wave][4 * q + j][64 + 16 * nt + r];
        h1[j][nt] = (float)Ast[wave][4 * q + j][16 * nt + r];
      }
      float z = 0.0f;
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) z = fmaf(s.W3[16 * nt + r], h2[j][nt], z);
      // sum over the 16-lane row: lanes xor 1, 2, then (their quads and eights
      // alike by then) the mirrored quad and eight
      z += dpp_f<0xB1>(z);
      z += dpp_f<0x4E>(z);
      z += dpp_f<0x141>(z);
      z += dpp_f<0x140>(z);
      const float sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-(z + s.b3) * kLog2e));
      d3[j] = ok ? dv[j] * sg * (1.0f - sg) : 0.0f;
#pragma unroll
      for (int c = 0; c < 3; ++c) x[j][c] = ok ? x[j][c] : 0.0f;
    }
    // dh2 (result layout), dW3, db2, db3
    h4 A2[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float dh = h2[j][nt] > 0.0f ? d3[j] * s.W3[16 * nt + r] : 0.0f;
        gW3[nt] = fmaf(d3[j], h2[j][nt], gW3[nt]);
        gb2[nt] += dh;
        A2[nt][j] = (_Float16)dh;
        T[wave][4 * q + j][16 * nt + r] = (_Float16)dh;
      }
    if (r == 0) gb3 += d3[0] + d3[1] + d3[2] + d3[3];
    // dW2[o][i] += sum_m dh2[m][o] h1[m][i]
    h4 B1[4];
#pragma unroll
    for (int it = 0; it < 4; ++it)
#pragma unroll
      for (int j = 0; j < 4; ++j) B1[it][j] = (_Float16)h1[j][it];
#pragma unroll
    for (int ot = 0; ot < 4; ++ot)
#pragma unroll
      for (int it = 0; it < 4; ++it) gW2[ot][it] = mfma16(A2[ot], B1[it], gW2[ot][it]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // dh1 = (dh2 W2) * (h1 > 0): operand A[m][o] read back transposed
    h8 A3[2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int j = 0; j < 8; ++j) A3[kt][j] = T[wave][r][32 * kt + 8 * q + j];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      f4 C = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) C = mfma32(A3[kt], B2[kt][it], C);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float dh1 = h1[j][it] > 0.0f ? C[j] : 0.0f;
        gb1[it] += dh1;
#pragma unroll
        for (int c = 0; c < 3; ++c) gW1[it][c] = fmaf(dh1, x[j][c], gW1[it][c]);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  // per-unit sums: add the four quarters (lanes r, r+16, r+32, r+48)
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    for (int o = 16; o < 64; o <<= 1) {
      gW3[nt] += __shfl_xor(gW3[nt], o);
      gb2[nt] += __shfl_xor(gb2[nt], o);
      gb1[nt] += __shfl_xor(gb1[nt], o);
#pragma unroll
      for (int c = 0; c < 3; ++c) gW1[nt][c] += __shfl_xor(gW1[nt][c], o);
    }
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) gb3 += __shfl_xor(gb3, o);
  // (w0 + w2) + (w1 + w3) through LDS, which the tiles no longer use
  __syncthreads();
  auto each = [&](auto f) {
#pragma unroll
    for (int ot = 0; ot < 4; ++ot)
#pragma unroll
      for (int it = 0; it < 4; ++it)
#pragma unroll
        for (int j = 0; j < 4; ++j) f(kG_W2 + (16 * ot + 4 * q + j) * kHid + 16 * it + r, gW2[ot][it][j]);
    if (q == 0) {
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        const int h = 16 * nt + r;
        f(kG_W3 + h, gW3[nt]);
        f(kG_b2 + h, gb2[nt]);
        f(kG_b1 + h, gb1[nt]);
#pragma unroll
        for (int c = 0; c < 3; ++c) f(kG_W1 + 3 * h + c, gW1[nt][c]);
      }
    }
    if (lane == 0) f(kG_b3, gb3);
  };
  if (wave >= 2) each([&](int e, float v) { u.sum[wave - 2][e] = v; });
  __syncthreads();
  if (wave < 2) each([&](int e, float v) { u.sum[wave][e] += v; });
  __syncthreads();
  float* P = part + (int64_t)blockIdx.x * kG_N;
  for (int e = threadIdx.x; e < kG_N; e += 256) P[e] = u.sum[0][e] + u.sum[1][e];
}

struct MlpGradPtrs {
  float *W1, *b1, *W2, *b2, *W3, *b3;
};

// Sum of the gradient slots, entry by entry: each workgroup takes 64
// entries (one per lane, coalesced over the slots' rows); its kRedWaves
// wavefronts take consecutive ranges of the slots, sixteen running sums per
// lane so that sixteen loads are in flight, and the wavefronts' sums are added
// in wavefront order: a fixed order for any slot count.
constexpr int kRedWaves = 16;

__global__ __launch_bounds__(64 * kRedWaves) void k_mlp_reduce(const float* __restrict__ part, int64_t slots,
                                                              MlpGradPtrs g) {
  __shared__ float red[kRedWaves][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + lane;
  const int64_t per = (slots + kRedWaves - 1) / kRedWaves;
  const int64_t k0 = wave * per, k1 = min(slots, k0 + per);
  float p[16] = {};
  if (e < kG_N) {
    int64_t k = k0;
    for (; k + 16 <= k1; k += 16) {
#pragma unroll
      for (int u = 0; u < 16; ++u) p[u] += part[(k + u) * kG_N + e];
    }
    for (; k < k1; ++k) p[0] += part[k * kG_N + e];
  }
#pragma unroll
  for (int n = 8; n >= 1; n >>= 1)
#pragma unroll
    for (int u = 0; u < n; ++u) p[u] += p[u + n];
  red[wave][lane] = p[0];
  __syncthreads();
  if (wave != 0 || e >= kG_N) return;
  float s = 0.0f;
#pragma unroll
  for (int w = 0; w < kRedWaves; ++w) s += red[w][lane];
  if (e < kG_b2) g.W2[e] = s;
  else if (e < kG_W3) g.b2[e - kG_b2] = s;
  else if (e < kG_b3) g.W3[e - kG_W3] = s;
  else if (e < kG_W1) g.b3[0] = s;
  else if (e < kG_b1) g.W1[e - kG_W1] = s;
  else g.b1[e - kG_b1] = s;
}

// ------------------------------------------------------------------ features

// A constant held in scalar registers: a polynomial step then is one v_fma_f64
// with a scalar addend, instead of a copy of the constant into the
// accumulator and a v_fmac_f64.
__device__ inline double in_sgpr(double c) {
  asm("" : "+s"(c));
  return c;
}

// Reciprocal of a normal double by one Newton step on the hardware estimate
// (2^-23 or better), relative error below 1e-13: the features are rounded to
// float32.
__device__ inline double rcp_newton(double d) {
  const double r = __builtin_amdgcn_rcp(d);
  return fma(r, fma(-d, r, 1.0), r);
}

// log x for x > 0 (+inf included), relative error below 1e-12: x = 2^e m with
// m in [1/sqrt 2, sqrt 2), log m = 2 atanh(s), s = (m - 1)/(m + 1), as s times
// the degree-5 polynomial in s^2 that interpolates 2 atanh(s)/s at the
// Chebyshev nodes of [0, 0.02944] (2.7e-14).
__device__ inline float log_f32(double x) {
  double m = __builtin_amdgcn_frexp_mant(x);
  int e = __builtin_amdgcn_frexp_exp(x);
  const bool low = m < 0.70710678118654752;
  m = low ? m + m : m;
  e -= low ? 1 : 0;
  const double s = (m - 1.0) * rcp_newton(m + 1.0), z = s * s;
  double q = in_sgpr(0.19608097136405317);
  q = fma(q, z, in_sgpr(0.22174249811019753));
  q = fma(q, z, in_sgpr(0.2857216614814168));
  q = fma(q, z, in_sgpr(0.39999994891811563));
  q = fma(q, z, in_sgpr(0.6666666667957932));
  q = fma(q, z, in_sgpr(1.9999999999999472));
  const float r = (float)fma((double)e, 0.69314718055994531, s * q);
  return __builtin_isinf(x) ? INFINITY : r;
}

// sqrt(y2) for y2 of up to 2e298 or so, 1e-150 at the least, by one step on the
// reciprocal square root's estimate.
__device__ inline double sqrt_newton(double y2) {
  const double c = fmax(y2, 1e-300), h = __builtin_amdgcn_rsq(c), t0 = c * h;
  return fma(0.5 * t0, fma(-t0, h, 1.0), t0);
}

// atan2(y, ax) for y, ax >= 0, and pi less that where `neg`; relative error
// below 1e-12: the octant's ratio t = min/max, reduced by atan t = pi/4 +
// atan((t - 1)/(t + 1)) above tan(pi/8) (numerator and denominator, so one
// reciprocal serves both), then z P(z^2) with the degree-7 polynomial that
// interpolates atan(z)/z at the Chebyshev nodes of [0, tan^2(pi/8)] (7.6e-13).
// 0 and 0 give NaN.
__device__ inline float angle_f32(double y, double ax, bool neg) {
  const double mn = fmin(y, ax), mx = fmax(y, ax);
  const bool big = mn > 0.41421356237309505 * mx;
  const double num = big ? mn - mx : mn, den = big ? mn + mx : mx;
  const double z = num * rcp_newton(den), w = z * z;
  double q = in_sgpr(-0.03765508568903965);
  q = fma(q, w, in_sgpr(0.06974196550225259));
  q = fma(q, w, in_sgpr(-0.08992552657899722));
  q = fma(q, w, in_sgpr(0.11103456882226026));
  q = fma(q, w, in_sgpr(-0.14285386552286725));
  q = fma(q, w, in_sgpr(0.1999999305351789));
  q = fma(q, w, in_sgpr(-0.3333333327692213));
  q = fma(q, w, in_sgpr(0.9999999999992447));
  double a = fma(z, q, big ? 0.78539816339744831 : 0.0);
  a = y > ax ? 1.5707963267948966 - a : a;
  return (float)(neg ? 3.1415926535897931 - a : a);
}

struct __attribute__((packed, aligned(4))) Feat3 {
  float f0, f1, f2;
};

// Per match: f0 = log max(|r|, delta) with r = x2~^T E_n x1~ (float64),
// f1 = log |Q_n|, f2 = angle between R_i^T x1~ and R_j^T x2~.  One wavefront
// per 1,024-match work item, one match per lane and row.  From the pair's
// relative pose alone: with a = R_ij x1~ (the angle is that between a and
// x2~) and c = a x x2~, r = t_hat . c and the angle is atan2(|c|, a . x2~), 18
// float64 operations.  Bound by float64 VALU issue (~75 operations per match,
// 12 bytes out and 8 to 32 in): the library log, atan2 and sqrt with the
// rotations per wavefront and a search for the wavefront's pair: 81 us a call
// over 4.9M bfloat16 matches, this 36 us (20 us at the copy rate).
template <int DT>
__global__ __launch_bounds__(256) void k_features(const void* __restrict__ uv, const int64_t* __restrict__ off,
                                                  const int64_t* __restrict__ wi_off,
                                                  const int32_t* __restrict__ wi_pair, int64_t n_wi,
                                                  const double* __restrict__ pose, double delta,
                                                  float* __restrict__ feats) {
  const int lane = threadIdx.x & 63;
  // wave-uniform, so that the pair's data are scalar loads
  const int64_t w = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (w >= n_wi) return;
  const int64_t n = wi_pair[w];
  const int64_t start = off[n] + (w - wi_off[n]) * kChunk;
  const int64_t stop = min(off[n + 1], start + kChunk);
  const float f1 = logf((float)(off[n + 1] - off[n]));
  double R[9], th[3];
#pragma unroll
  for (int k = 0; k < 9; ++k) R[k] = pose[n * 12 + k];
#pragma unroll
  for (int k = 0; k < 3; ++k) th[k] = pose[n * 12 + 9 + k];
  for (int64_t m = start + lane; m < stop; m += kLanes) {
    double u1, v1, u2, v2;
    if constexpr (DT == FM_F32) {
      const float4 v = reinterpret_cast<const float4*>(uv)[m];
      u1 = v.x; v1 = v.y; u2 = v.z; v2 = v.w;
    } else if constexpr (DT == FM_BF16) {
      const uint2 v = reinterpret_cast<const uint2*>(uv)[m];
      u1 = __uint_as_float(v.x << 16); v1 = __uint_as_float(v.x & 0xffff0000u);
      u2 = __uint_as_float(v.y << 16); v2 = __uint_as_float(v.y & 0xffff0000u);
    } else {
      const double2* d = reinterpret_cast<const double2*>(uv) + 2 * m;
      const double2 p = d[0], q = d[1];
      u1 = p.x; v1 = p.y; u2 = q.x; v2 = q.y;
    }
    const double a0 = fma(R[0], u1, fma(R[1], v1, R[2])), a1 = fma(R[3], u1, fma(R[4], v1, R[5])),
                 a2 = fma(R[6], u1, fma(R[7], v1, R[8]));
    const double c0 = fma(-a2, v2, a1), c1 = fma(a2, u2, -a0), c2 = fma(a0, v2, -a1 * u2);
    double res = fabs(fma(th[0], c0, fma(th[1], c1, th[2] * c2)));
    const double y2 = fma(c0, c0, fma(c1, c1, c2 * c2)), x = fma(a0, u2, fma(a1, v2, a2));
    double y = sqrt_newton(y2), ax = fabs(x);
    // Past the range of the estimates (float64 coordinates beyond about 1e74, or
    // ones that are not finite, which x then is not either), told by the
    // exponents (2e298 and above): of finite coordinates infinities count as
    // atan2 counts them and large values are scaled; otherwise the angle is
    // NaN, and the residual the form x2~^T (E x1~), whose sums of infinities
    // the triple product does not have.
    const unsigned top = max((unsigned)__double2hiint(y2) & 0x7fffffffu, (unsigned)__double2hiint(x) & 0x7fffffffu);
    if (__builtin_expect(top >= 0x7de00000u, 0)) {
      const bool fin = isfinite(u1) && isfinite(v1) && isfinite(u2) && isfinite(v2);
      const bool nan = !fin || isnan(y2) || isnan(x), yi = isinf(y2), xi = isinf(ax);
      y = nan ? 0.0 : (yi ? 1.0 : (xi ? 0.0 : y * 0x1p-600));
      ax = nan ? 0.0 : (xi ? 1.0 : (yi ? 0.0 : ax * 0x1p-600));
      if (!fin) {
        double e[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const int p = (k + 1) % 3, q = (k + 2) % 3;   // row k of [t_hat]_x R
          const double E0 = th[p] * R[3 * q] - th[q] * R[3 * p], E1 = th[p] * R[3 * q + 1] - th[q] * R[3 * p + 1],
                       E2 = th[p] * R[3 * q + 2] - th[q] * R[3 * p + 2];
          e[k] = E0 * u1 + E1 * v1 + E2;
        }
        res = fabs(u2 * e[0] + v2 * e[1] + e[2]);
      }
    }
    Feat3 f;
    f.f0 = log_f32(res > delta ? res : delta);
    f.f1 = f1;
    f.f2 = angle_f32(y, ax, x < 0.0);
    reinterpret_cast<Feat3*>(feats)[m] = f;
  }
}

// ------------------------------------------------------------------ host side

static fm_status mlp_ptrs(fm_ctx* ctx, const fm_mlp* w, MlpPtrs& p) {
  if (!w || !w->W1 || !w->b1 || !w->W2 || !w->b2 || !w->W3 || !w->b3 || !w->feat_mean || !w->feat_std)
    return fm_fail(ctx, FM_EINVAL, "MLP weight pointer is NULL");
  p = MlpPtrs{w->W1, w->b1, w->W2, w->b2, w->W3, w->b3, w->feat_mean, w->feat_std};
  return FM_OK;
}

static unsigned mlp_blocks(fm_ctx* ctx, int64_t M) {
  const int64_t tiles = (M + 15) / 16;
  int64_t b = (tiles + 3) / 4;
  const int64_t cap = (int64_t)ctx->num_cu * 2;
  return (unsigned)(b < cap ? (b > 0 ? b : 1) : cap);
}

extern "C" fm_status fm_mlp_forward(fm_ctx* ctx, int64_t M, const float* feats, const fm_mlp* w, float out_scale,
                                    float* out, void* act, fm_stream stream) {
  if (!ctx) return FM_EINVAL;
  if (M < 0) return fm_fail(ctx, FM_ESHAPE, "fm_mlp_forward: M < 0");
  MlpPtrs p;
  fm_status rc = mlp_ptrs(ctx, w, p);
  if (rc != FM_OK) return rc;
  if (M == 0) return FM_OK;
  if (!feats || !out) return fm_fail(ctx, FM_EINVAL, "fm_mlp_forward: NULL feats or out");
  FM_HIP_TRY(ctx, hipSetDevice(ctx->device));
  // three workgroups per CU: what the registers let be resident
  const int64_t groups = (M + kFwdMatches - 1) / kFwdMatches, cap = 3 * (int64_t)ctx->num_cu;
  const int64_t want = (groups + kFwdWaves - 1) / kFwdWaves;
  const dim3 grid((unsigned)(want < cap ? want : cap)), block(64 * kFwdWaves);
  if (act)
    hipLaunchKernelGGL(k_mlp_forward<true>, grid, block, 0, (hipStream_t)stream, M, feats,
                       p, out_scale, out, (_Float16*)act);
  else
    hipLaunchKernelGGL(k_mlp_forward<false>, grid, block, 0, (hipStream_t)stream, M, feats,
                       p, out_scale, out, (_Float16*)nullptr);
  FM_CHECK_LAUNCH(ctx);
  return FM_OK;
}

extern "C" fm_status fm_mlp_backward(fm_ctx* ctx, int64_t M, const float* feats, const fm_mlp* w, const void* act,
                                     const float* dout, fm_mlp_grad* g, fm_stream stream) {
  if (!ctx) return FM_EINVAL;
  if (M < 0) return fm_fail(ctx, FM_ESHAPE, "fm_mlp_backward: M < 0");
  MlpPtrs p;
  fm_status rc = mlp_ptrs(ctx, w, p);
  if (rc != FM_OK) return rc;
  if (!g || !g->W1 || !g->b1 || !g->W2 || !g->b2 || !g->W3 || !g->b3)
    return fm_fail(ctx, FM_EINVAL, "fm_mlp_backward: gradient pointer is NULL");
  if (M > 0 && (!feats || !act || !dout)) return fm_fail(ctx, FM_EINVAL, "fm_mlp_backward: NULL input");
  FM_HIP_TRY(ctx, hipSetDevice(ctx->device));
  const unsigned blocks = mlp_blocks(ctx, M);
  const int64_t slots = blocks;
  const size_t need = sizeof(float) * (size_t)slots * kG_N;
  if (ctx->ws_bytes < need) {
    FM_HIP_TRY(ctx, hipStreamSynchronize((hipStream_t)stream));
    (void)hipFree(ctx->ws);
    ctx->ws = nullptr;
    ctx->ws_bytes = 0;
    hipError_t e = hipMalloc(&ctx->ws, need);
    if (e != hipSuccess) return fm_fail(ctx, FM_ENOMEM, "fm_mlp_backward: workspace: %s", hipGetErrorString(e));
    ctx->ws_bytes = need;
  }
  float* part = (float*)ctx->ws;
  if (M > 0) {
    hipLaunchKernelGGL(k_mlp_backward, dim3(blocks), dim3(256), 0, (hipStream_t)stream, M, feats, p,
                       (const _Float16*)act, dout, part);
    FM_CHECK_LAUNCH(ctx);
  }
  MlpGradPtrs gp{g->W1, g->b1, g->W2, g->b2, g->W3, g->b3};
  hipLaunchKernelGGL(k_mlp_reduce, dim3((kG_N + 63) / 64), dim3(64 * kRedWaves), 0, (hipStream_t)stream, part,
                     M > 0 ? slots : (int64_t)0, gp);
  FM_CHECK_LAUNCH(ctx);
  return FM_OK;
}


extern "C" fm_status fm_match_features(fm_ctx* ctx, fm_scene* s, const float* params, float delta, float* feats,
                                       fm_stream stream) {
  if (!ctx) return FM_EINVAL;
  if (!s || s->ctx != ctx) return fm_fail(ctx, FM_EINVAL, "fm_match_features: bad scene");
  if (!params || (!feats && s->M > 0)) return fm_fail(ctx, FM_EINVAL, "fm_match_features: NULL argument");
  if (!(delta > 0.0f)) return fm_fail(ctx, FM_EINVAL, "fm_match_features: delta must be > 0");
  FM_HIP_TRY(ctx, hipSetDevice(ctx->device));
  hipStream_t st = (hipStream_t)stream;
  fm_status rc = fm_launch_pair_poses(s, params, st);
  if (rc != FM_OK || s->n_wi == 0) return rc;
  const dim3 grid(grid_for(s->n_wi, 4)), block(256);
  switch (s->dtype) {
    case FM_F32:
      hipLaunchKernelGGL(k_features<FM_F32>, grid, block, 0, st, s->uv, s->offsets, s->wi_off, s->wi_pair, s->n_wi,
                         s->ess, (double)delta, feats);
      break;
    case FM_BF16:
      hipLaunchKernelGGL(k_features<FM_BF16>, grid, block, 0, st, s->uv, s->offsets, s->wi_off, s->wi_pair, s->n_wi,
                         s->ess, (double)delta, feats);
      break;
    default:
      hipLaunchKernelGGL(k_features<FM_F64>, grid, block, 0, st, s->uv, s->offsets, s->wi_off, s->wi_pair, s->n_wi,
                         s->ess, (double)delta, feats);
      break;
  }
  FM_CHECK_LAUNCH(ctx);
  return FM_OK;
}

// ------------------------------------------------------------------ allocation-free backward

// Gradient slots of fm_mlp_backward_noalloc: a file-scope device array (each
// GPU the library runs on holds its own copy until the process ends) sized
// for kNoAllocBlocks workgroups, a slot of kG_N floats each
// (2.3 MB).  Host code never passes `scratch` itself to a kernel (its host
// name is a stand-in, not a device address): the device address comes from
// hipGetSymbolAddress, taken once per device with that device current.
constexpr int kNoAllocBlocks = 128;
constexpr int64_t kNoAllocSlots = kNoAllocBlocks;
static __device__ __align__(256) float scratch[kNoAllocSlots * kG_N];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static float* g_scratch_dev[kMaxDevices];

// The device address of `scratch` on the context's device (which the caller
// has made current), looked up on the first call on that device.
static fm_status scratch_ptr(fm_ctx* ctx, float** out) {
  if (ctx->device < 0 || ctx->device >= kMaxDevices)
    return fm_fail(ctx, FM_EINVAL, "fm_mlp_backward_noalloc: device %d beyond %d", ctx->device, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[ctx->device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return fm_fail(ctx, FM_EHIP, "fm_mlp_backward_noalloc: hipGetSymbolAddress: %s", hipGetErrorString(e));
    g_scratch_dev[ctx->device] = (float*)p;
  }
  *out = g_scratch_dev[ctx->device];
  return FM_OK;
}

extern "C" fm_status fm_mlp_backward_noalloc(fm_ctx* ctx, int64_t M, const float* feats, const fm_mlp* w,
                                             const void* act, const float* dout, fm_mlp_grad* g, fm_stream stream) {
  if (!ctx) return FM_EINVAL;
  if (M < 0) return fm_fail(ctx, FM_ESHAPE, "fm_mlp_backward_noalloc: M < 0");
  MlpPtrs p;
  fm_status rc = mlp_ptrs(ctx, w, p);
  if (rc != FM_OK) return rc;
  if (!g || !g->W1 || !g->b1 || !g->W2 || !g->b2 || !g->W3 || !g->b3)
    return fm_fail(ctx, FM_EINVAL, "fm_mlp_backward_noalloc: gradient pointer is NULL");
  if (M > 0 && (!feats || !act || !dout)) return fm_fail(ctx, FM_EINVAL, "fm_mlp_backward_noalloc: NULL input");
  FM_HIP_TRY(ctx, hipSetDevice(ctx->device));
  float* part = nullptr;
  if ((rc = scratch_ptr(ctx, &part)) != FM_OK) return rc;
  // the launch of fm_mlp_backward, capped at the workgroups the scratch holds
  // slots for (identical launch, so identical results, up to 8,192 matches)
  unsigned blocks = mlp_blocks(ctx, M);
  if (blocks > (unsigned)kNoAllocBlocks) blocks = kNoAllocBlocks;
  const int64_t slots = blocks;
  if (slots > kNoAllocSlots)
    return fm_fail(ctx, FM_ESHAPE, "fm_mlp_backward_noalloc: %lld gradient slots exceed the %lld the scratch holds",
                   (long long)slots, (long long)kNoAllocSlots);
  if (M > 0) {
    hipLaunchKernelGGL(k_mlp_backward, dim3(blocks), dim3(256), 0, (hipStream_t)stream, M, feats, p,
                       (const _Float16*)act, dout, part);
    FM_CHECK_LAUNCH(ctx);
  }
  MlpGradPtrs gp{g->W1, g->b1, g->W2, g->b2, g->W3, g->b3};
  hipLaunchKernelGGL(k_mlp_reduce, dim3((kG_N + 63) / 64), dim3(64 * kRedWaves), 0, (hipStream_t)stream, part,
                     M > 0 ? slots : (int64_t)0, gp);
  FM_CHECK_LAUNCH(ctx);
  return FM_OK;
}
