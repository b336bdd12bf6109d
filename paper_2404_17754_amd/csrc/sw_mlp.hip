// Learned initial guess (gfx950): a per-DOF network 10 -> 64 -> 64 -> 1
// (ReLU) predicting a correction to quadratic extrapolation of the last
// increments.  Inference runs on the matrix cores (v_mfma_f32_16x16x16_f16,
// FP16 weights and activations, FP32 accumulation); training uses FP32
// forward / back-propagation kernels and Adam.  Feature definitions: the
// backward differences of orders 0..3 of the last four increments of the DOF
// and of their element-neighbour means, divided by the largest magnitude s of
// those increments, and the node's Vs/500 and rho/2000; guess = p2 + s * y
// with p2 = 3 d0 - 3 d1 + d2.  The differences are formed in FP64 before the
// rounding to FP16: the higher ones are small (the third is the error the
// quadratic extrapolation made at the last step), and formed after the
// rounding they would be lost in it.
#include <hip/hip_runtime.h>

#include "sw_device.h"
#include "sw_internal.h"

namespace sw {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
// vector loads from a caller's rows, which need be aligned to single values only
typedef float float2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));

// ---------------------------------------------------------------- network

// Network weights held in registers by every lane of a wave, laid out for
// the 16x16x16 and 16x16x32 MFMA in transposed form (rows = hidden units,
// columns = the 16 DOFs of one pass): lane l (q = l / 16, r = l % 16) holds
//   w1[b]    = W1[16b + r][4q .. 4q+3]          (A operand, layer 1)
//   b1[b]    = b1[16b + 4q .. 16b + 4q + 3]      (accumulator init)
//   w2[c][p] = W2[16c + r][32p + 4q .. +3] and [32p + 16 + 4q .. +3]
//              (A operand, layer 2: the sum over the units of both halves in
//              the order in which layer 1 leaves them in the lanes)
//   b2[c], w3[c] likewise for units 16c + 4q .. +3
struct MlpRegs {
  half4 w1[4];
  floatx4 b1[4];
  half8 w2[4][2];
  floatx4 b2[4];
  floatx4 w3[4];
  float b3;
};

__device__ __forceinline__ floatx4 load4(const float* __restrict__ p) {
  const float4 v = *reinterpret_cast<const float4*>(p);
  return floatx4{v.x, v.y, v.z, v.w};
}

__device__ __forceinline__ void mlp_load(const float* __restrict__ th, MlpRegs& R) {
  const int l = threadIdx.x & 63, q = l >> 4, r = l & 15;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    // features 4q .. 4q+3 of ten (8-byte aligned rows)
    const float2* w = reinterpret_cast<const float2*>(th + MLP_OFF_W1 + (16 * b + r) * MLP_IN + 4 * q);
    const float2 lo = q < 3 ? w[0] : make_float2(0.0f, 0.0f), hi = q < 2 ? w[1] : make_float2(0.0f, 0.0f);
    R.w1[b] = half4{(_Float16)lo.x, (_Float16)lo.y, (_Float16)hi.x, (_Float16)hi.y};
    R.b1[b] = load4(th + MLP_OFF_B1 + 16 * b + 4 * q);
    R.b2[b] = load4(th + MLP_OFF_B2 + 16 * b + 4 * q);
    R.w3[b] = load4(th + MLP_OFF_W3 + 16 * b + 4 * q);
  }
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const float* w = th + MLP_OFF_W2 + (16 * c + r) * MLP_H + 32 * p + 4 * q;
      const floatx4 lo = load4(w), hi = load4(w + 16);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        R.w2[c][p][j] = (_Float16)lo[j];
        R.w2[c][p][4 + j] = (_Float16)hi[j];
      }
    }
  R.b3 = th[MLP_OFF_B3];
}

// Network output for the 16 inputs of one pass.  xin: lane (q, r) holds
// features 4q .. 4q+3 of input r.  Returns y of input r in every lane.
__device__ __forceinline__ float mlp_eval16(const half4 xin, const MlpRegs& R) {
  half8 h1[2];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const floatx4 d = __builtin_amdgcn_mfma_f32_16x16x16f16(R.w1[b], xin, R.b1[b], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) h1[b >> 1][4 * (b & 1) + j] = (_Float16)fmaxf(d[j], 0.0f);
  }
  float part = 0.0f;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    floatx4 acc = R.b2[c];
#pragma unroll
    for (int p = 0; p < 2; ++p) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(R.w2[c][p], h1[p], acc, 0, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) part += R.w3[c][j] * fmaxf(acc[j], 0.0f);
  }
  part += __shfl_xor(part, 16, 64);
  part += __shfl_xor(part, 32, 64);
  return part + R.b3;
}

// y[i] = net(X[i, 0..9]) for i < n (matrix-core path, as in the guess).  A
// wavefront keeps the weights for all its passes (so few wavefronts: 20 KB of
// weights each) and loads the next pass's inputs, in one load, before it
// evaluates one.  The call on 1 M rows: 45-49 us (18 of it the call itself, as
// on one row), 87-90 with four loads of one value per lane and 16384
// wavefronts; 8 M rows 222 and 359.
__global__ __launch_bounds__(TPB) void k_mlp_forward(int64_t n, const float* __restrict__ X,
                                                     const float* __restrict__ theta, float* __restrict__ y) {
  const int l = threadIdx.x & 63, q = l >> 4, r = l & 15;
  const int64_t nwave = ((int64_t)gridDim.x * TPB) >> 6;
  int64_t g = ((int64_t)blockIdx.x * TPB + threadIdx.x) >> 6;
  auto load = [&](int64_t pass) {
    const int64_t i = pass * 16 + r;
    floatx4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (i < n && q < 2) v = *reinterpret_cast<const float4u*>(X + i * MLP_IN + 4 * q);
    if (i < n && q == 2) {
      const float2u lo = *reinterpret_cast<const float2u*>(X + i * MLP_IN + 8);
      v.x = lo.x;
      v.y = lo.y;
    }
    return v;
  };
  floatx4 nx = load(g);
  MlpRegs R;
  mlp_load(theta, R);
  for (; g * 16 < n; g += nwave) {
    const floatx4 x = nx;
    nx = load(g + nwave);
    const float v = mlp_eval16(half4{(_Float16)x.x, (_Float16)x.y, (_Float16)x.z, (_Float16)x.w}, R);
    const int64_t i = g * 16 + r;
    if (q == 0 && i < n) y[i] = v;
  }
}

void launch_mlp_forward(int64_t n, const float* X, const float* theta, float* y, hipStream_t s) {
  if (n <= 0) return;
  unsigned g = (unsigned)((n / 16 + 3) / 4 + 1);
  if (g > 1024) g = 1024;
  hipLaunchKernelGGL(k_mlp_forward, dim3(g), dim3(TPB), 0, s, n, X, theta, y);
}

// ------------------------------------------------------------ features

struct GuessIn {
  double d[4];
  float nb[4];
  float vs, rho;
};

__device__ __forceinline__ void load_features(const MlpFeat& F, int64_t dof, GuessIn& o) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    o.d[k] = F.hist[(int64_t)((F.head - k) & 3) * F.n_dof + dof];
    o.nb[k] = F.nbh[(int64_t)((F.nb_head - k) & 3) * F.n_dof + dof];
  }
  const int64_t node = dof / 3;
  o.vs = F.node_mat[2 * node];
  o.rho = F.node_mat[2 * node + 1];
}

// scale s and the normalised feature quartet of lane group q
__device__ __forceinline__ double feat_scale(const GuessIn& g) {
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) s = fmax(s, fmax(fabs(g.d[k]), fabs((double)g.nb[k])));
  return s;
}

// backward differences of orders 0..3 of a[0..3] (newest first)
__device__ __forceinline__ void differences(const double a[4], double o[4]) {
  o[0] = a[0];
  o[1] = a[0] - a[1];
  o[2] = a[0] - 2.0 * a[1] + a[2];
  o[3] = a[0] - 3.0 * a[1] + 3.0 * a[2] - a[3];
}

// the ten features (FP32; the network rounds them to FP16)
__device__ __forceinline__ void features(const GuessIn& g, double s, float f[MLP_IN]) {
  const double inv = s > 0.0 ? 1.0 / s : 0.0;
  double nb[4], dd[4], dn[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) nb[k] = (double)g.nb[k];
  differences(g.d, dd);
  differences(nb, dn);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    f[k] = (float)(dd[k] * inv);
    f[4 + k] = (float)(dn[k] * inv);
  }
  f[8] = g.vs / 500.0f;
  f[9] = g.rho / 2000.0f;
}

__device__ __forceinline__ half4 feat_quartet(const GuessIn& g, double s, int q) {
  float f[MLP_IN];
  features(g, s, f);
  half4 x;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int k = 4 * q + j;
    x[j] = (_Float16)(k < MLP_IN ? f[k] : 0.0f);
  }
  return x;
}

// x = p2 + s * net(features) per DOF (corr: the correction s * net alone);
// x = 0 when ||b|| = 0 or s = 0
__global__ __launch_bounds__(TPB) void k_mlp_guess(MlpFeat F, const float* __restrict__ theta,
                                                   double* __restrict__ x, const CgCtl* ctl, int corr) {
  MlpRegs R;
  mlp_load(theta, R);
  const bool zero = !(ctl->bb > 0.0);
  const int l = threadIdx.x & 63, q = l >> 4, r = l & 15;
  const int64_t wave = ((int64_t)blockIdx.x * TPB + threadIdx.x) >> 6;
  const int64_t nwave = ((int64_t)gridDim.x * TPB) >> 6;
  for (int64_t g = wave; g * 16 < F.n_dof; g += nwave) {
    const int64_t dof = g * 16 + r;
    GuessIn in{};
    if (dof < F.n_dof) load_features(F, dof, in);
    const double s = feat_scale(in);
    const float y = mlp_eval16(feat_quartet(in, s, q), R);
    if (q == 0 && dof < F.n_dof) {
      const double p2 = corr ? 0.0 : 3.0 * in.d[0] - 3.0 * in.d[1] + in.d[2];
      x[dof] = (zero || !(s > 0.0)) ? 0.0 : p2 + s * (double)y;
    }
  }
}

void launch_mlp_guess(const MlpFeat& F, const float* theta, double* x, const CgCtl* ctl, bool corr, hipStream_t s) {
  unsigned g = (unsigned)((F.n_dof / 16 + 3) / 4 + 1);
  if (g > 8192) g = 8192;
  hipLaunchKernelGGL(k_mlp_guess, dim3(g), dim3(TPB), 0, s, F, theta, x, ctl, corr ? 1 : 0);
}

// Counter-based sampling: SplitMix64 finaliser of (seed, step, j).
__device__ __forceinline__ uint64_t splitmix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Training rows for `count` DOFs drawn by (seed, step, j): the ten features
// (before the step), the target (du - p2) / s and the weight s^2.  Rows go
// to out[(row0 + j) mod capacity][12].
__global__ __launch_bounds__(TPB) void k_mlp_collect(MlpFeat F, const double* __restrict__ du, int count,
                                                     uint64_t seed, int64_t step, int64_t row0, int64_t capacity,
                                                     float* __restrict__ out) {
  const int j = blockIdx.x * TPB + threadIdx.x;
  if (j >= count) return;
  const uint64_t h = splitmix64(seed ^ splitmix64((uint64_t)step * 0x100000001B3ull + (uint64_t)j));
  const int64_t dof = (int64_t)(h % (uint64_t)F.n_dof);
  GuessIn in;
  load_features(F, dof, in);
  const double s = feat_scale(in);
  const double inv = s > 0.0 ? 1.0 / s : 0.0;
  float* o = out + ((row0 + j) % capacity) * MLP_ROW;
  float f[MLP_IN];
  features(in, s, f);
  for (int k = 0; k < MLP_IN; ++k) o[k] = f[k];
  const double p2 = 3.0 * in.d[0] - 3.0 * in.d[1] + in.d[2];
  o[10] = (float)((du[dof] - p2) * inv);
  o[11] = (float)(s * s);
}

void launch_mlp_collect(const MlpFeat& F, const double* du, int count, uint64_t seed, int64_t step, int64_t row0,
                        int64_t capacity, float* out, hipStream_t s) {
  if (count <= 0) return;
  hipLaunchKernelGGL(k_mlp_collect, dim3((count + TPB - 1) / TPB), dim3(TPB), 0, s, F, du, count, seed, step, row0,
                     capacity, out);
}

// -------------------------------------------------------------- training

// Gradient kernel: a wavefront takes 16 samples at a time through FP32 matrix
// instructions (16x16x4: products and sums as in scalar FP32 code), four
// wavefronts to a workgroup.  Hidden units are rows and samples columns, so
// that a layer's output is the next one's right operand as it stands.  The
// rows of a block are in the order grad_unit, which gives lane (q, r) the units
// 16 b + 4 j + q of sample r: the instruction (b, j) sums over four consecutive
// units (features), and a unit's input is the same chain of additions as in
// scalar code (so the units at the edge of the rectifier are on the same side
// of it; in another order some of a batch's half million are not).  Only the
// weight gradients, sums over the samples, need the activations with the
// samples across the lanes: they go through the LDS.  Per wavefront and 16
// samples 12 + 64 + 16 instructions forward, 64 back, 64 + 16 for the weight
// gradients, 32 cycles each: 3.5 us; the rest is latency (the rows, weights
// and accumulators of a workgroup that has one pass to make).
// One step of many, with Adam, 8192 rows: 406 us as one work-item per sample in
// scalar loops, 21.4 so (17.6 at 100 rows; 33 with the weights fetched one load
// after the other and the sums of a wavefront four to an LDS bank, 28.7 with an
// addition of the loss per wavefront instead of one per workgroup).
// FP32 sums run over at most GFLUSH * 16 = 128 samples, then in FP64.
constexpr int GW = 4, GS = 16, GFLUSH = 8;
constexpr int GLD = 17, GLD2 = 65, GLDX = 13;  // row strides that spread the LDS banks
// the workgroup's sums in the order of theta, the rows of W2 apart by GACC
// (lanes 16 apart add into rows four apart: 4 * GACC doubles are half the banks)
constexpr int GACC = 68, GRAD_ACC = MLP_NP + MLP_H * (GACC - MLP_H);
__device__ __forceinline__ int grad_at(int j) {
  return j < MLP_OFF_W2 ? j : j < MLP_OFF_W2 + MLP_H * MLP_H ? j + (j - MLP_OFF_W2) / MLP_H * (GACC - MLP_H)
                                                               : j + MLP_H * (GACC - MLP_H);
}
struct GradLds {
  double acc[GRAD_ACC + (GRAD_ACC & 1)];
  double loss[2 * GW];
  float w1[MLP_H * GLD], w2[MLP_H * GLD2], b1[MLP_H], b2[MLP_H], w3[MLP_H];
  struct {
    float h1[MLP_H * GLD], d1[MLP_H * GLD], d2[MLP_H * GLD], x[GS * GLDX];
  } wave[GW];
};

// the unit of a block of 16 in its row r
__device__ __forceinline__ int grad_unit(int r) { return 4 * (r & 3) + (r >> 2); }

// sum over the 16 lanes of a row, in every lane
__device__ __forceinline__ float row_sum(float v) {
  auto add = [](float a, int moved) { return a + __int_as_float(moved); };
  v = add(v, __builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xf, 0xf, true));
  v = add(v, __builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xf, 0xf, true));
  v = add(v, __builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xf, 0xf, true));
  return add(v, __builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xf, 0xf, true));
}

// Gradient of L = sum w (y - t)^2 / sum w, accumulated un-normalised:
// grad += sum_i 2 w_i (y_i - t_i) dy_i/dtheta, loss2 += (sum w e^2, sum w).
// Samples: rows i < n of S (all, in order) when nb == 0; otherwise nb rows
// drawn by (seed, batch) with replacement.
__global__ __launch_bounds__(64 * GW) void k_mlp_grad(const float* __restrict__ S, int64_t n, int64_t nb,
                                                      uint64_t seed, int64_t batch, const float* __restrict__ theta,
                                                      double* __restrict__ grad, double* __restrict__ loss2) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  GradLds& L = *reinterpret_cast<GradLds*>(smem_raw);
  const int tid = threadIdx.x, l = tid & 63, wv = tid >> 6, q = l >> 4, r = l & 15;
  const int ru = grad_unit(r);
  const int64_t total = nb > 0 ? nb : n, step = (int64_t)gridDim.x * GW * GS;
  int64_t c0 = (int64_t)blockIdx.x * GW * GS;
  // values q, 4 + q and 8 + q of sample r (10 and 11: target and weight)
  auto load_row = [&](int64_t k) {
    floatx4 x = {0.0f, 0.0f, 0.0f, 0.0f};
    if (k < total) {
      int64_t i = k;
      if (nb > 0) i = (int64_t)(splitmix64(seed ^ splitmix64((uint64_t)batch * 0x100000001B3ull + (uint64_t)k)) %
                                (uint64_t)n);
#pragma unroll
      for (int j = 0; j < 3; ++j) x[j] = S[i * MLP_ROW + 4 * j + q];
    }
    return x;
  };
  floatx4 xr = load_row(c0 + wv * GS + r);
  // the weights, every load before the first is waited for
  constexpr int N2 = MLP_H * MLP_H / (4 * 64 * GW), N1 = MLP_H * 16 / (64 * GW);
  floatx4 t2[N2];
  float t1[N1];
#pragma unroll
  for (int k = 0; k < N2; ++k)
    t2[k] = *reinterpret_cast<const float4u*>(theta + MLP_OFF_W2 + 4 * (tid + k * 64 * GW));
#pragma unroll
  for (int k = 0; k < N1; ++k) {
    const int j = tid + k * 64 * GW;
    t1[k] = theta[MLP_OFF_W1 + (j / 16) * MLP_IN + (j % 16 < MLP_IN ? j % 16 : 0)];
  }
#pragma unroll 4
  for (int j = tid; j < GRAD_ACC; j += 64 * GW) L.acc[j] = 0.0;
#pragma unroll
  for (int k = 0; k < N2; ++k) {
    const int j = 4 * (tid + k * 64 * GW);
#pragma unroll
    for (int c = 0; c < 4; ++c) L.w2[(j / MLP_H) * GLD2 + j % MLP_H + c] = t2[k][c];
  }
#pragma unroll
  for (int k = 0; k < N1; ++k) {
    const int j = tid + k * 64 * GW;
    L.w1[(j / 16) * GLD + j % 16] = j % 16 < MLP_IN ? t1[k] : 0.0f;
  }
  if (tid < MLP_H) {
    L.b1[tid] = theta[MLP_OFF_B1 + tid];
    L.b2[tid] = theta[MLP_OFF_B2 + tid];
    L.w3[tid] = theta[MLP_OFF_W3 + tid];
  }
  const float b3 = theta[MLP_OFF_B3];
  __syncthreads();
  auto& W = L.wave[wv];
  const floatx4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  floatx4 g2[4][4], g1[4], gb2[4], gw3[4];  // weight gradients; biases and output layer per lane's sample
  float gb3 = 0.0f;
  auto clear = [&] {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      g1[c] = gb2[c] = gw3[c] = zero;
#pragma unroll
      for (int b = 0; b < 4; ++b) g2[c][b] = zero;
    }
    gb3 = 0.0f;
  };
  // FP32 sums into the workgroup's FP64 ones
  auto flush = [&] {
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int u = 16 * c + 4 * q + j;
#pragma unroll
        for (int b = 0; b < 4; ++b) atomicAdd(&L.acc[MLP_OFF_W2 + u * GACC + 16 * b + r], (double)g2[c][b][j]);
        if (r <= MLP_IN)  // column 10 of the inputs is one: the bias
          atomicAdd(&L.acc[grad_at(r < MLP_IN ? MLP_OFF_W1 + u * MLP_IN + r : MLP_OFF_B1 + u)], (double)g1[c][j]);
        const float sb = row_sum(gb2[c][j]), sw = row_sum(gw3[c][j]);
        if (r == 0) {
          const int v = 16 * c + 4 * j + q;
          atomicAdd(&L.acc[grad_at(MLP_OFF_B2 + v)], (double)sb);
          atomicAdd(&L.acc[grad_at(MLP_OFF_W3 + v)], (double)sw);
        }
      }
    const float s3 = row_sum(gb3);
    if (l == 0) atomicAdd(&L.acc[grad_at(MLP_OFF_B3)], (double)s3);
    clear();
  };
  clear();
  double lw = 0.0, ww = 0.0;
  for (int pass = 1; c0 < total; c0 += step, ++pass) {
    const bool live = c0 + wv * GS + r < total;
    const floatx4 x = xr;
    xr = load_row(c0 + step + wv * GS + r);
    const float xf[3] = {x.x, x.y, q < 2 ? x.z : 0.0f};
    const float target = __shfl(x.z, 32 + r, 64), weight = __shfl(x.z, 48 + r, 64);
    floatx4 h1[4], h2[4], d2[4], z;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
#pragma unroll
      for (int j = 0; j < 4; ++j) z[j] = L.b1[16 * b + 4 * j + q];
#pragma unroll
      for (int j = 0; j < 3; ++j)
        z = __builtin_amdgcn_mfma_f32_16x16x4f32(L.w1[(16 * b + ru) * GLD + 4 * j + q], xf[j], z, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) h1[b][j] = fmaxf(z[j], 0.0f);
    }
    floatx4 y = {b3, b3, b3, b3};  // the output, in every row alike
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
      for (int j = 0; j < 4; ++j) z[j] = L.b2[16 * c + 4 * j + q];
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          z = __builtin_amdgcn_mfma_f32_16x16x4f32(L.w2[(16 * c + ru) * GLD2 + 16 * b + 4 * j + q], h1[b][j], z, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        h2[c][j] = fmaxf(z[j], 0.0f);
        y = __builtin_amdgcn_mfma_f32_16x16x4f32(L.w3[16 * c + 4 * j + q], h2[c][j], y, 0, 0, 0);
      }
    }
    const float e = y[0] - target;
    const float dy = live ? 2.0f * weight * e : 0.0f;
    if (live && q == 0) {
      lw += (double)weight * (double)e * (double)e;
      ww += (double)weight;
      gb3 += dy;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int u = 16 * c + 4 * j + q;
        d2[c][j] = h2[c][j] > 0.0f ? dy * L.w3[u] : 0.0f;
        gb2[c][j] += d2[c][j];
        gw3[c][j] += live ? dy * h2[c][j] : 0.0f;
        W.h1[u * GLD + r] = h1[c][j];
        W.d2[u * GLD + r] = d2[c][j];
      }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      z = zero;
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          z = __builtin_amdgcn_mfma_f32_16x16x4f32(L.w2[(16 * c + 4 * j + q) * GLD2 + 16 * b + ru], d2[c][j], z, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) W.d1[(16 * b + 4 * j + q) * GLD + r] = h1[b][j] > 0.0f ? z[j] : 0.0f;
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) W.x[r * GLDX + 4 * j + q] = 4 * j + q == MLP_IN ? 1.0f : xf[j];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int sm = 4 * t + q;  // the sample of this lane in the sums over samples
      const float xb = r <= MLP_IN ? W.x[sm * GLDX + r] : 0.0f;
      float ha[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) ha[b] = W.h1[(16 * b + r) * GLD + sm];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float da = W.d2[(16 * c + r) * GLD + sm];
#pragma unroll
        for (int b = 0; b < 4; ++b) g2[c][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(da, ha[b], g2[c][b], 0, 0, 0);
        g1[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(W.d1[(16 * c + r) * GLD + sm], xb, g1[c], 0, 0, 0);
      }
    }
    if (pass % GFLUSH == 0) flush();
    __syncthreads();
  }
  flush();
  lw = wave_sum(lw);
  ww = wave_sum(ww);
  if (l == 0) {
    L.loss[wv] = lw;
    L.loss[GW + wv] = ww;
  }
  __syncthreads();
  if (tid < 2) {  // one addition a workgroup to each (12 ns apiece on one address)
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < GW; ++k) t += L.loss[GW * tid + k];
    atomic_add(&loss2[tid], t);
  }
#pragma unroll 4
  for (int j = tid; j < MLP_NP; j += 64 * GW) {
    const double a = L.acc[grad_at(j)];
    if (a != 0.0) atomic_add(&grad[j], a);
  }
}

void launch_mlp_grad(const float* S, int64_t n, int64_t nb, uint64_t seed, int64_t batch, const float* theta,
                     double* grad, double* loss2, hipStream_t s) {
  const int64_t total = nb > 0 ? nb : n;
  if (total <= 0) return;
  unsigned g = (unsigned)((total + GW * GS - 1) / (GW * GS));
  if (g > 256) g = 256;  // one per compute unit (LDS: 117 KB)
  hipLaunchKernelGGL(k_mlp_grad, dim3(g), dim3(64 * GW), sizeof(GradLds), s, S, n, nb, seed, batch, theta, grad,
                     loss2);
}

// Adam on the FP32 master weights with the gradient normalised by sum w;
// clears the gradient for the next batch.
__global__ __launch_bounds__(TPB) void k_mlp_adam(float* __restrict__ theta, float* __restrict__ m,
                                                  float* __restrict__ v, double* __restrict__ grad,
                                                  const double* __restrict__ loss2, int64_t step, float lr) {
  const int j = blockIdx.x * TPB + threadIdx.x;
  if (j >= MLP_NP) return;
  const double sw = loss2[1];
  const float g = sw > 0.0 ? (float)(grad[j] / sw) : 0.0f;
  grad[j] = 0.0;
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float mj = b1 * m[j] + (1.0f - b1) * g;
  const float vj = b2 * v[j] + (1.0f - b2) * g * g;
  m[j] = mj;
  v[j] = vj;
  const float mh = mj / (1.0f - powf(b1, (float)step));
  const float vh = vj / (1.0f - powf(b2, (float)step));
  theta[j] -= lr * mh / (sqrtf(vh) + eps);
}

void launch_mlp_adam(float* theta, float* m, float* v, double* grad, const double* loss2, int64_t step, float lr,
                     hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_adam, dim3((MLP_NP + TPB - 1) / TPB), dim3(TPB), 0, s, theta, m, v, grad, loss2, step,
                     lr);
}

// ----------------------------------------------- element-to-node averages

// out[node][k] (+)= (1/valence(node)) * sum over the node's elements of an
// element value: mode 0, the element mean of the node field in (3
// components, FP64); mode 1, (Vs, rho) of the element's material.  Interior
// nodes are stored, shared nodes added atomically (out cleared beforehand).
template <int K>
__global__ __launch_bounds__(TPB) void k_elem_to_node(MeshDev m, const double* __restrict__ in,
                                                      const uint8_t* __restrict__ emat,
                                                      const MatDev* __restrict__ mats, float* __restrict__ out) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* acc = reinterpret_cast<double*>(smem_raw);
  int32_t* gid = reinterpret_cast<int32_t*>(acc + K * m.max_tile_nodes);
  float* xs = reinterpret_cast<float*>(gid + m.max_tile_nodes);
  const int t = blockIdx.x;
  const int n0 = m.tile_node_off[t];
  const int nt = m.tile_node_off[t + 1] - n0;
  const int nint = m.tile_nint[t];
  const int64_t ib = (int64_t)m.tile_int_base[t];
  for (int j = threadIdx.x; j < nt; j += TPB) gid[j] = m.tile_nodes[n0 + j];
  __syncthreads();
  for (int k = threadIdx.x; k < K * nt; k += TPB) {
    acc[k] = 0.0;
    if constexpr (K == 3) xs[k] = (float)in[3 * (int64_t)gid[k / 3] + (k % 3)];
  }
  __syncthreads();
  for (int e = m.tile_elem_off[t] + threadIdx.x; e < m.tile_elem_off[t + 1]; e += TPB) {
    int ln[10];
    for (int a = 0; a < 10; ++a) ln[a] = conn_node(m, a, e);
    float val[K];
    if constexpr (K == 3) {
      for (int c = 0; c < 3; ++c) {
        float s = 0.0f;
        for (int a = 0; a < 10; ++a) s += xs[3 * ln[a] + c];
        val[c] = 0.1f * s;
      }
    } else {
      const MatDev mt = mats[emat[e]];
      val[0] = (float)(mt.zs / mt.rho);
      val[K - 1] = (float)mt.rho;
    }
    for (int a = 0; a < 10; ++a)
      for (int c = 0; c < K; ++c) atomicAdd(&acc[K * ln[a] + c], (double)val[c]);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < K * nt; k += TPB) {
    const int j = k / K;
    const int64_t g = gid[j];
    const float v = (float)(acc[k] * (double)m.inv_valence[g]);
    if (j < nint)
      out[K * (ib + j) + (k - K * j)] = v;
    else
      atomic_add(&out[K * g + (k - K * j)], v);
  }
}

void launch_neighbour_mean(const MeshDev& m, const double* in, float* out, hipStream_t s) {
  const size_t lds = (size_t)m.max_tile_nodes * (3 * sizeof(double) + sizeof(int32_t) + 3 * sizeof(float));
  hipLaunchKernelGGL(k_elem_to_node<3>, dim3(m.n_tiles), dim3(TPB), lds, s, m, in, (const uint8_t*)nullptr,
                     (const MatDev*)nullptr, out);
}

void launch_node_material(const MeshDev& m, const uint8_t* emat, const MatDev* mats, float* out, hipStream_t s) {
  const size_t lds = (size_t)m.max_tile_nodes * (2 * sizeof(double) + sizeof(int32_t));
  hipLaunchKernelGGL(k_elem_to_node<2>, dim3(m.n_tiles), dim3(TPB), lds, s, m, (const double*)nullptr, emat, mats,
                     out);
}

}  // namespace sw
