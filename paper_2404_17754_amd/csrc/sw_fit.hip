// Input estimation of Section 2 on the GPU (gfx950): the records' side of
// the least-squares problem.
//
// The input along j is sum_l c_jl p(t - l dT), dT = m time steps; the
// response is U_i^k(t) = sum_{j,l} G_ij^k(t - l m) c_jl with G_j the Green's
// records (velocity along i at receiver k for the unit impulse along j).
// With the record cut into nb = n_steps / m blocks of m steps, every entry
// of the normal equations is a sum of block inner products
//     C[(j,b), (j',b')] = sum_{k,i} w_ki sum_{r<m} G_j[b m + r] G_j'[b' m + r]
// (and the same with the observed record in place of G_j'), so one weighted
// Gram matrix of 4 nb block columns (3 nb of Green's blocks, nb of observed
// blocks) holds all of them; the host sums its diagonals into A and b.
#include <hip/hip_runtime.h>

#include "sw_device.h"
#include "sw_internal.h"

namespace sw {

// o2[pair] = sum_t obs[t][pair]^2: MP neighbouring pairs by PAIR_NT / MP times a
// workgroup (by_pair_width)
template <int MP>
__global__ __launch_bounds__(PAIR_NT) void k_fit_pair_norms(int n_pairs, int64_t n_steps,
                                                            const double* __restrict__ obs, double* __restrict__ o2) {
  __shared__ double sh[PAIR_NT / 64 * MP];
  const int pr = blockIdx.x * MP + threadIdx.x % MP;
  double s = 0.0;
  if (pr < n_pairs) {
#pragma unroll 4
    for (int64_t t = threadIdx.x / MP; t < n_steps; t += PAIR_NT / MP) {
      const double o = obs[t * n_pairs + pr];
      s += o * o;
    }
  }
  s = pair_sum<MP>(s, sh);
  if (threadIdx.x < MP && pr < n_pairs) o2[pr] = s;
}

// w[pair] = 1 / o2[pair], zero for pairs whose norm is <= 1e-12 of the
// largest (silent records carry no weight)
__global__ __launch_bounds__(TPB) void k_fit_weights(int n_pairs, const double* __restrict__ o2,
                                                     double* __restrict__ w) {
  __shared__ double sh[TPB / 64];
  __shared__ double smax;
  double mx = 0.0;
  for (int i = threadIdx.x; i < n_pairs; i += TPB) mx = fmax(mx, sqrt(o2[i]));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    double m = 0.0;
    for (int i = 0; i < TPB / 64; ++i) m = fmax(m, sh[i]);
    smax = m;
  }
  __syncthreads();
  const double thr = 1e-12 * smax;
  for (int i = threadIdx.x; i < n_pairs; i += TPB) {
    const double nrm = sqrt(o2[i]);
    w[i] = nrm > thr ? 1.0 / o2[i] : 0.0;
  }
}

// Block column `col` (< 4 nb) at row (r, pair): Green's block (j, b) for
// col = j nb + b (j < 3), observed block b for col = 3 nb + b.
struct FitSrc {
  const double* g[3];
  const double* obs;
  int n_pairs, m, nb;
};

__device__ __forceinline__ const double* fit_col(const FitSrc& S, int col) {
  const int j = col / S.nb, b = col - j * S.nb;
  return (j < 3 ? S.g[j] : S.obs) + (int64_t)b * S.m * S.n_pairs;
}

// C = X^T diag(w) X for the 4 nb block columns, on the FP64 matrix
// instructions (16x16x4), 64 x 64 output tiles (the upper ones).  The m times
// of a block by the pairs are one contiguous run of rows in the records, taken
// in chunks of FK across the times (with chunks that ended at each time, three
// pairs filled 3 of a chunk's 32 rows).  A workgroup takes a share (blockIdx.y) of the chunks, and the shares' results
// are added in their order by k_fit_sum, since the few tiles of a fit (10 at
// 200 columns) would leave most of the chip idle.  Four wavefronts of 32 x 32.
// 200 columns of 24000 rows: 1354 us with one output per work-item and rows
// read pair by pair (one value of a line), 134 so.
typedef double doublex4 __attribute__((ext_vector_type(4)));
constexpr int FT = 64, FK = 32, FLD = FK + 1;
__global__ __launch_bounds__(256) void k_fit_gram(FitSrc S, const double* __restrict__ w, int ncol, int nt,
                                                  double* __restrict__ part) {
  __shared__ double xa[FT * FLD], xb[FT * FLD];
  // tile pair (ta <= tb) of the upper triangle
  int ta = 0, rest = blockIdx.x;
  while (rest >= nt - ta) rest -= nt - ta++;
  const int tb = ta + rest;
  const int tid = threadIdx.x, l = tid & 63, wv = tid >> 6;
  const int64_t rows = (int64_t)S.m * S.n_pairs, chunks = (rows + FK - 1) / FK;
  const int64_t c0 = chunks * blockIdx.y / gridDim.y, c1 = chunks * (blockIdx.y + 1) / gridDim.y;
  // each work-item loads row kk of a chunk of columns row0, row0 + 8, ...
  const int kk = tid % FK, row0 = tid / FK;
  constexpr int PER = FT * FK / 256;
  const double *pa[PER], *pb[PER];  // null past the last column
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int ca = ta * FT + row0 + q * (256 / FK), cb = tb * FT + row0 + q * (256 / FK);
    pa[q] = ca < ncol ? fit_col(S, ca) : nullptr;
    pb[q] = cb < ncol ? fit_col(S, cb) : nullptr;
  }
  double ra[PER], rb[PER];
  // the row's pair, moved along from chunk to chunk
  int pair = (int)((c0 * FK + kk) % S.n_pairs);
  const int pair_step = FK % S.n_pairs;
  auto load = [&](int64_t c) {
    const int64_t at = c * FK + kk;
    const bool in = at < rows;
    const double wp = in ? w[pair] : 0.0;
    pair += pair_step;
    if (pair >= S.n_pairs) pair -= S.n_pairs;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      ra[q] = in && pa[q] ? wp * pa[q][at] : 0.0;
      rb[q] = in && pb[q] ? pb[q][at] : 0.0;
    }
  };
  doublex4 acc[2][2] = {};
  const int a0 = (wv >> 1) * 32 + (l & 15), b0 = (wv & 1) * 32 + (l & 15), k0 = l >> 4;
  if (c0 < c1) load(c0);
  for (int64_t c = c0; c < c1; ++c) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      xa[(row0 + q * (256 / FK)) * FLD + kk] = ra[q];
      xb[(row0 + q * (256 / FK)) * FLD + kk] = rb[q];
    }
    __syncthreads();
    if (c + 1 < c1) load(c + 1);
#pragma unroll
    for (int k = 0; k < FK; k += 4) {
      double av[2], bv[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        av[i] = xa[(a0 + 16 * i) * FLD + k + k0];
        bv[i] = xb[(b0 + 16 * i) * FLD + k + k0];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i], bv[j], acc[i][j], 0, 0, 0);
    }
  }
  // result rows 4 v + l / 16, column l % 16 of each 16 x 16 block
  double* out = part + (size_t)blockIdx.y * ncol * ncol;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = ta * FT + (wv >> 1) * 32 + 16 * i + 4 * v + (l >> 4), col = tb * FT + b0 + 16 * j;
        if (row < ncol && col < ncol && row <= col) out[(size_t)row * ncol + col] = acc[i][j][v];
      }
}

// C's upper triangle = the sum of the shares in their order, mirrored (the
// (a, b) and (b, a) products round differently: one of them serves both).
// part may be C itself when there is one share.  A row of workgroups takes
// every SUM_ROWS-th row: the second grid dimension ends at 65535.
constexpr int SUM_ROWS = 1024;
__global__ __launch_bounds__(TPB) void k_fit_sum(int ncol, int shares, const double* part, double* C) {
  const int col = blockIdx.x * TPB + threadIdx.x;
  for (int row = blockIdx.y; row < ncol; row += SUM_ROWS) {
    if (col >= ncol || col < row) continue;
    const size_t at = (size_t)row * ncol + col;
    double s = 0.0;
    for (int k = 0; k < shares; ++k) s += part[(size_t)k * ncol * ncol + at];
    C[at] = s;
    C[(size_t)col * ncol + row] = s;
  }
}

// U[t][pair] = sum_j sum_{l <= t/m, l < n_shift} c[j][l] G_j[t - l m][pair]:
// at the same (r, pair) the times b m + r are a convolution over the blocks b;
// a work-item makes OB consecutive blocks, so that a record value is loaded
// once for OB results.  cp: the coefficients with zeros at both ends.  50
// blocks and shifts, 1200 pairs: 108 us with a load per product, 24 so.
constexpr int OB = 8;
__global__ __launch_bounds__(TPB) void k_fit_response(FitSrc S, int n_shift, const double* __restrict__ c,
                                                      double* __restrict__ U) {
  extern __shared__ double cp[];
  const int ld = n_shift + 2 * OB;
  for (int i = threadIdx.x; i < 3 * ld; i += TPB) {
    const int j = i / ld, k = i - j * ld - OB;
    cp[i] = k >= 0 && k < n_shift ? c[j * n_shift + k] : 0.0;
  }
  __syncthreads();
  const int64_t stride = (int64_t)S.m * S.n_pairs, x = (int64_t)blockIdx.x * TPB + threadIdx.x;
  if (x >= stride) return;
  const int b0 = blockIdx.y * OB;
  double acc[OB];
#pragma unroll
  for (int o = 0; o < OB; ++o) acc[o] = 0.0;
  // source block i reaches result block b0 + o through shift b0 + o - i
  const int i0 = max(0, b0 - n_shift + 1), i1 = min(S.nb, b0 + OB);
  for (int j = 0; j < 3; ++j) {
    const double* g = S.g[j] + x;
    const double* cj = cp + j * ld + OB + b0;
#pragma unroll 4
    for (int i = i0; i < i1; ++i) {
      const double v = g[i * stride];
#pragma unroll
      for (int o = 0; o < OB; ++o) acc[o] += cj[o - i] * v;
    }
  }
#pragma unroll
  for (int o = 0; o < OB; ++o)
    if (b0 + o < S.nb) U[(b0 + o) * stride + x] = acc[o];
}

void launch_fit_weights(int n_pairs, int64_t n_steps, const double* obs, double* o2, double* w, hipStream_t s) {
  by_pair_width(n_pairs, [&](auto w) {
    constexpr int MP = decltype(w)::value;
    hipLaunchKernelGGL(k_fit_pair_norms<MP>, dim3((n_pairs + MP - 1) / MP), dim3(PAIR_NT), 0, s, n_pairs, n_steps, obs,
                       o2);
  });
  hipLaunchKernelGGL(k_fit_weights, dim3(1), dim3(TPB), 0, s, n_pairs, o2, w);
}

void launch_fit_gram(const double* const g[3], const double* obs, int n_pairs, int m, int nb, const double* w,
                     double* C, double* scratch, int64_t scratch_len, hipStream_t s) {
  FitSrc S{{g[0], g[1], g[2]}, obs, n_pairs, m, nb};
  const int ncol = 4 * nb, nt = (ncol + FT - 1) / FT, tiles = nt * (nt + 1) / 2;
  // shares: two workgroups per compute unit, as far as there are chunks and
  // room for the shares' results
  const int64_t chunks = ((int64_t)m * n_pairs + FK - 1) / FK, room = scratch_len / ((int64_t)ncol * ncol);
  int64_t shares = (512 + tiles - 1) / tiles;
  shares = shares < chunks ? shares : chunks;
  shares = shares < room ? shares : room;
  double* part = shares > 1 ? scratch : C;
  if (shares < 1) shares = 1;
  hipLaunchKernelGGL(k_fit_gram, dim3(tiles, (unsigned)shares), dim3(256), 0, s, S, w, ncol, nt, part);
  hipLaunchKernelGGL(k_fit_sum, dim3((ncol + TPB - 1) / TPB, ncol < SUM_ROWS ? ncol : SUM_ROWS), dim3(TPB), 0, s, ncol,
                     (int)shares, part, C);
}

void launch_fit_response(const double* const g[3], int n_pairs, int m, int n_shift, int64_t n_steps,
                         const double* c, double* U, hipStream_t s) {
  FitSrc S{{g[0], g[1], g[2]}, nullptr, n_pairs, m, (int)(n_steps / m)};
  const size_t lds = 3 * (size_t)(n_shift + 2 * OB) * sizeof(double);
  hipLaunchKernelGGL(k_fit_response, dim3(nblocks((int64_t)m * n_pairs), (S.nb + OB - 1) / OB), dim3(TPB), lds, s, S,
                     n_shift, c, U);
}

}  // namespace sw
