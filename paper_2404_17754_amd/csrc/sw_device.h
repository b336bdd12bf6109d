// Device helpers shared by the kernel sources: 64-wide wavefront and
// workgroup reductions, hardware floating-point atomics, grid sizing.
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace sw {

constexpr int TPB = 256;

// One step of a butterfly over a row of 16 lanes, in the vector registers
// (CTRL: a DPP lane selection that permutes the row).
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  union {
    double d;
    int i[2];
  } u{v}, w;
  w.i[0] = __builtin_amdgcn_mov_dpp(u.i[0], CTRL, 0xf, 0xf, true);
  w.i[1] = __builtin_amdgcn_mov_dpp(u.i[1], CTRL, 0xf, 0xf, true);
  return v + w.d;
}
__device__ __forceinline__ double read_lane(double v, int lane) {
  union {
    double d;
    int i[2];
  } u{v};
  u.i[0] = __builtin_amdgcn_readlane(u.i[0], lane);
  u.i[1] = __builtin_amdgcn_readlane(u.i[1], lane);
  return u.d;
}

// Sum over the wavefront, in every lane.  In the vector registers: six
// shuffles through the LDS crossbar cost 0.7 us for a pair of sums, at the
// end of every kernel with a dot product.
__device__ __forceinline__ double wave_sum(double v) {
  v = dpp_add<0xB1>(v);   // lane ^ 1
  v = dpp_add<0x4E>(v);   // lane ^ 2
  v = dpp_add<0x141>(v);  // the other four of eight
  v = dpp_add<0x140>(v);  // the other eight of sixteen
  return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

// Sum of v over a TPB-thread workgroup, valid on thread 0.
__device__ __forceinline__ double block_sum(double v, double* sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) sh[wid] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < TPB / 64; ++i) t += sh[i];
  }
  return t;
}

// Sum of v over an NT-thread workgroup (sh holds NT / 64 doubles), valid on
// thread 0.
template <int NT>
__device__ __forceinline__ double block_sum_n(double v, double* sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) sh[wid] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) t += sh[i];
  }
  return t;
}

// Two sums at once over an NT-thread workgroup (sh holds 2 * NT / 64
// doubles), valid on thread 0.
template <int NT = TPB>
__device__ __forceinline__ void block_sum2(double& a, double& b, double* sh) {
  a = wave_sum(a);
  b = wave_sum(b);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) {
    sh[wid] = a;
    sh[NT / 64 + wid] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    a = 0.0;
    b = 0.0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) {
      a += sh[i];
      b += sh[NT / 64 + i];
    }
  }
}

// Three sums at once over an NT-thread workgroup (sh holds 3 * NT / 64
// doubles), valid on thread 0.
template <int NT>
__device__ __forceinline__ void block_sum3(double& a, double& b, double& c, double* sh) {
  a = wave_sum(a);
  b = wave_sum(b);
  c = wave_sum(c);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) {
    sh[wid] = a;
    sh[NT / 64 + wid] = b;
    sh[2 * NT / 64 + wid] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    a = b = c = 0.0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) {
      a += sh[i];
      b += sh[NT / 64 + i];
      c += sh[2 * NT / 64 + i];
    }
  }
}

// Sums over the times of records that lie pair by pair within a time:
// workgroups of PAIR_NT work-items with MP neighbouring pairs side by side
// (work-item t: pair t % MP), so that a load of many pairs is whole lines and a
// few long records still have many work-items each.  MP by the pairs (misfit
// call, us, at MP = 1 / 4 / 8 / 16): 6 pairs of 20000 steps 38 / 48 / 63 / 97,
// 18 of 100000 253 / 283 / 295 / 426, 60 of 20000 80 / 78 / 91 / 116, 300 of
// 5000 68 / 46 / 48 / 54, 1200 of 20000 586 / 269 / 146 / 171, 9000 of 500
// 135 / 92 / 75 / 68.
constexpr int PAIR_NT = 1024;
template <typename F>
void by_pair_width(int n_pairs, F&& launch) {
  if (n_pairs <= 24)
    launch(std::integral_constant<int, 1>());
  else if (n_pairs <= 300)
    launch(std::integral_constant<int, 4>());
  else if (n_pairs <= 1500)
    launch(std::integral_constant<int, 8>());
  else
    launch(std::integral_constant<int, 16>());
}

// The sums of such a workgroup's values, valid on the first MP work-items; sh
// holds PAIR_NT / 64 * MP doubles.
template <int MP>
__device__ __forceinline__ double pair_sum(double v, double* sh) {
#pragma unroll
  for (int off = MP; off < 64; off *= 2) v += __shfl_xor(v, off, 64);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane < MP) sh[wid * MP + lane] = v;
  __syncthreads();
  if (threadIdx.x < MP) {
    v = 0.0;
#pragma unroll
    for (int k = 0; k < PAIR_NT / 64; ++k) v += sh[k * MP + threadIdx.x];
  }
  return v;
}

// A pointer read from a table in memory, known to point to global memory: its
// loads and stores are global ones (without this they are flat ones, which
// also occupy the LDS counters and wait with the LDS accesses).
template <typename U>
__device__ __forceinline__ U* as_global(U* p) {
  return (U*)(__attribute__((address_space(1))) U*)(uintptr_t)p;
}

__device__ __forceinline__ void atomic_add(double* p, double v) { unsafeAtomicAdd(p, v); }
__device__ __forceinline__ void atomic_add(float* p, float v) { unsafeAtomicAdd(p, v); }

static inline unsigned nblocks(int64_t n) { return (unsigned)((n + TPB - 1) / TPB); }

// Total of N partial sums written by earlier kernels (same address for every
// thread).
template <int N>
__device__ __forceinline__ double slot_sum(const double* s) {
  double t = 0.0;
#pragma unroll
  for (int i = 0; i < N; ++i) t += s[i];
  return t;
}

// Totals of two sets of NSLOT = 32 partial sums, one load per lane of the
// wavefront.  Added up one after the other by every work-item (slot_sum),
// two sets cost 3.3 us at the start of a kernel (the scalar registers hold
// less than one set, so the loads wait for the additions).
__device__ __forceinline__ void slot_sum2(const double* a, const double* b, double& ta, double& tb) {
  const int lane = threadIdx.x & 63;
  double v = lane < 32 ? a[lane] : b[lane - 32];
  v = dpp_add<0xB1>(v);   // lane ^ 1
  v = dpp_add<0x4E>(v);   // lane ^ 2
  v = dpp_add<0x141>(v);  // the other four of eight
  v = dpp_add<0x140>(v);  // the other eight of sixteen
  ta = read_lane(v, 0) + read_lane(v, 16);
  tb = read_lane(v, 32) + read_lane(v, 48);
}

// ---- 3x3 block-Jacobi preconditioner

__device__ __forceinline__ float to_t(__half v, float) { return __half2float(v); }
__device__ __forceinline__ float to_t(float v, float) { return v; }
__device__ __forceinline__ double to_t(double v, double) { return v; }

// the six values (xx yy zz yz xz xy) of node i's block
template <typename T, typename PT>
__device__ __forceinline__ void bj_load(const PT* __restrict__ P, int64_t i, T v[6]) {
#pragma unroll
  for (int k = 0; k < 6; ++k) v[k] = to_t(P[6 * i + k], T());
}
// FP16 blocks: three 32-bit loads of two values each (12-byte records are
// 4-byte aligned)
template <>
__device__ __forceinline__ void bj_load<float, __half>(const __half* __restrict__ P, int64_t i, float v[6]) {
  const __half2* P2 = reinterpret_cast<const __half2*>(P) + 3 * i;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float2 f = __half22float2(P2[k]);
    v[2 * k] = f.x;
    v[2 * k + 1] = f.y;
  }
}

// z = B r for a symmetric 3x3 block (xx yy zz yz xz xy)
template <typename T>
__device__ __forceinline__ void bj_mul(const T v[6], const T r[3], T z[3]) {
  const T a = v[0], b = v[1], c = v[2], yz = v[3], xz = v[4], xy = v[5];
  z[0] = a * r[0] + xy * r[1] + xz * r[2];
  z[1] = xy * r[0] + b * r[1] + yz * r[2];
  z[2] = xz * r[0] + yz * r[1] + c * r[2];
}

// z = P r for the block of node i, stored in PT, applied in T
template <typename T, typename PT>
__device__ __forceinline__ void bj_apply(const PT* __restrict__ P, int64_t i, const T r[3], T z[3]) {
  T v[6];
  bj_load<T, PT>(P, i, v);
  bj_mul(v, r, z);
}

}  // namespace sw
