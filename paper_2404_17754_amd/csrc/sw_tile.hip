// LDS-tiled element-by-element kernels (gfx950).
//
// One workgroup per tile (see sw_mesh.cpp): it gathers the tile's node
// values into LDS, applies every element of the tile (and the boundary
// faces owned by those elements) with LDS atomics into a per-tile
// accumulator, then writes the tile's interior nodes with plain coalesced
// stores and its shared nodes with one global atomic per value.  Against a
// scatter of every element entry to global memory this cuts global atomics
// from 30 per tet to about 2 per tet, and the ones left are address-sorted.
#include <hip/hip_runtime.h>

#include "sw_bf16.h"
#include "sw_device.h"
#include "sw_elem.h"
#include "sw_internal.h"
#include "sw_layout.h"

#include <algorithm>

namespace sw {

// Load through the constant address space: with a uniform index this is a
// scalar load, which is not counted with the vector loads (those complete
// in order, so waiting for one waits for every older one).  For the
// per-tile offsets and counts, constant during a kernel.
template <typename U>
__device__ __forceinline__ U ldc(const U* p, int64_t i) {
  return ((const __attribute__((address_space(4))) U*)p)[i];
}

// A tile's LDS, all of it dynamic (so that it starts at address 0): the input
// values in T first (an element's stored byte offsets address them as they
// are), FP64 accumulators (LDS FP64 atomics are much faster than FP32 ones on
// this target: 25 cycles against 192 at a tile's addresses), room for the
// sums over the workgroup, the ids of the shared nodes, the material table.
template <typename T>
__host__ __device__ constexpr size_t tile_lds_acc(int nmax) {
  return (3 * (size_t)nmax * sizeof(T) + 7) / 8 * 8;
}
constexpr int TILE_SUMS = 24;  // three sums for each wavefront of the largest workgroup
template <typename T>
struct TileLds {
  T* xs;
  double *ys, *sh;
  int32_t* gid;
  T* matl;
  __device__ __forceinline__ TileLds(unsigned char* smem, int nmax)
      : xs(reinterpret_cast<T*>(smem)),
        ys(reinterpret_cast<double*>(smem + tile_lds_acc<T>(nmax))),
        sh(ys + 3 * nmax),
        gid(reinterpret_cast<int32_t*>(sh + TILE_SUMS)),
        matl(reinterpret_cast<T*>(gid + (nmax + (nmax & 1)))) {}
};
template <typename T>
static size_t tile_lds(int nmax, int n_mat) {
  return tile_lds_acc<T>(nmax) + (3 * (size_t)nmax + TILE_SUMS) * sizeof(double) +
         (nmax + (nmax & 1)) * sizeof(int32_t) + 3 * (size_t)n_mat * sizeof(T);
}

// Per-element inputs fetched from global memory in vector loads (5 in FP32,
// 8 in FP64, and the material id): the nodes' offsets, and the precomputed
// barycentric gradients and volume in the pass's precision (coalesced
// streams, no dependent gather).
template <typename T>
struct ElemIn {
  uint4 c8;
  uint32_t c2;
  T geo[10];
  int mid;
  // offset in bytes of node k's first value in an FP32 node array
  __device__ __forceinline__ uint32_t off(int k) const {
    const uint32_t w = k < 2 ? c8.x : k < 4 ? c8.y : k < 6 ? c8.z : k < 8 ? c8.w : c2;
    return k & 1 ? w >> 16 : w & 0xffffu;
  }
};

// element i (0-based) of the tile whose elements start at eb: uniform base
// pointers with one 32-bit offset per array
template <typename T>
__device__ __forceinline__ void load_elem(const MeshDev& m, const uint8_t* __restrict__ emat, int eb, uint32_t i,
                                          ElemIn<T>& o) {
  o.c8 = (m.conn8 + eb)[i];
  o.c2 = (m.conn2 + eb)[i];
  if constexpr (sizeof(T) == 4) {
    const float4* g4 = reinterpret_cast<const float4*>(m.geo32) + eb;
    const float2* g2 = reinterpret_cast<const float2*>(m.geo32 + 8 * m.tet_stride) + eb;
    const float4 a = g4[i], b = (g4 + m.tet_stride)[i];
    const float2 c = g2[i];
    o.geo[0] = a.x, o.geo[1] = a.y, o.geo[2] = a.z, o.geo[3] = a.w;
    o.geo[4] = b.x, o.geo[5] = b.y, o.geo[6] = b.z, o.geo[7] = b.w;
    o.geo[8] = c.x, o.geo[9] = c.y;
  } else {
    const double2* g2 = reinterpret_cast<const double2*>(m.geo64) + eb;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const double2 v = (g2 + k * m.tet_stride)[i];
      o.geo[2 * k] = v.x;
      o.geo[2 * k + 1] = v.y;
    }
  }
  o.mid = (emat + eb)[i];
}

// g_0 = -(g_1 + g_2 + g_3), summed in the order tet_geometry uses, so the
// FP64 operator is the one computed from the coordinates bit for bit
template <typename T>
__device__ __forceinline__ void elem_geometry(const ElemIn<T>& in, Geo<T>& G) {
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    G.g[1][d] = in.geo[d];
    G.g[2][d] = in.geo[3 + d];
    G.g[3][d] = in.geo[6 + d];
    G.g[0][d] = -(in.geo[d] + in.geo[3 + d] + in.geo[6 + d]);
  }
  G.vol = in.geo[9];
}

// Element work of tile t on the values gathered in LDS, accumulated into ys
// (x.A x, which CG passes need, is taken afterwards from the tile's node
// values: tile_scatter).  Work-item i takes the tile's element i, i + NT,
// ...: the layout has grouped the elements of each half-wavefront and
// numbered the tile's interior nodes so that the nodes one LDS instruction
// reaches rarely share a bank (and rarely coincide), while the element loads
// stay coalesced.  PF: the next element's data are loaded before the current
// one is computed (FP32; in FP64 the registers would halve the occupancy).
// STIFF / MASS / DYN: which operator terms are on, and whether each element
// checks its coefficients (element_apply).  hook() runs once, right after the
// first element's loads are issued: the gather of the tile's values, with the
// barrier that ends it.  DET: each element's ten nodal results go to its
// slots of A.eout instead of the LDS accumulator.
template <typename T, int NT, bool PF, bool STIFF, bool MASS, bool DYN, bool DET, typename Hook>
__device__ __forceinline__ void tile_element_loop(const MeshDev& m, const uint8_t* __restrict__ emat,
                                                  const TileArgs<T>& A, int t, const TileLds<T>& lds, Hook&& hook) {
  const T* xs = lds.xs;
  double* ys = lds.ys;
  const T* matl = lds.matl;
  const int eb = ldc(m.tile_elem_off, t);
  const int n_e = ldc(m.tile_elem_off, t + 1) - eb;
  ElemIn<T> nx;
  int i = threadIdx.x;
  if (i < n_e) load_elem<T>(m, emat, eb, i, nx);
  hook();
  for (; i < n_e; i += NT) {
    if (!PF && i != (int)threadIdx.x) load_elem<T>(m, emat, eb, i, nx);
    const ElemIn<T> cur = nx;
    if (PF && i + NT < n_e) load_elem<T>(m, emat, eb, i + NT, nx);
    Geo<T> G;
    elem_geometry(cur, G);
    const T lam = matl[3 * cur.mid], mu = matl[3 * cur.mid + 1], rho = matl[3 * cur.mid + 2];
    T w[10][3];
#pragma unroll
    for (int k = 0; k < 10; ++k) {
#pragma unroll
      for (int c = 0; c < 3; ++c)
        w[k][c] = reinterpret_cast<const T*>(reinterpret_cast<const char*>(xs) + cur.off(k) * (sizeof(T) / 4))[c];
    }
    // each node's force goes to the LDS accumulator as soon as it is
    // complete (no 30-value force array held in registers)
    element_apply<T, STIFF, MASS, DYN>(G, lam, mu, A.sK, A.sM * rho * G.vol, w,
                                  [&](int k, T f0, T f1, T f2) {
                                    if constexpr (DET) {
                                      double* eo = A.eout + (size_t)(eb + i) * 30 + 3 * k;
                                      eo[0] = (double)f0;
                                      eo[1] = (double)f1;
                                      eo[2] = (double)f2;
                                    } else {
                                      double* yk = reinterpret_cast<double*>(reinterpret_cast<char*>(ys) +
                                                                             2 * cur.off(k));
                                      atomicAdd(yk, (double)f0);
                                      atomicAdd(yk + 1, (double)f1);
                                      atomicAdd(yk + 2, (double)f2);
                                    }
                                  });
  }
}

// The boundary faces owned by the elements of tile t (DET: their results to
// the face slots of A.fout).
template <typename T, int NT, bool DET>
__device__ __forceinline__ void tile_faces(const MeshDev& m, const uint8_t* __restrict__ emat,
                                           const MatDev* __restrict__ mats, const TileArgs<T>& A, int t,
                                           const TileLds<T>& lds) {
  const T* xs = lds.xs;
  double* ys = lds.ys;
  if (A.sC != (T)0 || A.vin != nullptr) {
    const int f1 = ldc(m.tile_face_off, t + 1);
    for (int f = ldc(m.tile_face_off, t) + threadIdx.x; f < f1; f += NT) {
      int ln[6];
      int64_t gn[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        ln[k] = m.fconn_loc[k * m.face_stride + f];
        gn[k] = m.fconn[k * m.face_stride + f];
      }
      double P[3][3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
#pragma unroll
        for (int d = 0; d < 3; ++d) P[k][d] = m.xyz[3 * gn[k] + d];
      }
      const FaceGeo g = face_geometry(P);
      const MatDev mt = mats[emat[m.face_elem[f]]];
      T out[6][3];
#pragma unroll
      for (int k = 0; k < 6; ++k) out[k][0] = out[k][1] = out[k][2] = (T)0;
      if (A.sC != (T)0) {
        T w[6][3];
        if (A.xf != nullptr) {
#pragma unroll
          for (int k = 0; k < 6; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) w[k][c] = A.xf[3 * gn[k] + c];
        } else {
          // as LDS accesses (merged with the branch above they become flat ones)
          const auto* xl = (const __attribute__((address_space(3))) T*)xs;
#pragma unroll
          for (int k = 0; k < 6; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) w[k][c] = xl[3 * ln[k] + c];
        }
        const T n[3] = {(T)g.n[0], (T)g.n[1], (T)g.n[2]};
        face_dashpot_apply<T>(n, (T)g.area, (T)mt.zp, (T)mt.zs, A.sC, w, out);
      }
      if (A.vin != nullptr && m.face_role[f] == 2) {
        // incident wave: traction 2 Z v_in, consistent load A/3 on the edge nodes
        const double nv = g.n[0] * A.vin[0] + g.n[1] * A.vin[1] + g.n[2] * A.vin[2];
        const double w3 = g.area / 3.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const T f3 = (T)(w3 * 2.0 * (mt.zs * A.vin[c] + (mt.zp - mt.zs) * nv * g.n[c]));
          out[3][c] += f3;
          out[4][c] += f3;
          out[5][c] += f3;
        }
      }
      if constexpr (DET) {
        double* fo = A.fout + (size_t)f * 18;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
#pragma unroll
          for (int c = 0; c < 3; ++c) fo[3 * k + c] = (double)out[k][c];
        }
      } else {
#pragma unroll
        for (int k = 0; k < 6; ++k) {
#pragma unroll
          for (int c = 0; c < 3; ++c) atomicAdd(&ys[3 * ln[k] + c], (double)out[k][c]);
        }
      }
    }
  }
}

// Which terms a pass has, fixed at compile time where that pays: TERMS_A the
// stiffness and the mass (CG passes, FP32: no per-node branches), TERMS_ANY
// checked per element (FP64, where the branch-free form needs more registers
// than the passes can spare).
enum { TERMS_ANY = 0, TERMS_A = 1 };

// Element and face work of tile t.
template <typename T, int NT, bool PF, int TERMS, bool DET, typename Hook>
__device__ __forceinline__ void tile_elements(const MeshDev& m, const uint8_t* __restrict__ emat,
                                              const MatDev* __restrict__ mats, const TileArgs<T>& A, int t,
                                              const TileLds<T>& lds, Hook&& hook) {
  if constexpr (TERMS == TERMS_A)
    tile_element_loop<T, NT, PF, true, true, false, DET>(m, emat, A, t, lds, hook);
  else if (A.sK != (T)0 || A.sM != (T)0)
    tile_element_loop<T, NT, PF, true, true, true, DET>(m, emat, A, t, lds, hook);
  else
    hook();
  tile_faces<T, NT, DET>(m, emat, mats, A, t, lds);
}

// Results of tile t: interior nodes (one contiguous range) with plain
// stores, shared nodes with address-sorted global atomics.  Returns this
// work-item's share of the tile's x.(A x)_tile = sum over the tile's nodes
// of the input value times the tile's partial sum: summed over the tiles it
// is x.A x (a node's full value is the sum of its tiles' partials), with one
// product per node value instead of one per element entry.  USER: the
// interior nodes go to A.yu in the user's node order (gid holds their ids).
template <typename T, int NT, bool USER = false>
__device__ __forceinline__ double tile_scatter(const MeshDev& m, const TileArgs<T>& A, int t,
                                               const TileLds<T>& lds) {
  const T* xs = lds.xs;
  const double* ys = lds.ys;
  const int nt = ldc(m.tile_node_off, t + 1) - ldc(m.tile_node_off, t);
  const int nint = ldc(m.tile_nint, t);
  const int64_t ib3 = 3 * (int64_t)ldc(m.tile_int_base, t);
  T* __restrict__ y = A.y;
  double energy = 0.0;
  for (int k = threadIdx.x; k < 3 * nint; k += NT) {
    const double v = ys[k];
    energy += (double)xs[k] * v;
    if constexpr (USER) {
      const int j = k / 3;
      A.yu[3 * (int64_t)lds.gid[j] + (k - 3 * j)] = (T)v;
    } else {
      y[ib3 + k] = (T)v;
    }
  }
  // shared nodes: address-sorted global atomics
  for (int k = 3 * nint + threadIdx.x; k < 3 * nt; k += NT) {
    const int j = k / 3;
    const double v = ys[k];
    energy += (double)xs[k] * v;
    atomic_add(&y[3 * (int64_t)lds.gid[j] + (k - 3 * j)], (T)v);
  }
  return energy;
}

// A tile's nodes, NPT per work-item: the interior ones are one contiguous
// range of ids, the shared ones come from the tile's node list.  A work-item
// past the last node holds node 0 (a valid address, loaded and unused).
template <int NT, int NPT>
struct TileNodes {
  int nt, nint;
  int32_t g[NPT];
  __device__ __forceinline__ void load(const MeshDev& m, int t) {
    const int n0 = ldc(m.tile_node_off, t);
    nt = ldc(m.tile_node_off, t + 1) - n0;
    nint = ldc(m.tile_nint, t);
    const int ib = ldc(m.tile_int_base, t);
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
      const int j = threadIdx.x + q * NT;
      g[q] = j < nint ? ib + j : 0;
      if (j >= nint && j < nt) g[q] = m.tile_nodes[n0 + j];
    }
  }
};
// Work-items 256 take five nodes each, 512 three: the largest tile.
template <int NT>
constexpr int tile_npt() {
  return (TILE_MAX_NODES + NT - 1) / NT;
}

// The material table (lam, mu, rho per material), rounded to T, into LDS: a
// load from global memory would wait on the element's material id.
// The first NT values are loaded (mat_load) well before they are stored.
__device__ __forceinline__ double mat_load(const MatDev* __restrict__ mats, int n_mat, int i) {
  return i < 3 * n_mat ? (&mats[i / 3].lam)[i % 3] : 0.0;
}
template <typename T, int NT>
__device__ __forceinline__ void mat_store(const MatDev* __restrict__ mats, int n_mat, double first, T* matl) {
  if ((int)threadIdx.x < 3 * n_mat) matl[threadIdx.x] = (T)first;
  for (int i = threadIdx.x + NT; i < 3 * n_mat; i += NT) matl[i] = (T)mat_load(mats, n_mat, i);
}

// Input of a pass: x1; a1 x1 + a2 x2; x1 in bfloat16 (x1h); x1 in the user's
// node order (A.map: the nodes' user ids), the results of the interior nodes
// then going to A.yu in that order too: that gather and scatter take the place
// of two kernels that permute the vectors.  9.6 M tets, FP32: this pass 428 us
// and 83 for the shared nodes' results (k_shared_out), against 326 and 290.
// (The shared nodes added in the user's order by atomics: 770 in all, the
// addresses of a wavefront then lying in as many cache lines.)
enum { IN_ONE = 0, IN_TWO = 1, IN_BF16 = 2, IN_USER = 3 };

template <typename T, int NT, int IN, int NPT>
__device__ __forceinline__ void tile_gather(const TileArgs<T>& A, const TileNodes<NT, NPT>& N,
                                            const TileLds<T>& lds) {
  // every load before the first is waited for: one memory latency a tile
  T v[NPT][3], u[IN == IN_TWO ? NPT : 1][3];
  int32_t uid[IN == IN_USER ? NPT : 1];
  if constexpr (IN == IN_USER) {
#pragma unroll
    for (int q = 0; q < NPT; ++q) uid[q] = A.map[N.g[q]];
  }
#pragma unroll
  for (int q = 0; q < NPT; ++q) {
    const int64_t g3 = 3 * (int64_t)(IN == IN_USER ? uid[q] : N.g[q]);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if constexpr (IN == IN_BF16)
        v[q][c] = bf16_value(A.x1h[g3 + c]);
      else
        v[q][c] = A.x1[g3 + c];
      if constexpr (IN == IN_TWO) u[q][c] = A.x2[g3 + c];
    }
  }
#pragma unroll
  for (int q = 0; q < NPT; ++q) {
    const int j = threadIdx.x + q * NT;
    if (j < N.nt) {
      lds.gid[j] = IN == IN_USER && j < N.nint ? uid[q] : N.g[q];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if constexpr (IN == IN_TWO) v[q][c] = A.a1 * v[q][c] + A.a2 * u[q][c];
        lds.xs[3 * j + c] = v[q][c];
        lds.ys[3 * j + c] = 0.0;
      }
    }
  }
}

// One tile of an operator pass; returns the work-item's share of x.A x.
// DET: the element and face results go to their slots (no scatter, no energy;
// the node pass and a fixed-order dot product follow).
template <typename T, int NT, int IN, int TERMS, bool DET>
__device__ __forceinline__ double tile_body(const MeshDev& m, const uint8_t* __restrict__ emat,
                                            const MatDev* __restrict__ mats, const TileArgs<T>& A, int t,
                                            const TileLds<T>& lds) {
  TileNodes<NT, tile_npt<NT>()> N;
  N.load(m, t);
  const double mat = mat_load(mats, A.n_mat, threadIdx.x);
  tile_elements<T, NT, sizeof(T) == 4, TERMS, DET>(m, emat, mats, A, t, lds, [&] {
    mat_store<T, NT>(mats, A.n_mat, mat, lds.matl);
    tile_gather<T, NT, IN>(A, N, lds);
    __syncthreads();
  });
  if constexpr (DET) return 0.0;
  __syncthreads();
  return tile_scatter<T, NT, IN == IN_USER>(m, A, t, lds);
}

// One tile of the right-hand side pass,
//   y = sM M (a1 x1 + a2 x2) + sC C_abs xf + F(vin) + sK K (k1 + k2 x2):
// the mass on its input, then the stiffness on the other, which waits in
// registers (30 of the mass loop's spare ones) for its turn in the LDS.  Two
// passes gather v and add every shared node to global memory twice: with the
// permutation of the result 1.55 ms on 9.6 M tets, this pass 1.08, with the
// interior nodes stored in the user's order (USER, as in tile_scatter) 1.04.
template <int NT, bool USER>
__device__ __forceinline__ void tile_rhs(const MeshDev& m, const uint8_t* __restrict__ emat,
                                         const MatDev* __restrict__ mats, const TileArgs<double>& A, int t,
                                         const TileLds<double>& lds) {
  constexpr int NPT = tile_npt<NT>();
  TileNodes<NT, NPT> N;
  N.load(m, t);
  const double mat = mat_load(mats, A.n_mat, threadIdx.x);
  double kv[NPT][3];
  tile_element_loop<double, NT, false, false, true, false, false>(m, emat, A, t, lds, [&] {
    mat_store<double, NT>(mats, A.n_mat, mat, lds.matl);
    double v1[NPT][3], v2[NPT][3];
    int32_t uid[USER ? NPT : 1];
    if constexpr (USER) {
#pragma unroll
      for (int q = 0; q < NPT; ++q) uid[q] = A.map[N.g[q]];
    }
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
      const int64_t g3 = 3 * (int64_t)N.g[q];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        v1[q][c] = A.x1[g3 + c];
        v2[q][c] = A.x2[g3 + c];
        kv[q][c] = A.k1[g3 + c];
      }
    }
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
      const int j = threadIdx.x + q * NT;
#pragma unroll
      for (int c = 0; c < 3; ++c) kv[q][c] += A.k2 * v2[q][c];
      if (j < N.nt) {
        lds.gid[j] = N.g[q];
        if constexpr (USER) {
          if (j < N.nint) lds.gid[j] = uid[q];
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          lds.xs[3 * j + c] = A.a1 * v1[q][c] + A.a2 * v2[q][c];
          lds.ys[3 * j + c] = 0.0;
        }
      }
    }
    __syncthreads();
  });
  tile_faces<double, NT, false>(m, emat, mats, A, t, lds);
  tile_element_loop<double, NT, false, true, false, false, false>(m, emat, A, t, lds, [&] {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
      const int j = threadIdx.x + q * NT;
      if (j < N.nt) {
#pragma unroll
        for (int c = 0; c < 3; ++c) lds.xs[3 * j + c] = kv[q][c];
      }
    }
    __syncthreads();
  });
  __syncthreads();
  tile_scatter<double, NT, USER>(m, A, t, lds);
}

// Share of n tiles (or work items) of workgroup b: XCD x = b mod 8
// (workgroups are dealt to the 8 XCDs round-robin) takes the contiguous
// eighth [lo, hi), so that neighbouring tiles, which share nodes, meet in one
// L2; this workgroup the items lo + first, + step, ...
struct XcdShare {
  int at, hi, step;
  __device__ __forceinline__ explicit XcdShare(int n) {
    const int xcd = blockIdx.x & 7;
    at = (int)(((int64_t)n * xcd) >> 3) + (int)(blockIdx.x >> 3);
    hi = (int)(((int64_t)n * (xcd + 1)) >> 3);
    step = gridDim.x >> 3;
  }
};

// Operator pass of one case.  iter >= 0: as part of CG iteration `iter` (x.A x
// into ctl->pAp[0]; nothing when the solve is done; the first iteration ends
// a solve whose residual meets the tolerance; the first workgroup clears the
// scalar slots the next update kernel accumulates into).
// FP32, 9.6 M tets: 326-335 us (1.16 GB moved: 3.5 TB/s).  Of the compute
// units' busy cycles the vector units issue in 73 % and the LDS works in 65 %
// (a third of that bank conflicts), and the waves wait half of theirs: latency
// that three wavefronts per SIMD (LDS: 46 KB a tile) do not cover.  With the
// element data in single words and the next tile's values loaded behind the
// elements of the one before it took 347 us; that pipeline costs 40 registers,
// which now hold the next element's data.  FP64: 867 us a pass with the values gathered one after the
// other, 620 with every load issued before the first is waited for.
// LOOP: a workgroup walks several tiles (a capped grid), else it has one.
template <typename T, int NT, int IN, int TERMS, bool DET, bool LOOP>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 3 : 2))) void k_tile(
    MeshDev m, const uint8_t* __restrict__ emat, const MatDev* __restrict__ mats, TileArgs<T> A, CgCtl* ctl,
    int iter) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const TileLds<T> lds(smem_raw, m.max_tile_nodes);
  if (iter >= 0) {
    const int par = iter & 1;
    if (ctl->done) return;
    if (iter == 0 && slot_sum<NSLOT>(ctl->rr[0]) <= ctl->tol2) {
      if (blockIdx.x == 0 && threadIdx.x == 0) ctl->done = 1;
      return;
    }
    if (blockIdx.x == 0 && threadIdx.x < NSLOT) {
      ctl->rz[par ^ 1][threadIdx.x] = 0.0;
      ctl->rr[par ^ 1][threadIdx.x] = 0.0;
    }
  }
  const XcdShare share(m.n_tiles);
  if (share.at >= share.hi) return;
  double energy = tile_body<T, NT, IN, TERMS, DET>(m, emat, mats, A, share.at, lds);
  if constexpr (LOOP) {
    for (int t = share.at + share.step; t < share.hi; t += share.step) {
      __syncthreads();
      energy += tile_body<T, NT, IN, TERMS, DET>(m, emat, mats, A, t, lds);
    }
  }
  if (!DET && iter >= 0) {
    const double s = block_sum_n<NT>(energy, lds.sh);
    if (threadIdx.x == 0) atomic_add(&ctl->pAp[0][blockIdx.x % NSLOT], s);
  }
}

// Deterministic node pass: y[ystride * i + yoff + c] (= or +=) the sum over
// node i's element slots, then its face slots, in increasing slot order
// (elems / faces: whether the pass wrote them).  A CG iteration (iter >= 0)
// whose solve is done does nothing.
__global__ __launch_bounds__(TPB) void k_node_gather(MeshDev m, const double* __restrict__ eout,
                                                     const double* __restrict__ fout, double* __restrict__ y,
                                                     int ystride, int yoff, int accumulate, int elems, int faces,
                                                     const CgCtl* ctl, int iter) {
  if (iter >= 0 && ctl->done) return;
  for (int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x; i < m.n_nodes; i += (int64_t)gridDim.x * TPB) {
    double a[3] = {0.0, 0.0, 0.0};
    if (elems)
      for (int j = m.inc_off[i]; j < m.inc_off[i + 1]; ++j) {
        const double* e = eout + 3 * (size_t)m.inc[j];
        a[0] += e[0];
        a[1] += e[1];
        a[2] += e[2];
      }
    if (faces)
      for (int j = m.finc_off[i]; j < m.finc_off[i + 1]; ++j) {
        const double* f = fout + 3 * (size_t)m.finc[j];
        a[0] += f[0];
        a[1] += f[1];
        a[2] += f[2];
      }
    double* yi = y + (int64_t)ystride * i + yoff;
#pragma unroll
    for (int c = 0; c < 3; ++c) yi[c] = accumulate ? yi[c] + a[c] : a[c];
  }
}

// slots[b] = workgroup b's share of x.y, one workgroup per slot (a
// fixed-order sum); nothing when the CG solve in ctl is done.
__global__ __launch_bounds__(TPB) void k_dot_slots(int64_t n, const double* __restrict__ x,
                                                   const double* __restrict__ y, double* __restrict__ slots,
                                                   const CgCtl* ctl) {
  __shared__ double sh[2 * TPB / 64];
  if (ctl->done) return;
  double acc = 0.0;
  for (int64_t k = (int64_t)blockIdx.x * TPB + threadIdx.x; k < n; k += (int64_t)gridDim.x * TPB) acc += x[k] * y[k];
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) slots[blockIdx.x] = acc;
}

template <int NT, bool USER>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void k_tile_rhs(
    MeshDev m, const uint8_t* __restrict__ emat, const MatDev* __restrict__ mats, TileArgs<double> A) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const TileLds<double> lds(smem_raw, m.max_tile_nodes);
  const XcdShare share(m.n_tiles);
  if (share.at < share.hi) tile_rhs<NT, USER>(m, emat, mats, A, share.at, lds);
}

// A lane's tables and vectors as pointers to global memory (as_global).
template <typename T>
__device__ __forceinline__ TileLane<T> lane_of(const TileLane<T>* lanes, int l) {
  TileLane<T> L = lanes[l];
  L.m.conn8 = as_global(L.m.conn8);
  L.m.conn2 = as_global(L.m.conn2);
  L.m.tile_elem_off = as_global(L.m.tile_elem_off);
  L.m.tile_node_off = as_global(L.m.tile_node_off);
  L.m.tile_nodes = as_global(L.m.tile_nodes);
  L.m.tile_int_base = as_global(L.m.tile_int_base);
  L.m.tile_nint = as_global(L.m.tile_nint);
  L.m.tile_face_off = as_global(L.m.tile_face_off);
  L.m.xyz = as_global(L.m.xyz);
  L.m.geo32 = as_global(L.m.geo32);
  L.m.geo64 = as_global(L.m.geo64);
  L.m.fconn = as_global(L.m.fconn);
  L.m.fconn_loc = as_global(L.m.fconn_loc);
  L.m.face_elem = as_global(L.m.face_elem);
  L.m.face_role = as_global(L.m.face_role);
  L.emat = as_global(L.emat);
  L.mats = as_global(L.mats);
  L.A.x1 = as_global(L.A.x1);
  L.A.x2 = as_global(L.A.x2);
  L.A.k1 = as_global(L.A.k1);
  L.A.xf = as_global(L.A.xf);
  L.A.vin = as_global(L.A.vin);
  L.A.y = as_global(L.A.y);
  L.ctl = as_global(L.ctl);
  return L;
}

// The same pass for several cases (lanes) in one launch: work item b is
// (lane, tile) = work[b] (lane < 0: padding), lanes whose state is inactive
// return at once.  RHS: the right-hand side pass, else A applied to x1.
template <typename T, int NT, bool RHS>
__global__ __launch_bounds__(NT) void k_tile_lanes(const TileLane<T>* __restrict__ lanes,
                                                    const int2* __restrict__ work,
                                                    const LaneState* __restrict__ st) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int2 w = work[blockIdx.x];
  if (w.x < 0) return;
  if (st != nullptr && !st[w.x].active) return;
  const TileLane<T> L = lane_of(lanes, w.x);
  const TileLds<T> lds(smem_raw, L.m.max_tile_nodes);
  if constexpr (RHS)
    tile_rhs<NT, false>(L.m, L.emat, L.mats, L.A, w.y, lds);
  else
    tile_body<T, NT, IN_ONE, TERMS_ANY, false>(L.m, L.emat, L.mats, L.A, w.y, lds);
}

// FP32 operator pass of a CG iteration over the (lane, tile) items of several
// cases: items[k] = (lane, tile), tile-major with the lanes of a tile
// adjacent (they share the tile's mesh data through L2).  An item is skipped
// when its lane is inactive or its solve is done (or, on the first iteration,
// already converged): every workgroup evaluates the same condition, so a
// skipped lane's output is left untouched; the workgroup of the tile-0 item
// marks an already converged lane done, and else clears the slots the lane's
// next update kernel accumulates into.  nmax: the largest tile over the lanes
// (LDS layout).
template <int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(3))) void k_tile_lanes_cg(
    const TileLane<float>* __restrict__ lanes, const int2* __restrict__ items, int n_items, int nmax,
    const LaneState* __restrict__ st, int iter) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const TileLds<float> lds(smem_raw, nmax);
  const int par = iter & 1;
  XcdShare share(n_items);
  for (int k = share.at; k < share.hi; k += share.step) {
    // the same in every lane of the workgroup: readfirstlane tells the
    // compiler so, which keeps the lane's pointers in scalar registers
    const int2 item = items[k];
    const int l = __builtin_amdgcn_readfirstlane(item.x), t = __builtin_amdgcn_readfirstlane(item.y);
    if (st != nullptr && !st[l].active) continue;
    const TileLane<float> L = lane_of(lanes, l);
    CgCtl* c = L.ctl;
    if (c->done) continue;
    if (iter == 0 && slot_sum<NSLOT>(c->rr[0]) <= c->tol2) {
      if (t == 0 && threadIdx.x == 0) c->done = 1;
      continue;
    }
    if (t == 0 && threadIdx.x < NSLOT) {
      c->rz[par ^ 1][threadIdx.x] = 0.0;
      c->rr[par ^ 1][threadIdx.x] = 0.0;
    }
    const double energy = tile_body<float, NT, IN_ONE, TERMS_A, false>(L.m, L.emat, L.mats, L.A, t, lds);
    const double e = block_sum_n<NT>(energy, lds.sh);
    if (threadIdx.x == 0) atomic_add(&c->pAp[0][t % NSLOT], e);
    __syncthreads();
  }
}

// Operator pass of a two-kernel CG iteration (k_cg_step follows it), bound by
// latency: its chain is launch, control block and node ids (1.4 us), the
// values of z and p_old (1 us), the elements (4.4 us, half of it the LDS
// atomics of one compute unit), the scatter and the sum (1.2 us).  The
// direction p = z + beta p_old is formed while the tile's nodes are gathered
// and the tile's own nodes of p are stored, so the iteration has no direction
// kernel.  One workgroup per tile.  p_old and p are two buffers, since
// neighbouring tiles still read p_old; a tile stores its interior nodes and
// the shared nodes no earlier tile touches (tile_own_base).
// par: the iteration's parity; first: the solve's first iteration (p = z).
template <typename T, int NT, int WPE>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WPE))) void k_tile_dir(
    MeshDev m, const uint8_t* __restrict__ emat, const MatDev* __restrict__ mats, TileArgs<T> A,
    const T* __restrict__ p_old, T* __restrict__ p, CgCtl* ctl, int par, int first, int max_iter) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const TileLds<T> lds(smem_raw, m.max_tile_nodes);
  constexpr int NPT = tile_npt<NT>();
  const XcdShare share(m.n_tiles);
  const int t = share.at;
  const bool lead = blockIdx.x == 0, has_tile = t < share.hi;
  TileNodes<NT, NPT> N;
  int own = 0;
  if (has_tile) {
    N.load(m, t);
    own = ldc(m.tile_own_base, t);
  }
  const double mat = mat_load(mats, A.n_mat, threadIdx.x);
  // the previous iteration's residual decides whether this one runs: the
  // same test in every workgroup, on values no workgroup of this launch writes
  const double tol2 = ctl->tol2, rz_prev = ctl->rz_prev;
  const int iters = ctl->iters, done = ctl->done;
  double rr, rz;
  slot_sum2(ctl->rr[par], ctl->rz[par], rr, rz);
  const T beta = first ? (T)0 : (T)(rz / rz_prev);
  const bool stop = first ? rr <= tol2 : (!(rr > tol2) || iters >= max_iter);  // NaN stops too
  if (done) return;
  if (stop) {
    if (lead && threadIdx.x == 0) ctl->done = 1;
    return;
  }
  if (lead && threadIdx.x < NSLOT) {
    ctl->rz[par ^ 1][threadIdx.x] = 0.0;
    ctl->rr[par ^ 1][threadIdx.x] = 0.0;
  }
  if (!has_tile) return;
  const T* __restrict__ z = A.x1;
  auto gather = [&] {
    mat_store<T, NT>(mats, A.n_mat, mat, lds.matl);
    T zv[NPT][3], pv[NPT][3];
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
#pragma unroll
      for (int c = 0; c < 3; ++c) zv[q][c] = z[3 * (int64_t)N.g[q] + c];
    }
    if (!first) {
#pragma unroll
      for (int q = 0; q < NPT; ++q) {
#pragma unroll
        for (int c = 0; c < 3; ++c) pv[q][c] = p_old[3 * (int64_t)N.g[q] + c];
      }
    } else {
#pragma unroll
      for (int q = 0; q < NPT; ++q) pv[q][0] = pv[q][1] = pv[q][2] = (T)0;
    }
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
      const int j = threadIdx.x + q * NT;
      if (j < N.nt) {
        lds.gid[j] = N.g[q];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const T v = zv[q][c] + beta * pv[q][c];
          lds.xs[3 * j + c] = v;
          lds.ys[3 * j + c] = 0.0;
          if (j < N.nint || N.g[q] >= own) p[3 * (int64_t)N.g[q] + c] = v;
        }
      }
    }
    __syncthreads();
  };
  tile_elements<T, NT, sizeof(T) == 4 && NT == 256, sizeof(T) == 4 ? TERMS_A : TERMS_ANY, false>(m, emat, mats, A, t,
                                                                                                lds, gather);
  __syncthreads();
  const double energy = tile_scatter<T, NT>(m, A, t, lds);
  const double e = block_sum_n<NT>(energy, lds.sh);
  if (threadIdx.x == 0) atomic_add(&ctl->pAp[par][t % NSLOT], e);
}

// A whole CG iteration in one kernel.  With the operator applied to the
// preconditioned residual u_k = P r_k instead of the direction, w_k = A u_k,
// both sums that iteration k + 1 needs, r_k.u_k and u_k.A u_k, come from one
// pass (the conjugate gradients of Chronopoulos and Gear, 1989):
//   beta = rz_k / rz_(k-1),  alpha = rz_k / (u_k.A u_k - beta rz_k / alpha')
//   p = u_k + beta p,  s = w_k + beta s (= A p),  x += alpha p,  r -= alpha s
// Kernel k does these updates for its tile's nodes with the sums of kernel
// k - 1, forms u_k and applies the operator.  A node of several tiles is
// updated by each of them, in the same arithmetic on the same values, and
// stored by one (its first), so r and s have two buffers; w has three: read,
// added into, cleared for the next kernel.  The sums are kept mod 3 alike.
// stage: 0 the solve's first kernel (no update yet), 1 the second (no
// previous direction), 2 later ones.
// Bound by latency, as k_tile_dir, whose chain it has, with more loads in the
// gather and without the second kernel's launch, sums and pass over the
// vectors (5 us): a step of 6 tiles 0.97 -> 0.92 ms, of 375 tiles 2.03 ->
// 1.94, in FP64 of 186 tiles 2.34 -> 2.18.
template <typename T, typename PT, int NT, int NPT, int WPE>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WPE))) void k_tile_cg(
    MeshDev m, const uint8_t* __restrict__ emat, const MatDev* __restrict__ mats, TileArgs<T> A, OneCg<T> V,
    const PT* __restrict__ P, CgCtl* ctl, int ring, int par, int stage, int max_iter) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const TileLds<T> lds(smem_raw, m.max_tile_nodes);
  const XcdShare share(m.n_tiles);
  const int t = share.at;
  const bool lead = blockIdx.x == 0, has_tile = t < share.hi;
  TileNodes<NT, NPT> N;
  int own = 0;
  if (has_tile) {
    N.load(m, t);
    own = ldc(m.tile_own_base, t);
  }
  const double mat = mat_load(mats, A.n_mat, threadIdx.x);
  // the previous kernel's sums: the same test in every workgroup, on values
  // no workgroup of this launch writes
  const int last = stage == 0 ? 0 : (ring == 0 ? 2 : ring - 1), next = ring == 2 ? 0 : ring + 1;
  const double tol2 = ctl->tol2, rz_prev = ctl->one_rz[par ^ 1], alpha_prev = ctl->one_alpha[par ^ 1];
  const int iters = ctl->one_iters[par ^ 1], done = ctl->done;
  double rr, rz, uAu, unused;
  slot_sum2(ctl->rr[last], ctl->rz[last], rr, rz);
  slot_sum2(ctl->pAp[last], ctl->pAp[last], uAu, unused);
  const double beta_d = stage < 2 ? 0.0 : rz / rz_prev;
  const double alpha_d = rz / (stage < 2 ? uAu : uAu - beta_d * rz / alpha_prev);
  const T alpha = (T)alpha_d, beta = (T)beta_d;
  bool stop = false;  // a NaN stops all but the first iteration
  if (stage == 0) stop = rr <= tol2;
  if (stage == 2) stop = !(rr > tol2) || iters >= max_iter;
  if (done) return;
  if (stop) {
    if (lead && threadIdx.x == 0) ctl->done = 1;
    return;
  }
  if (lead) {
    if (threadIdx.x < NSLOT) {
      ctl->rz[next][threadIdx.x] = 0.0;
      ctl->rr[next][threadIdx.x] = 0.0;
      ctl->pAp[next][threadIdx.x] = 0.0;
    }
    if (stage > 0 && threadIdx.x == 0) {
      ctl->one_rz[par] = rz;
      ctl->one_alpha[par] = alpha_d;
      ctl->one_iters[par] = iters + 1;
    }
  }
  if (!has_tile) return;
  double rz_new = 0.0, rr_new = 0.0;
  auto gather = [&] {
    mat_store<T, NT>(mats, A.n_mat, mat, lds.matl);
    T rv[NPT][3], sv[NPT][3], wv[NPT][3], bl[NPT][6], pv[NPT][3], xv[NPT][3];
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
#pragma unroll
      for (int c = 0; c < 3; ++c) rv[q][c] = V.r_old[3 * (int64_t)N.g[q] + c];
      bj_load<T, PT>(P, N.g[q], bl[q]);
    }
    if (stage > 0) {
#pragma unroll
      for (int q = 0; q < NPT; ++q) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          wv[q][c] = V.w_old[3 * (int64_t)N.g[q] + c];
          xv[q][c] = V.x[3 * (int64_t)N.g[q] + c];
        }
      }
    }
    if (stage > 1) {
#pragma unroll
      for (int q = 0; q < NPT; ++q) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          sv[q][c] = V.s_old[3 * (int64_t)N.g[q] + c];
          pv[q][c] = V.p[3 * (int64_t)N.g[q] + c];
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < NPT; ++q) {
#pragma unroll
        for (int c = 0; c < 3; ++c) sv[q][c] = pv[q][c] = (T)0;
      }
    }
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
      const int j = threadIdx.x + q * NT;
      if (j < N.nt) {
        const int64_t g3 = 3 * (int64_t)N.g[q];
        const bool mine = j < N.nint || N.g[q] >= own;
        T r[3], u[3];
        if (stage > 0) {
          if (mine) {
            bj_mul(bl[q], rv[q], u);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              const T p = u[c] + beta * pv[q][c];
              V.p[g3 + c] = p;
              V.x[g3 + c] = xv[q][c] + alpha * p;
            }
          }
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            sv[q][c] = wv[q][c] + beta * sv[q][c];
            r[c] = rv[q][c] - alpha * sv[q][c];
          }
        } else {
#pragma unroll
          for (int c = 0; c < 3; ++c) r[c] = rv[q][c];
        }
        bj_mul(bl[q], r, u);
        lds.gid[j] = N.g[q];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          lds.xs[3 * j + c] = u[c];
          lds.ys[3 * j + c] = 0.0;
        }
        if (mine) {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            if (stage > 0) {
              V.r_new[g3 + c] = r[c];
              V.s_new[g3 + c] = sv[q][c];
              rz_new += (double)r[c] * (double)u[c];
              rr_new += (double)r[c] * (double)r[c];
            }
            if (j >= N.nint) V.w_clear[g3 + c] = (T)0;
          }
        }
      }
    }
    __syncthreads();
  };
  tile_elements<T, NT, sizeof(T) == 4 && NT == 256, sizeof(T) == 4 ? TERMS_A : TERMS_ANY, false>(m, emat, mats, A, t,
                                                                                                lds, gather);
  __syncthreads();
  double energy = tile_scatter<T, NT>(m, A, t, lds);
  block_sum3<NT>(energy, rz_new, rr_new, lds.sh);
  if (threadIdx.x == 0) {
    atomic_add(&ctl->pAp[ring][t % NSLOT], energy);
    if (stage > 0) {
      atomic_add(&ctl->rz[ring][t % NSLOT], rz_new);
      atomic_add(&ctl->rr[ring][t % NSLOT], rr_new);
    }
  }
}

// Workgroups of a pass over n tiles (or items): one each, a multiple of 8 (an
// eighth per XCD); at most `cap` when cap > 0, each then walking several.
static unsigned pass_grid(int n, int cap) {
  int per_xcd = std::max(1, (n + 7) / 8);
  if (cap > 0) per_xcd = std::max(1, std::min(per_xcd, cap / 8));
  return (unsigned)(8 * per_xcd);
}

template <typename T, int IN, int TERMS, bool DET>
static void launch_pass(const MeshDev& m, const uint8_t* emat, const MatDev* mats, const TileArgs<T>& a, CgCtl* ctl,
                        int iter, int grid_cap, hipStream_t s) {
  constexpr int NT = 256;
  const unsigned g = pass_grid(m.n_tiles, 0), gc = pass_grid(m.n_tiles, grid_cap);
  const size_t lds = tile_lds<T>(m.max_tile_nodes, a.n_mat);
  if constexpr (sizeof(T) == 4) {
    if (gc < g) {
      hipLaunchKernelGGL((k_tile<T, NT, IN, TERMS, DET, true>), dim3(gc), dim3(NT), lds, s, m, emat, mats, a, ctl,
                         iter);
      return;
    }
  }
  hipLaunchKernelGGL((k_tile<T, NT, IN, TERMS, DET, false>), dim3(g), dim3(NT), lds, s, m, emat, mats, a, ctl, iter);
}

// Whether a solve's iterations, past the reach of one kernel, run as two
// (k_tile_dir, k_cg_step) rather than three.  In FP64 always: 1374 us an
// iteration (share of the step's other work included) against 1597 on 9.6 M
// tets.  In FP32 up to 4000 tiles: 128 us against 141 at 3000 tiles, but 270
// against 255 at 6750, where the vectors no longer stay in the caches and the
// non-temporal accesses of the three kernels gain more.  A cap on the pass's
// workgroups that binds asks for workgroups that walk several tiles: three
// kernels.
constexpr int TWO_KERNEL_TILES_F32 = 4000;
bool two_kernel_cg(const MeshDev& m, int grid_cap, bool f32) {
  return !f32 || (m.n_tiles <= TWO_KERNEL_TILES_F32 && (grid_cap == 0 || grid_cap >= m.n_tiles));
}

// FP32: 512 work-items, one element each in a full tile, two workgroups per
// compute unit (four waves per SIMD): 48 us an iteration against 53 with 256
// at 844 tiles.  FP64 needs twice the registers, room for one workgroup of 512
// per compute unit: 45.6 us against 41.4 with 256 at 375 tiles.
template <typename T>
static void launch_tile_dir(const MeshDev& m, const uint8_t* emat, const MatDev* mats, const TileArgs<T>& a,
                            const T* p_old, T* p, CgCtl* ctl, int iter, int max_iter, hipStream_t s) {
  constexpr bool f32 = sizeof(T) == 4;
  constexpr int NT = f32 ? 512 : 256;
  hipLaunchKernelGGL((k_tile_dir<T, NT, f32 ? 4 : 2>), dim3(pass_grid(m.n_tiles, 0)), dim3(NT),
                     tile_lds<T>(m.max_tile_nodes, a.n_mat), s, m, emat, mats, a, p_old, p, ctl, iter & 1, iter == 0,
                     max_iter);
}
void launch_tile_dir_f64(const MeshDev& m, const uint8_t* emat, const MatDev* mats, const TileArgs<double>& a,
                         const double* p_old, double* p, CgCtl* ctl, int iter, int max_iter, hipStream_t s) {
  launch_tile_dir<double>(m, emat, mats, a, p_old, p, ctl, iter, max_iter, s);
}
void launch_tile_dir_f32(const MeshDev& m, const uint8_t* emat, const MatDev* mats, const TileArgs<float>& a,
                         const float* p_old, float* p, CgCtl* ctl, int iter, int max_iter, hipStream_t s) {
  launch_tile_dir<float>(m, emat, mats, a, p_old, p, ctl, iter, max_iter, s);
}

// Whether a solve's iterations run as one kernel (k_tile_cg), with one
// workgroup a tile.  Against two kernels, us an iteration (share of the step's
// other work included): FP32 11.8 / 14.4 at 48 tiles, 16.1 / 18.2 at 256, 24.6
// / 26.4 at 375, 57.3 / 59.7 at 1266, 72.3 / 74.5 at 1736, but 90.2 / 88.6 at
// 2187; FP64 11.7 / 14.4 at 48 tiles, 34.8 / 37.1 at 375, 64.6 / 67.4 at 824,
// but 108 / 92 at 1266: there the vectors and preconditioner blocks of the
// nodes that several tiles update cost more than the launch saved.
constexpr int ONE_KERNEL_TILES_F32 = 1800, ONE_KERNEL_TILES_F64 = 900;
bool one_kernel_cg(const MeshDev& m, int grid_cap, bool f32) {
  return m.n_tiles <= (f32 ? ONE_KERNEL_TILES_F32 : ONE_KERNEL_TILES_F64) &&
         (grid_cap == 0 || grid_cap >= m.n_tiles);
}

// NPT: nodes per work-item, as few as the largest tile needs (a node past the
// tile's last is loaded all the same): 12.3 us an iteration with three and
// 11.4 with one at 48 tiles of 64 elements.
template <typename T, typename PT, int NT, int NPT, int WPE>
static void launch_tile_cg(const MeshDev& m, const uint8_t* emat, const MatDev* mats, const TileArgs<T>& a,
                           const OneCg<T>& v, const PT* P, CgCtl* ctl, int iter, int max_iter, hipStream_t s) {
  if constexpr (NPT > 1) {
    if (m.max_tile_nodes <= NT * (NPT - 1)) {
      launch_tile_cg<T, PT, NT, NPT - 1, WPE>(m, emat, mats, a, v, P, ctl, iter, max_iter, s);
      return;
    }
  }
  hipLaunchKernelGGL((k_tile_cg<T, PT, NT, NPT, WPE>), dim3(pass_grid(m.n_tiles, 0)), dim3(NT),
                     tile_lds<T>(m.max_tile_nodes, a.n_mat), s, m, emat, mats, a, v, P, ctl, iter % 3, iter & 1,
                     iter < 2 ? iter : 2, max_iter);
}
void launch_tile_cg_f64(const MeshDev& m, const uint8_t* emat, const MatDev* mats, const TileArgs<double>& a,
                        const OneCg<double>& v, const double* P, CgCtl* ctl, int iter, int max_iter, hipStream_t s) {
  // FP64 leaves room for one workgroup of 512 per compute unit: 4.15 ms a step
  // against 3.50 with 256 at 375 tiles
  if (m.n_tiles <= 256)
    launch_tile_cg<double, double, 512, tile_npt<512>(), 2>(m, emat, mats, a, v, P, ctl, iter, max_iter, s);
  else
    launch_tile_cg<double, double, 256, tile_npt<256>(), 2>(m, emat, mats, a, v, P, ctl, iter, max_iter, s);
}
void launch_tile_cg_f32(const MeshDev& m, const uint8_t* emat, const MatDev* mats, const TileArgs<float>& a,
                        const OneCg<float>& v, const __half* P, CgCtl* ctl, int iter, int max_iter, hipStream_t s) {
  launch_tile_cg<float, __half, 512, tile_npt<512>(), 4>(m, emat, mats, a, v, P, ctl, iter, max_iter, s);
}

static unsigned node_grid(int64_t n_nodes) {
  unsigned g = nblocks(n_nodes);
  return g > 8192 ? 8192 : (g == 0 ? 1 : g);
}

void launch_tile_f64(const MeshDev& m, const uint8_t* emat, const MatDev* mats, const TileArgs<double>& a,
                     CgCtl* ctl, int iter, hipStream_t s) {
  if (!a.eout) {
    if (a.map)
      launch_pass<double, IN_USER, TERMS_ANY, false>(m, emat, mats, a, ctl, iter, 0, s);
    else
      launch_pass<double, IN_ONE, TERMS_ANY, false>(m, emat, mats, a, ctl, iter, 0, s);
    return;
  }
  // deterministic: element and face slots, the node pass in slot order, and
  // p.Ap as a fixed-order dot product (a CG pass has x1 = p)
  if (a.x2)
    launch_pass<double, IN_TWO, TERMS_ANY, true>(m, emat, mats, a, ctl, iter, 0, s);
  else
    launch_pass<double, IN_ONE, TERMS_ANY, true>(m, emat, mats, a, ctl, iter, 0, s);
  const int elems = a.sK != 0.0 || a.sM != 0.0, faces = a.sC != 0.0 || a.vin != nullptr;
  hipLaunchKernelGGL(k_node_gather, dim3(node_grid(m.n_nodes)), dim3(TPB), 0, s, m, a.eout, a.fout, a.y, 3, 0,
                     a.accumulate, elems, faces, ctl, iter);
  if (iter >= 0)
    hipLaunchKernelGGL(k_dot_slots, dim3(NSLOT), dim3(TPB), 0, s, 3 * m.n_nodes, a.x1, a.y, ctl->pAp[0], ctl);
}
void launch_tile_f32(const MeshDev& m, const uint8_t* emat, const MatDev* mats, const TileArgs<float>& a,
                     CgCtl* ctl, int iter, int grid_cap, hipStream_t s) {
  if (a.sK != 0.0f && a.sM != 0.0f) {
    if (a.x1h)
      launch_pass<float, IN_BF16, TERMS_A, false>(m, emat, mats, a, ctl, iter, grid_cap, s);
    else if (a.map)
      launch_pass<float, IN_USER, TERMS_A, false>(m, emat, mats, a, ctl, iter, grid_cap, s);
    else
      launch_pass<float, IN_ONE, TERMS_A, false>(m, emat, mats, a, ctl, iter, grid_cap, s);
  } else if (a.map) {
    launch_pass<float, IN_USER, TERMS_ANY, false>(m, emat, mats, a, ctl, iter, grid_cap, s);
  } else {
    launch_pass<float, IN_ONE, TERMS_ANY, false>(m, emat, mats, a, ctl, iter, grid_cap, s);
  }
}

void launch_tile_rhs(const MeshDev& m, const uint8_t* emat, const MatDev* mats, const TileArgs<double>& a,
                     hipStream_t s) {
  const dim3 grid(pass_grid(m.n_tiles, 0));
  const size_t lds = tile_lds<double>(m.max_tile_nodes, a.n_mat);
  if (a.map)
    hipLaunchKernelGGL((k_tile_rhs<256, true>), grid, dim3(256), lds, s, m, emat, mats, a);
  else
    hipLaunchKernelGGL((k_tile_rhs<256, false>), grid, dim3(256), lds, s, m, emat, mats, a);
}

void launch_tile_lanes_f64(const TileLane<double>* lanes, const int2* work, int n_work, int max_tile_nodes, int max_mat,
                           bool rhs, const LaneState* st, hipStream_t s) {
  const size_t lds = tile_lds<double>(max_tile_nodes, max_mat);
  if (rhs)
    hipLaunchKernelGGL((k_tile_lanes<double, 256, true>), dim3(n_work), dim3(256), lds, s, lanes, work, st);
  else
    hipLaunchKernelGGL((k_tile_lanes<double, 256, false>), dim3(n_work), dim3(256), lds, s, lanes, work, st);
}
void launch_tile_lanes_f32(const TileLane<float>* lanes, const int2* items, int n_items, int max_tile_nodes,
                           int max_mat, const LaneState* st, int iter, int grid_cap, hipStream_t s) {
  hipLaunchKernelGGL((k_tile_lanes_cg<256>), dim3(pass_grid(n_items, grid_cap)), dim3(256),
                     tile_lds<float>(max_tile_nodes, max_mat), s, lanes, items, n_items, max_tile_nodes, st, iter);
}

// ------------------------------------------------------------ geometry

// Barycentric gradients (rows of the inverse Jacobian, L1..L3) and the volume
// of every element from the FP64 coordinates, in FP64 (geo64) and rounded to
// FP32 (geo32).
__global__ __launch_bounds__(TPB) void k_geom(MeshDev m, float* __restrict__ geo32, double* __restrict__ geo64) {
  __shared__ int32_t gid[TILE_MAX_NODES];
  const int t = blockIdx.x;
  const int n0 = m.tile_node_off[t];
  const int nt = m.tile_node_off[t + 1] - n0;
  for (int j = threadIdx.x; j < nt; j += TPB) gid[j] = m.tile_nodes[n0 + j];
  __syncthreads();
  for (int e = m.tile_elem_off[t] + threadIdx.x; e < m.tile_elem_off[t + 1]; e += TPB) {
    double X[4][3];
    for (int k = 0; k < 4; ++k) {
      const int64_t g = gid[conn_node(m, k, e)];
      for (int d = 0; d < 3; ++d) X[k][d] = m.xyz[3 * g + d];
    }
    Geo<double> G;
    tet_geometry<double>(X, G);
    const double v[10] = {G.g[1][0], G.g[1][1], G.g[1][2], G.g[2][0], G.g[2][1],
                          G.g[2][2], G.g[3][0], G.g[3][1], G.g[3][2], G.vol};
    double2* g64 = reinterpret_cast<double2*>(geo64);
    float4* g32 = reinterpret_cast<float4*>(geo32);
#pragma unroll
    for (int k = 0; k < 5; ++k) g64[k * m.tet_stride + e] = make_double2(v[2 * k], v[2 * k + 1]);
#pragma unroll
    for (int k = 0; k < 2; ++k)
      g32[k * m.tet_stride + e] =
          make_float4((float)v[4 * k], (float)v[4 * k + 1], (float)v[4 * k + 2], (float)v[4 * k + 3]);
    reinterpret_cast<float2*>(geo32 + 8 * m.tet_stride)[e] = make_float2((float)v[8], (float)v[9]);
  }
}

__global__ __launch_bounds__(TPB) void k_pack_conn(int64_t stride, const uint16_t* __restrict__ c,
                                                   uint4* __restrict__ conn8, uint32_t* __restrict__ conn2) {
  const int64_t e = (int64_t)blockIdx.x * TPB + threadIdx.x;
  if (e >= stride) return;
  uint32_t w[5];
#pragma unroll
  for (int k = 0; k < 5; ++k)
    w[k] = 4u * c[(2 * k) * stride + e] | (4u * c[(2 * k + 1) * stride + e]) << 16;
  conn8[e] = make_uint4(w[0], w[1], w[2], w[3]);
  conn2[e] = w[4];
}
void launch_pack_conn(const MeshDev& m, const uint16_t* conn_loc, uint4* conn8, uint32_t* conn2, hipStream_t s) {
  hipLaunchKernelGGL(k_pack_conn, dim3(nblocks(m.tet_stride)), dim3(TPB), 0, s, m.tet_stride, conn_loc, conn8, conn2);
}

void launch_geom(const MeshDev& m, float* geo32, double* geo64, hipStream_t s) {
  hipLaunchKernelGGL(k_geom, dim3(m.n_tiles), dim3(TPB), 0, s, m, geo32, geo64);
}

// ------------------------------------------------------------ diagonal

// DET: values 3 half .. 3 half + 2 of each node's block go to the element
// and face slots (eout, fout) instead of the LDS accumulator; a node pass
// sums them in slot order.
template <bool DET>
__global__ __launch_bounds__(TPB) void k_tile_diag(MeshDev m, const uint8_t* __restrict__ emat,
                                                   const MatDev* __restrict__ mats, double cM, double cK, double cC,
                                                   double* __restrict__ diag6, int half, double* __restrict__ eout,
                                                   double* __restrict__ fout) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* ds = reinterpret_cast<double*>(smem_raw);
  const int t = blockIdx.x;
  const int n0 = m.tile_node_off[t];
  const int nt = m.tile_node_off[t + 1] - n0;
  const int nint = m.tile_nint[t];
  const int64_t ib6 = 6 * (int64_t)m.tile_int_base[t];
  const int32_t* __restrict__ gid = m.tile_nodes + n0;
  for (int k = threadIdx.x; k < 6 * nt; k += TPB) ds[k] = 0.0;
  __syncthreads();
  const int e1 = m.tile_elem_off[t + 1];
  for (int e = m.tile_elem_off[t] + threadIdx.x; e < e1; e += TPB) {
    int ln[10];
    for (int k = 0; k < 10; ++k) ln[k] = conn_node(m, k, e);
    double X[4][3];
    for (int k = 0; k < 4; ++k)
      for (int d = 0; d < 3; ++d) X[k][d] = m.xyz[3 * (int64_t)gid[ln[k]] + d];
    Geo<double> G;
    tet_geometry<double>(X, G);
    const MatDev mt = mats[emat[e]];
    double out[10][6];
    diag_blocks<double>(G, mt.lam, mt.mu, mt.rho, cM, cK, out);
    if constexpr (DET) {
      // static register indices (a run-time index would put out[][] in scratch)
#pragma unroll
      for (int k = 0; k < 10; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c)
          eout[30 * (size_t)e + 3 * k + c] = half ? out[k][3 + c] : out[k][c];
    } else {
      for (int k = 0; k < 10; ++k)
        for (int j = 0; j < 6; ++j) atomicAdd(&ds[6 * ln[k] + j], out[k][j]);
    }
  }
  if (cC != 0.0) {
    const int f1 = m.tile_face_off[t + 1];
    for (int f = m.tile_face_off[t] + threadIdx.x; f < f1; f += TPB) {
      double P[3][3];
      for (int k = 0; k < 3; ++k)
        for (int d = 0; d < 3; ++d) P[k][d] = m.xyz[3 * (int64_t)m.fconn[k * m.face_stride + f] + d];
      const FaceGeo g = face_geometry(P);
      const MatDev mt = mats[emat[m.face_elem[f]]];
      const double dz = mt.zp - mt.zs;
      const double Z[6] = {mt.zs + dz * g.n[0] * g.n[0], mt.zs + dz * g.n[1] * g.n[1], mt.zs + dz * g.n[2] * g.n[2],
                           dz * g.n[1] * g.n[2],         dz * g.n[0] * g.n[2],         dz * g.n[0] * g.n[1]};
      for (int k = 0; k < 6; ++k) {
        const int l = m.fconn_loc[k * m.face_stride + f];
        const double sc = cC * g.area / 180.0 * (k < 3 ? 6.0 : 32.0);
        if constexpr (DET) {
#pragma unroll
          for (int c = 0; c < 3; ++c) fout[18 * (size_t)f + 3 * k + c] = sc * (half ? Z[3 + c] : Z[c]);
        } else {
          for (int j = 0; j < 6; ++j) atomicAdd(&ds[6 * l + j], sc * Z[j]);
        }
      }
    }
  }
  if constexpr (DET) return;
  __syncthreads();
  for (int k = threadIdx.x; k < 6 * nint; k += TPB) diag6[ib6 + k] = ds[k];
  for (int k = 6 * nint + threadIdx.x; k < 6 * nt; k += TPB) {
    const int j = k / 6;
    atomic_add(&diag6[6 * (int64_t)gid[j] + (k - 6 * j)], ds[k]);
  }
}

void launch_tile_diag(const MeshDev& m, const uint8_t* emat, const MatDev* mats, double cM, double cK, double cC,
                      double* diag6, hipStream_t s, double* eout, double* fout) {
  const size_t lds = 6 * (size_t)m.max_tile_nodes * sizeof(double);
  if (!eout) {
    hipLaunchKernelGGL(k_tile_diag<false>, dim3(m.n_tiles), dim3(TPB), lds, s, m, emat, mats, cM, cK, cC, diag6, 0,
                       nullptr, nullptr);
    return;
  }
  for (int half = 0; half < 2; ++half) {
    hipLaunchKernelGGL(k_tile_diag<true>, dim3(m.n_tiles), dim3(TPB), lds, s, m, emat, mats, cM, cK, cC, diag6, half,
                       eout, fout);
    hipLaunchKernelGGL(k_node_gather, dim3(node_grid(m.n_nodes)), dim3(TPB), 0, s, m, eout, fout, diag6, 6, 3 * half,
                       0, 1, cC != 0.0 ? 1 : 0, nullptr, -1);
  }
}

// Inverse of each symmetric 3x3 block [[a xy xz][xy b yz][xz yz c]] by
// cofactors, in FP64; FP32 copy for the mixed-precision inner solve.
__global__ void k_fill_zero_d(double* p) { *p = 0.0; }

__global__ __launch_bounds__(TPB) void k_invert(int64_t n, const double* __restrict__ d6, double* __restrict__ p64,
                                                double* pmax, int* bad) {
  __shared__ double sh[TPB / 64];
  const int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x;
  double mx = 0.0;
  if (i < n) {
    const double a = d6[6 * i + 0], b = d6[6 * i + 1], c = d6[6 * i + 2];
    const double yz = d6[6 * i + 3], xz = d6[6 * i + 4], xy = d6[6 * i + 5];
    const double c00 = b * c - yz * yz, c11 = a * c - xz * xz, c22 = a * b - xy * xy;
    const double c12 = -(a * yz - xy * xz), c02 = xy * yz - b * xz, c01 = -(xy * c - yz * xz);
    const double det = a * c00 + xy * c01 + xz * c02;
    if (!(det > 0.0) || !(a > 0.0)) *bad = 1;
    const double id = 1.0 / det;
    const double r[6] = {c00 * id, c11 * id, c22 * id, c12 * id, c02 * id, c01 * id};
    for (int k = 0; k < 6; ++k) p64[6 * i + k] = r[k];
    mx = fmax(fmax(r[0], r[1]), r[2]);
    if (!(mx > 0.0)) mx = 0.0;
  }
  // largest diagonal entry: positive doubles order like their bit patterns
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < TPB / 64; ++w) mx = fmax(mx, sh[w]);
    mx = fmax(mx, sh[0]);
    atomicMax(reinterpret_cast<unsigned long long*>(pmax), (unsigned long long)__double_as_longlong(mx));
  }
}

__global__ __launch_bounds__(TPB) void k_to_half(int64_t n6, const double* __restrict__ p64,
                                                 const double* __restrict__ pmax, __half* __restrict__ p16) {
  const double s = *pmax > 0.0 ? 1.0 / *pmax : 0.0;
  for (int64_t k = (int64_t)blockIdx.x * TPB + threadIdx.x; k < n6; k += (int64_t)gridDim.x * TPB)
    p16[k] = __float2half((float)(p64[k] * s));
}

void launch_invert_blocks(int64_t n_nodes, const double* diag6, double* pinv64, __half* pinv16, double* pmax,
                          int* bad, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_zero_d, dim3(1), dim3(1), 0, s, pmax);
  hipLaunchKernelGGL(k_invert, dim3(nblocks(n_nodes)), dim3(TPB), 0, s, n_nodes, diag6, pinv64, pmax, bad);
  unsigned g = nblocks(6 * n_nodes);
  if (g > 8192) g = 8192;
  hipLaunchKernelGGL(k_to_half, dim3(g), dim3(TPB), 0, s, 6 * n_nodes, pinv64, pmax, pinv16);
}

}  // namespace sw
