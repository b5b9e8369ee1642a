// Device helpers shared by the operator kernels: mesh arguments and the
// sum-factorization sweep over LDS tiles.
#pragma once

#include <hip/hip_runtime.h>

#include "ctab.h"
#include "dgwm_internal.h"

namespace dgwm {

// Everything a kernel needs about the mesh, passed by value.
struct MeshDev {
  int nx, ny, nz;
  int fully_periodic;
  int lower_slot, upper_slot, nslots;  // enriched-layer slots (-1: wall not enriched)
  double hx, hz;
  const double* hy;   // ny cell heights
  double ihx, ihz;    // 1 / hx, 1 / hz
  const double* ihy;  // ny reciprocal cell heights
  const double* tab;  // 1-D tables (tab_layout)
  const double* psi;  // [enr][psi_pts][4]
  int psi_pts;
  int psi_off[7];     // offsets of volume (0) and faces 0..5 inside one cell's psi table
  double nu, theta;
  double pen;         // ip_factor (k+1)^2
  double wall_mult;
  int64_t enr_off;    // start of the enrichment block in the velocity vector
  // curved geometry (nullptr for affine box cells)
  const double* geo;  // [cell][geo_stride][J^{-1} (9), weight]
  int geo_stride;
  const double* tauF; // [cell][face]
  int nq_wn;          // wall-normal points of enriched cells (the point layout of their tables)
  const double* nut;  // eddy viscosity [enr][psi_pts] of the multiscale viscous operator (else nullptr)
  int ops_off;        // offset of the Poisson operator tables (poi_ops) inside tab
  int lin_off;        // offset of the velocity's 1-D operators (lin_ops) inside tab
  int proj_off;       // offset of the projection table
};

// Enriched index of cell (ex, ey, ez) or -1.
__device__ __forceinline__ int64_t enr_index(const MeshDev& M, int ex, int ey, int ez) {
  if (M.fully_periodic) return -1;
  int slot = -1;
  if (ey == 0 && M.lower_slot >= 0) slot = M.lower_slot;
  else if (ey == M.ny - 1 && M.upper_slot >= 0) slot = M.upper_slot;
  if (slot < 0) return -1;
  return ex + M.nx * (slot + M.nslots * ez);  // below 2^31 like the cell count
}

// The mesh's 1-D tables in the constant address space: uniform reads become
// scalar loads, also where the pointer itself comes from memory (batched
// launches).  The tables are written once, at set-up.  Every call gives a
// pointer that the compiler takes for a new one, so coefficients are loaded
// again where they are used instead of being held (and spilled) in between.
template <typename T>
using ConstTab = const __attribute__((address_space(4))) T*;
template <typename T>
__device__ __forceinline__ ConstTab<T> const_tab(const double* p) {
  const uintptr_t a = (uintptr_t)p;
  uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)a), hi = __builtin_amdgcn_readfirstlane((int)(a >> 32));
  asm volatile("" : "+s"(lo), "+s"(hi));
  return (ConstTab<T>)((uintptr_t)lo | ((uintptr_t)hi << 32));
}

// Neighbour of cell e = (ex, ey, ez) across face (D, S), or -1 for a wall.
__device__ __forceinline__ int cell_nb(const MeshDev& M, int e, int ex, int ey, int ez, int D, int S) {
  const int j = D == 0 ? ex : (D == 1 ? ey : ez);
  const int nmax = D == 0 ? M.nx : (D == 1 ? M.ny : M.nz);
  const int step = D == 0 ? 1 : (D == 1 ? M.nx : M.nx * M.ny);
  if (S ? j == nmax - 1 : j == 0) {
    if (D == 1 && !M.fully_periodic) return -1;
    return S ? e - (nmax - 1) * step : e + (nmax - 1) * step;
  }
  return S ? e + step : e - step;
}

// Line (a, b) of nodes along direction D (a, b: indices of the tangential
// directions in order): first node and stride in a cell's vector.
template <int NP>
__device__ __forceinline__ void vec_line(int D, int a, int b, int& base, int& stride) {
  base = D == 0 ? NP * (a + NP * b) : (D == 1 ? a + NP * NP * b : a + NP * b);
  stride = D == 0 ? 1 : (D == 1 ? NP : NP * NP);
}

// psi of enriched cell en on its face f (2 D + side), projected onto the face
// basis (Pi x Pi), at face node (a, b): what a polynomial test sees of it.  For
// y faces, whose rule is n_q x n_q on both sides.
template <int NP, int NQ>
__device__ __forceinline__ double psi_face_node(const MeshDev& M, int en, int f, int a, int b) {
  const double* ps = M.psi + ((size_t)en * M.psi_pts + M.psi_off[1 + f]) * 4;
  const double* p1 = M.tab + M.proj_off + a * NQ;
  const double* p2 = M.tab + M.proj_off + b * NQ;
  double acc = 0;
#pragma unroll 1
  for (int q2 = 0; q2 < NQ; ++q2) {
    double t = 0;
#pragma unroll
    for (int q1 = 0; q1 < NQ; ++q1) t += p1[q1] * ps[(q1 + NQ * q2) * 4];
    acc += p2[q2] * t;
  }
  return acc;
}

// LDS layout of one nodal component: node (i, j, m) at i + SJ j + SK m, SC
// values; the odd row length spreads the lines that a wavefront touches over
// the banks.
template <int NP>
struct NodeLds {
  static constexpr int SJ = NP | 1, SK = SJ * NP, SC = SK * NP;
  static __device__ __forceinline__ void line(int D, int a, int b, int& base, int& stride) {
    base = D == 0 ? SJ * a + SK * b : (D == 1 ? a + SK * b : a + SJ * b);
    stride = D == 0 ? 1 : (D == 1 ? SJ : SK);
  }
};

// block -> contiguous cell ranges per XCD (workgroups are dealt round-robin
// over the 8 XCDs), so that neighbouring cells share an L2
__device__ __forceinline__ int xcd_block(int nb, int bid) {
  const int q8 = nb >> 3, r8 = nb & 7, xcd = bid & 7, m8 = bid >> 3;
  return xcd * q8 + (xcd < r8 ? xcd : r8) + m8;
}

// The value of the neighbouring lane (lane ^ 1), without LDS.
__device__ __forceinline__ float pair_swap(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ double pair_swap(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0xB1, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0xB1, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

// Apply a 1-D matrix along direction DIR (0 = x fastest) to `ncomp` stacked
// 3-D arrays held in LDS.
//   in : extents (I0, I1, I2), component stride IS
//   out: extent DIR replaced by MO, component stride OS
//   mat: row-major, out = mat * in (mat is MO x NI) or, with TR, out = mat^T in
//        (mat is NI x MO).  ADD accumulates into out.  Every output is scaled.
// One thread per pencil (line along DIR) and component; the pencil is kept in
// registers, the matrix entries are uniform across the wavefront (read from
// LDS as broadcasts when `mat` points there).
template <int DIR, int I0, int I1, int I2, int MO, bool TR, bool ADD, typename T, typename MT>
__device__ __forceinline__ void sweep(const T* __restrict__ in, int IS, T* __restrict__ out, int OS,
                                      const MT* __restrict__ mat, T scale, int ncomp) {
  constexpr int NI = DIR == 0 ? I0 : (DIR == 1 ? I1 : I2);
  constexpr int O0 = DIR == 0 ? MO : I0;
  constexpr int O1 = DIR == 1 ? MO : I1;
  constexpr int P0 = DIR == 0 ? I1 : I0;
  constexpr int P1 = DIR == 2 ? I1 : I2;
  constexpr int NPEN = P0 * P1;
  constexpr int SIN = DIR == 0 ? 1 : (DIR == 1 ? I0 : I0 * I1);
  constexpr int SOUT = DIR == 0 ? 1 : (DIR == 1 ? O0 : O0 * O1);
  for (int t = threadIdx.x; t < NPEN * ncomp; t += blockDim.x) {
    const int c = t / NPEN, p = t - c * NPEN;
    const int a = p % P0, b = p / P0;
    int ib, ob;
    if (DIR == 0) {
      ib = I0 * (a + I1 * b);
      ob = O0 * (a + O1 * b);
    } else if (DIR == 1) {
      ib = a + I0 * I1 * b;
      ob = a + O0 * O1 * b;
    } else {
      ib = a + I0 * b;
      ob = a + O0 * b;
    }
    const T* src = in + c * IS + ib;
    T* dst = out + c * OS + ob;
    T v[NI];
#pragma unroll
    for (int n = 0; n < NI; ++n) v[n] = src[n * SIN];
#pragma unroll
    for (int m = 0; m < MO; ++m) {
      T s = 0;
#pragma unroll
      for (int n = 0; n < NI; ++n) s += T(TR ? mat[n * MO + m] : mat[m * NI + n]) * v[n];
      if (ADD)
        dst[m * SOUT] += scale * s;
      else
        dst[m * SOUT] = scale * s;
    }
  }
}

// As sweep, with a compile-time matrix MAT::at(row, col) (MO x NI, or NI x MO
// with TR): every entry is a literal of the unrolled code.
// The workgroup size NT is a compile-time constant, so a line count below NT
// gives each thread at most one line and the table literals stay local to
// straight-line code.
// tofs rotates the thread-to-line assignment, so that independent sweeps of
// one phase fill the threads a previous sweep left idle.
// With MEM the coefficients are read instead from mp (the same matrix,
// row-major, in device memory): in FP64 a literal costs two scalar moves per
// use, while one wide scalar load brings eight coefficients.
template <int DIR, int I0, int I1, int I2, int MO, bool TR, bool ADD, typename MAT, int NT = 256, bool MEM = false,
          typename T>
__device__ __forceinline__ void sweep_c(const T* __restrict__ in, int IS, T* __restrict__ out, int OS, T scale,
                                        int ncomp, int tofs = 0, const double* __restrict__ mp = nullptr) {
  constexpr int NI = DIR == 0 ? I0 : (DIR == 1 ? I1 : I2);
  constexpr int O0 = DIR == 0 ? MO : I0;
  constexpr int O1 = DIR == 1 ? MO : I1;
  constexpr int P0 = DIR == 0 ? I1 : I0;
  constexpr int P1 = DIR == 2 ? I1 : I2;
  constexpr int NPEN = P0 * P1;
  constexpr int SIN = DIR == 0 ? 1 : (DIR == 1 ? I0 : I0 * I1);
  constexpr int SOUT = DIR == 0 ? 1 : (DIR == 1 ? O0 : O0 * O1);
  const int t0 = (int)threadIdx.x >= tofs ? (int)threadIdx.x - tofs : (int)threadIdx.x + NT - tofs;
  for (int t = t0; t < NPEN * ncomp; t += NT) {
    const int c = t / NPEN, p = t - c * NPEN;
    const int a = p % P0, b = p / P0;
    int ib, ob;
    if (DIR == 0) {
      ib = I0 * (a + I1 * b);
      ob = O0 * (a + O1 * b);
    } else if (DIR == 1) {
      ib = a + I0 * I1 * b;
      ob = a + O0 * O1 * b;
    } else {
      ib = a + I0 * b;
      ob = a + O0 * b;
    }
    const T* src = in + c * IS + ib;
    T* dst = out + c * OS + ob;
    T v[NI];
#pragma unroll
    for (int n = 0; n < NI; ++n) v[n] = src[n * SIN];
#pragma unroll
    for (int m = 0; m < MO; ++m) {
      T s = 0;
#pragma unroll
      for (int n = 0; n < NI; ++n)
        s += T(MEM ? mp[TR ? n * MO + m : m * NI + n] : (TR ? MAT::at(n, m) : MAT::at(m, n))) * v[n];
      if (ADD)
        dst[m * SOUT] += scale * s;
      else
        dst[m * SOUT] = scale * s;
    }
  }
}

// In-place square sweep (MO = NI): every thread reads its whole line into
// registers before writing it back, and lines are disjoint, so input and
// output may be the same array (no __restrict__ here on purpose).
template <int DIR, int I0, int I1, int I2, bool TR, typename MAT, int NT = 256, bool MEM = false, typename T>
__device__ __forceinline__ void sweep_c_inplace(T* a, int IS, T scale, int ncomp, int tofs = 0,
                                                const double* __restrict__ mp = nullptr) {
  constexpr int NI = DIR == 0 ? I0 : (DIR == 1 ? I1 : I2);
  constexpr int P0 = DIR == 0 ? I1 : I0;
  constexpr int P1 = DIR == 2 ? I1 : I2;
  constexpr int NPEN = P0 * P1;
  constexpr int SIN = DIR == 0 ? 1 : (DIR == 1 ? I0 : I0 * I1);
  const int t0 = (int)threadIdx.x >= tofs ? (int)threadIdx.x - tofs : (int)threadIdx.x + NT - tofs;
  for (int t = t0; t < NPEN * ncomp; t += NT) {
    const int c = t / NPEN, p = t - c * NPEN;
    const int aa = p % P0, b = p / P0;
    const int ib = DIR == 0 ? I0 * (aa + I1 * b) : (DIR == 1 ? aa + I0 * I1 * b : aa + I0 * b);
    T* line = a + c * IS + ib;
    T v[NI];
#pragma unroll
    for (int n = 0; n < NI; ++n) v[n] = line[n * SIN];
    T w[NI];
#pragma unroll
    for (int m = 0; m < NI; ++m) {
      T s = 0;
#pragma unroll
      for (int n = 0; n < NI; ++n)
        s += T(MEM ? mp[TR ? n * NI + m : m * NI + n] : (TR ? MAT::at(n, m) : MAT::at(m, n))) * v[n];
      w[m] = scale * s;
    }
#pragma unroll
    for (int m = 0; m < NI; ++m) line[m * SIN] = w[m];
  }
}

// Deterministic block sum of three per-thread partials (fixed order:
// butterfly within each wavefront, then waves in index order).
template <typename T>
__device__ __forceinline__ void block_sum3(T v[3], T* red /* >= 3 * nwaves */) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    T x = v[c];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
    if (lane == 0) red[3 * wave + c] = x;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    T s = 0;
    for (int w = 0; w < nw; ++w) s += red[3 * w + threadIdx.x];
    v[0] = s;  // thread c holds component c
  }
}

// Workgroup sum of N per-thread values; thread i < N receives sum i in v[0].
template <int N, typename T>
__device__ __forceinline__ void block_sum_n(T* v, T* red /* >= N * nwaves */) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int c = 0; c < N; ++c) {
    T x = v[c];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
    if (lane == 0) red[N * wave + c] = x;
  }
  __syncthreads();
  if (threadIdx.x < N) {
    T s = 0;
    for (int w = 0; w < nw; ++w) s += red[N * w + threadIdx.x];
    v[0] = s;
  }
}

}  // namespace dgwm
