// Linear operators of the velocity on cells without enrichment (arXiv
// 1705.08813, Sec. 4.2), evaluated from 1-D operators instead of quadrature.
// On a box cell every integral of a product of basis functions separates into
// 1-D integrals, and the velocity rule (n_q >= k + 1 points) integrates them
// exactly, so the quadrature sums of the definition and the 1-D forms below
// agree up to rounding.
#include <algorithm>

#include "batch.h"

namespace dgwm {

namespace {

// Cells per workgroup: one thread per line of nodes and component.
template <int NP>
struct SepShape {
  static constexpr int NP2 = NP * NP, NP3 = NP2 * NP;
  static constexpr int TPC = 3 * NP2;                        // threads of a cell
  static constexpr int CB = 256 / TPC;                       // cells of a workgroup
  // LDS layout of one component: node (i, j, m) at i + SJ j + SK m; the odd
  // row length spreads the lines that a wavefront touches over the banks
  static constexpr int SJ = NP | 1, SK = SJ * NP, SC = SK * NP;
  static constexpr int JP = 12 * NP2;                        // tangential jumps [D][2][side][NP2]
};

// Line (a, b) of nodes along direction D: first node and stride, in a vector
// of the cell (GLOBAL) or in LDS.
template <int NP>
__device__ __forceinline__ void vec_line(int D, int a, int b, int& base, int& stride) {
  constexpr int NP2 = NP * NP;
  base = D == 0 ? NP * (a + NP * b) : (D == 1 ? a + NP2 * b : a + NP * b);
  stride = D == 0 ? 1 : (D == 1 ? NP : NP2);
}
template <int NP>
__device__ __forceinline__ void lds_line(int D, int a, int b, int& base, int& stride) {
  using Sh = SepShape<NP>;
  base = D == 0 ? Sh::SJ * a + Sh::SK * b : (D == 1 ? a + Sh::SK * b : a + Sh::SJ * b);
  stride = D == 0 ? 1 : (D == 1 ? Sh::SJ : Sh::SK);
}

// Neighbour of cell e across face (D, S), or -1 for a wall.
__device__ __forceinline__ int sep_nb(const MeshDev& M, int e, int ex, int ey, int ez, int D, int S) {
  const int j = D == 0 ? ex : (D == 1 ? ey : ez);
  const int nmax = D == 0 ? M.nx : (D == 1 ? M.ny : M.nz);
  const int step = D == 0 ? 1 : (D == 1 ? M.nx : M.nx * M.ny);
  if (S ? j == nmax - 1 : j == 0) {
    if (D == 1 && !M.fully_periodic) return -1;
    return S ? e - (nmax - 1) * step : e + (nmax - 1) * step;
  }
  return S ? e + step : e - step;
}

// What a cell's line along D meets at its two ends: the neighbours' values
// and normal derivatives, the penalties, and walls.
template <typename T>
struct Ends {
  T v[2], d[2], tau[2];
  bool wall[2];
};

// Viscous interior-penalty operator (adjoint sign theta) of a cell and its six
// polynomial neighbours in nodal form,
//   V u = nu |J| (M x M x M) R,   R_c = sum_D Q_D u_c + ih_c Dn_c (sum_{d != c} W_d) + sum_s l_s Y_{c,s},
// with the mass matrix M taken out of every term so that one array per
// component collects them all:
//   Q_D u_c   the scalar interior-penalty operator along D (gradient terms
//             twice for D = c), M^{-1} applied along D;
//   W_d       = ih_d M^{-1} (int N_i' u_d - sum_faces sg N_i {u_d}), the
//             central weak derivative of u_d along its own direction; its
//             nodal derivative along c gives (grad phi_c)_d (grad u)^T_{cd} and
//             the tangential part of {{2 nu eps(u)}} n on the faces normal to d;
//   Y_{c,s}   the adjoint term of the faces normal to c, tested with the
//             tangential derivatives: -theta/2 sg sum_d ih_d E_d [u_d], on the
//             face plane and lifted by l_s = M^{-1} N(s).
// A thread owns one line of nodes of one component along each direction in
// turn (3 (k+1)^2 threads a cell).  Every value is read and written by whole
// lines, coefficients come as wide scalar loads from the mesh's tables.
// MINV leaves out |J| M M M: the result is M^{-1} V u.
// On the 64 x 32 x 32 mesh, k = 4 (57,344 such cells): 215 us with M^{-1}, where
// the quadrature kernel took 1145 us and the inverse mass another 72 us; about
// 70 FMAs per unknown, so what bounds it are the seven reads of u (own cell and
// six neighbours, mostly from L2) and the barriers between the six phases.
template <typename T, int NP, bool MINV>
__device__ __forceinline__ void viscous_cells(const MeshDev& M, int lin_off, T theta, const T* __restrict__ u,
                                              T* __restrict__ r, int first, int ncells, int layer_lo, int nlayers) {
  using Sh = SepShape<NP>;
  constexpr int NP2 = Sh::NP2, NP3 = Sh::NP3, CB = Sh::CB;
  constexpr LinOps O = lin_ops(NP);
  __shared__ T s_u[CB * 3 * Sh::SC];
  __shared__ T s_w[CB * 3 * Sh::SC];
  __shared__ T s_r[CB * 3 * Sh::SC];
  __shared__ T s_j[CB * Sh::JP];
  __shared__ T s_e[NP2];
  const T* ops = sizeof(T) == 8 ? reinterpret_cast<const T*>(M.tab + lin_off)
                                : reinterpret_cast<const T*>(M.tab + lin_off + O.f32);
  const int tid = threadIdx.x;
  const int cell = tid / Sh::TPC, t = tid - cell * Sh::TPC;
  const int c = t / NP2, k = t - c * NP2;
  const int a = k % NP, b = k / NP;
  const bool live = cell < CB && first + cell < ncells;
  T* su = s_u + cell * 3 * Sh::SC;
  T* sw = s_w + cell * 3 * Sh::SC;
  T* sr = s_r + cell * 3 * Sh::SC;
  T* sj = s_j + cell * Sh::JP;
  if (tid < NP2) s_e[tid] = ops[O.E + tid];

  int e = 0;
  T ih[3] = {0, 0, 0};
  Ends<T> en[3];
  T x[NP], qz[NP];
  // the scalar operator on a line, its jumps and (D = c) its weak derivative
  auto line = [&](int D, const T (&p)[NP], const Ends<T>& n, T (&q)[NP]) {
    const T rd = ih[D], kap = c == D ? T(2) : T(1);
    T d0 = 0, d1 = 0;
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      d0 += ops[O.nd0 + l] * p[l];
      d1 += ops[O.nd1 + l] * p[l];
    }
    d0 *= rd;
    d1 *= rd;
    // mirror states on a wall: u+ = -u-, grad u+ = grad u-
    const T J0 = p[0] - (n.wall[0] ? -p[0] : n.v[0]), J1 = p[NP - 1] - (n.wall[1] ? -p[NP - 1] : n.v[1]);
    const T s0 = d0 + (n.wall[0] ? d0 : n.d[0]), s1 = d1 + (n.wall[1] ? d1 : n.d[1]);
    const T G0 = rd * (T(0.5) * kap * s0 + n.tau[0] * J0), G1 = rd * (n.tau[1] * J1 - T(0.5) * kap * s1);
    const T r2 = kap * rd * rd, H0 = T(0.5) * theta * r2 * J0, H1 = -T(0.5) * theta * r2 * J1;
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      T acc = 0;
#pragma unroll
      for (int m = 0; m < NP; ++m) acc += ops[O.A + l * NP + m] * p[m];
      q[l] = r2 * acc + ops[O.l0 + l] * G0 + ops[O.l1 + l] * G1 + ops[O.g0 + l] * H0 + ops[O.g1 + l] * H1;
    }
    if (c == D) {
      const T a0 = T(0.5) * (p[0] + (n.wall[0] ? p[0] : n.v[0]));
      const T a1 = T(0.5) * (p[NP - 1] + (n.wall[1] ? p[NP - 1] : n.v[1]));
      int wb, ws;
      lds_line<NP>(D, a, b, wb, ws);
      T* o = sw + c * Sh::SC + wb;
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        T acc = ops[O.l0 + l] * a0 - ops[O.l1 + l] * a1;
#pragma unroll
        for (int m = 0; m < NP; ++m) acc += ops[O.E + l * NP + m] * p[m];
        o[l * ws] = rd * acc;
      }
    } else {
      T* o = sj + (D * 2 + (c < D ? c : c - 1)) * 2 * NP2 + k;
      o[0] = J0;
      o[NP2] = J1;
    }
  };
  if (live) {
    const int i = first + cell;
    const int ex = i % M.nx, t0 = i / M.nx;
    const int ey = layer_lo + t0 % nlayers, ez = t0 / nlayers;
    e = ex + M.nx * (ey + M.ny * ez);
    ih[0] = T(M.ihx);
    ih[1] = T(M.ihy[ey]);
    ih[2] = T(M.ihz);
    const T* uc = u + ((int64_t)e * 3 + c) * NP3;
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = uc[NP * k + l];
    const T pen = T(M.pen);
#pragma unroll
    for (int D = 0; D < 3; ++D) {
      int vb, vs;
      vec_line<NP>(D, a, b, vb, vs);
#pragma unroll
      for (int S = 0; S < 2; ++S) {
        const int nb = sep_nb(M, e, ex, ey, ez, D, S);
        T rn = ih[D], v = 0, d = 0;
        if (nb >= 0) {
          const T* pn = u + ((int64_t)nb * 3 + c) * NP3 + vb;
          // the neighbour below (S = 0) meets the cell at its xi_D = 1, the one above at its xi_D = 0
          const int nd = S ? O.nd0 : O.nd1;
#pragma unroll
          for (int l = 0; l < NP; ++l) {
            const T y = pn[l * vs];
            d += ops[nd + l] * y;
            if (l == (S ? 0 : NP - 1)) v = y;
          }
          if (D == 1) rn = T(M.ihy[S ? (ey + 1 == M.ny ? 0 : ey + 1) : (ey == 0 ? M.ny - 1 : ey - 1)]);
          d *= rn;
        }
        en[D].wall[S] = nb < 0;
        en[D].v[S] = v;
        en[D].d[S] = d;
        en[D].tau[S] = nb < 0 ? T(M.pen * M.wall_mult) * ih[D] : pen * (rn > ih[D] ? rn : ih[D]);
      }
    }
    T q[NP];
    line(0, x, en[0], q);
    T* o = su + c * Sh::SC + Sh::SJ * k;  // line (a, b) along x starts at SJ a + SK b = SJ k
    T* ro = sr + c * Sh::SC + Sh::SJ * k;
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      o[l] = x[l];
      ro[l] = q[l];
    }
  }
  __syncthreads();

  if (live) {
    int lb, ls;
    T q[NP];
    lds_line<NP>(1, a, b, lb, ls);
    T* p = su + c * Sh::SC + lb;
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = p[l * ls];
    line(1, x, en[1], q);
    p = sr + c * Sh::SC + lb;
#pragma unroll
    for (int l = 0; l < NP; ++l) p[l * ls] += q[l];
    lds_line<NP>(2, a, b, lb, ls);
    p = su + c * Sh::SC + lb;
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = p[l * ls];
    line(2, x, en[2], qz);
  }
  __syncthreads();

  // cross terms, on the lines of component c along direction c
  if (live) {
    const int d1 = c == 0 ? 1 : 0, d2 = c == 2 ? 1 : 2;  // the tangential directions, d1 along a, d2 along b
    int lb, ls;
    lds_line<NP>(c, a, b, lb, ls);
    const T* w1 = sw + d1 * Sh::SC + lb;
    const T* w2 = sw + d2 * Sh::SC + lb;
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = w1[l * ls] + w2[l * ls];
    const T ihc = c == 0 ? ih[0] : (c == 1 ? ih[1] : ih[2]);
    const T ih1 = c == 0 ? ih[1] : ih[0], ih2 = c == 2 ? ih[1] : ih[2];
    T y[2];
    const T* j1 = sj + (c * 2) * 2 * NP2;      // jumps of component d1, then of d2, [side][NP2]
    const T* j2 = j1 + 2 * NP2;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      T s1 = 0, s2 = 0;
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        s1 += s_e[a * NP + j] * j1[s * NP2 + j + NP * b];
        s2 += s_e[b * NP + j] * j2[s * NP2 + a + NP * j];
      }
      y[s] = (s ? -T(0.5) : T(0.5)) * theta * ihc * (ih1 * s1 + ih2 * s2);
    }
    T* p = sr + c * Sh::SC + lb;
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      T acc = 0;
#pragma unroll
      for (int m = 0; m < NP; ++m) acc += ops[O.Dn + l * NP + m] * x[m];
      p[l * ls] += ihc * acc + ops[O.l0 + l] * y[0] + ops[O.l1 + l] * y[1];
    }
  }
  __syncthreads();

  const T nu = T(M.nu);
  if (live) {  // along z: add the z part; mass matrix
    int lb, ls;
    lds_line<NP>(2, a, b, lb, ls);
    T* p = sr + c * Sh::SC + lb;
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = p[l * ls] + qz[l];
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      T acc = 0;
      if (MINV) acc = x[l];
      else {
#pragma unroll
        for (int m = 0; m < NP; ++m) acc += ops[O.M + l * NP + m] * x[m];
      }
      p[l * ls] = acc;
    }
  }
  __syncthreads();
  if (!MINV) {
    if (live) {
      int lb, ls;
      lds_line<NP>(1, a, b, lb, ls);
      T* p = sr + c * Sh::SC + lb;
#pragma unroll
      for (int l = 0; l < NP; ++l) x[l] = p[l * ls];
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        T acc = 0;
#pragma unroll
        for (int m = 0; m < NP; ++m) acc += ops[O.M + l * NP + m] * x[m];
        p[l * ls] = acc;
      }
    }
    __syncthreads();
  }
  if (live) {
    const T* p = sr + c * Sh::SC + Sh::SJ * k;
    T* o = r + ((int64_t)e * 3 + c) * NP3 + NP * k;
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = p[l];
    const T sc = MINV ? nu : nu / (ih[0] * ih[1] * ih[2]);
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      T acc = 0;
      if (MINV) acc = x[l];
      else {
#pragma unroll
        for (int m = 0; m < NP; ++m) acc += ops[O.M + l * NP + m] * x[m];
      }
      o[l] = sc * acc;
    }
  }
}

// block -> contiguous cell ranges per XCD (workgroups are dealt round-robin
// over the 8 XCDs), so that neighbouring cells share an L2
__device__ __forceinline__ int xcd_block(int nb, int bid) {
  const int q8 = nb >> 3, r8 = nb & 7, xcd = bid & 7, m8 = bid >> 3;
  return xcd * q8 + (xcd < r8 ? xcd : r8) + m8;
}

template <int NP, bool MINV>
__global__ __launch_bounds__(256) void viscous_regular_kernel(const MeshDev M, int lin_off,
                                                              const double* __restrict__ u, double* __restrict__ r,
                                                              int ncells, int layer_lo, int nlayers) {
  viscous_cells<double, NP, MINV>(M, lin_off, -1.0, u, r, xcd_block(gridDim.x, blockIdx.x) * SepShape<NP>::CB, ncells,
                                  layer_lo, nlayers);
}

}  // namespace

RegularLayers regular_layers(const dg_mesh* m) {
  RegularLayers L{};
  const bool el = !m->P.fully_periodic && m->lower_slot >= 0, eu = !m->P.fully_periodic && m->upper_slot >= 0;
  const int ny = m->P.ny;
  L.lo = el ? 1 : 0;
  const int hi = eu ? ny - 2 : ny - 1;
  L.nl = std::max(0, hi - L.lo + 1);
  if (L.nl == 0) return L;
  L.ilo = L.lo + (el ? 1 : 0);
  L.inl = std::max(0, hi - (eu ? 1 : 0) - L.ilo + 1);
  // the layers next to an enriched one
  if (el) {
    L.xlo = L.lo;
    L.xnl = 1;
    L.xstep = 1;
    if (eu && hi > L.lo) {
      L.xnl = 2;
      L.xstep = hi - L.lo;
    }
  } else if (eu) {
    L.xlo = hi;
    L.xnl = 1;
    L.xstep = 1;
  }
  return L;
}

int launch_viscous_regular(const dg_mesh* m, const double* u, double* out, int lo, int nl, bool inverse_mass,
                           hipStream_t s) {
  if (nl <= 0) return DG_OK;
  const MeshDev M = velocity_meshdev(m);
  const int off = lin_offset(m->np_u, m->P.nq_u, m->P.nq_wn);
  const int64_t nc = (int64_t)m->P.nx * nl * m->P.nz;
#define X(p)                                                                                                       \
  if (m->np_u == p) {                                                                                              \
    const unsigned nb = (unsigned)((nc + SepShape<p>::CB - 1) / SepShape<p>::CB);                                  \
    if (inverse_mass)                                                                                              \
      hipLaunchKernelGGL((viscous_regular_kernel<p, true>), dim3(nb), dim3(256), 0, s, M, off, u, out, (int)nc, lo, \
                         nl);                                                                                      \
    else                                                                                                           \
      hipLaunchKernelGGL((viscous_regular_kernel<p, false>), dim3(nb), dim3(256), 0, s, M, off, u, out, (int)nc,   \
                         lo, nl);                                                                                  \
    return check_hip(hipGetLastError(), "viscous kernel launch");                                                  \
  }
  X(3) X(4) X(5) X(6)
#undef X
  return set_error(DG_ERR_UNSUPPORTED, "viscous operator: degree not compiled");
}

}  // namespace dgwm
