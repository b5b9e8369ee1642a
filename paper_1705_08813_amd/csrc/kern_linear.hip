// Linear operators of the velocity on cells without enrichment (arXiv
// 1705.08813, Sec. 4.2), evaluated from 1-D operators instead of quadrature.
// On a box cell every integral of a product of basis functions separates into
// 1-D integrals, and the velocity rule (n_q >= k + 1 points) integrates them
// exactly, so the quadrature sums of the definition and the 1-D forms below
// agree up to rounding.
#include <algorithm>

#include "batch.h"
#include "ip_line.h"

namespace dgwm {

namespace {

// Cells per workgroup: one thread per line of nodes and component.
template <int NP>
struct SepShape {
  static constexpr int NP2 = NP * NP, NP3 = NP2 * NP;
  static constexpr int TPC = 3 * NP2;                        // threads of a cell
  static constexpr int CB = 256 / TPC;                       // cells of a workgroup
  static constexpr int SJ = NodeLds<NP>::SJ, SK = NodeLds<NP>::SK, SC = NodeLds<NP>::SC;
  static constexpr int JP = 12 * NP2;                        // tangential jumps [D][2][side][NP2]
};

// Viscous interior-penalty operator (adjoint sign -1) of a cell and its six
// neighbours in the nodal form of ip_line.h (an enriched neighbour's psi u~
// enters the jumps only, as on the interface faces of eq. viscous_multiscale,
// projected onto the face basis).
// A thread owns one line of nodes of one component along each direction in
// turn (3 (k+1)^2 threads a cell).  Every value is read and written by whole
// lines, coefficients come as wide scalar loads from the mesh's tables.
// MINV leaves out |J| M M M: the result is M^{-1} V u.
// On the 64 x 32 x 32 mesh, k = 4 (61,440 such cells, next to the walls' layers
// too): 239 us with M^{-1}, where the quadrature kernel took 1,145 us and the
// inverse mass another 72 us; about 70 FMAs per unknown, so what bounds it are
// the seven reads of u (own cell and six neighbours, mostly from L2) and the
// barriers between the six phases.
// (A function of its own under the kernel: there the compiler knows that u and
// r are apart also for the scalar loads; 0.6 us a launch.)
template <int NP, int NQ, bool MINV>
__device__ __forceinline__ void viscous_cells(const MeshDev& M, int lin_off, const double* __restrict__ u,
                                              double* __restrict__ r, int first, int ncells, int layer_lo,
                                              int nlayers) {
  using Sh = SepShape<NP>;
  constexpr int NP2 = Sh::NP2, NP3 = Sh::NP3, CB = Sh::CB;
  constexpr LinOps O = lin_ops(NP);
  __shared__ double s_u[CB * 3 * Sh::SC];
  __shared__ double s_w[CB * 3 * Sh::SC];
  __shared__ double s_r[CB * 3 * Sh::SC];
  __shared__ double s_j[CB * Sh::JP];
  __shared__ double s_e[NP2];
  const double* const ops_at = M.tab + lin_off;
  ConstTab<double> ops = const_tab<double>(ops_at);
  auto phase = [&]() __attribute__((always_inline)) {  // (see const_tab)
    __syncthreads();
    ops = const_tab<double>(ops_at);
  };
  constexpr double theta = -1.0;
  const int tid = threadIdx.x;
  const int cell = tid / Sh::TPC, t = tid - cell * Sh::TPC;
  const int c = t / NP2, k = t - c * NP2;
  const int a = k % NP, b = k / NP;
  const bool live = cell < CB && first + cell < ncells;
  double* su = s_u + cell * 3 * Sh::SC;
  double* sw = s_w + cell * 3 * Sh::SC;
  double* sr = s_r + cell * 3 * Sh::SC;
  double* sj = s_j + cell * Sh::JP;
  if (tid < NP2) s_e[tid] = ops[O.E + tid];

  int e = 0;
  double ih[3] = {0, 0, 0};
  IpEnds<double> en[3];
  double vn[3][2];  // the neighbours' values without psi u~
  double x[NP], qz[NP];
  // the scalar operator on a line, its jumps and (D = c) its weak derivative
  auto line = [&](int D, const double (&p)[NP], const IpEnds<double>& n, const double (&vn)[2],
                  double (&q)[NP]) __attribute__((always_inline)) {
    double J[2];
    ip_line(ops, c == D, ih[D], theta, n, p, q, J, [](double (&)[2]) {});
    if (c == D) {
      int wb, ws;
      NodeLds<NP>::line(D, a, b, wb, ws);
      ip_weak(ops, ih[D], n.wall[0], n.wall[1], vn[0], vn[1], p, sw + c * Sh::SC + wb, ws);
    } else {
      double* o = sj + (D * 2 + (c < D ? c : c - 1)) * 2 * NP2 + k;
      o[0] = J[0];
      o[NP2] = J[1];
    }
  };
  if (live) {
    const int i = first + cell;
    const int ex = i % M.nx, t0 = i / M.nx;
    const int ey = layer_lo + t0 % nlayers, ez = t0 / nlayers;
    e = ex + M.nx * (ey + M.ny * ez);
    ih[0] = M.ihx;
    ih[1] = M.ihy[ey];
    ih[2] = M.ihz;
    const double* uc = u + ((int64_t)e * 3 + c) * NP3;
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = uc[NP * k + l];
    const double pen = M.pen;
#pragma unroll
    for (int D = 0; D < 3; ++D) {
      int vb, vs;
      vec_line<NP>(D, a, b, vb, vs);
#pragma unroll
      for (int S = 0; S < 2; ++S) {
        const int nb = cell_nb(M, e, ex, ey, ez, D, S);
        double rn = ih[D], v = 0, d = 0;
        if (nb >= 0) {
          const double* pn = u + ((int64_t)nb * 3 + c) * NP3 + vb;
          // the neighbour below (S = 0) meets the cell at its xi_D = 1, the one above at its xi_D = 0
          const int nd = S ? O.nd0 : O.nd1;
#pragma unroll
          for (int l = 0; l < NP; ++l) {
            const double y = pn[l * vs];
            d += ops[nd + l] * y;
            if (l == (S ? 0 : NP - 1)) v = y;
          }
          if (D == 1) rn = M.ihy[S ? (ey + 1 == M.ny ? 0 : ey + 1) : (ey == 0 ? M.ny - 1 : ey - 1)];
          d *= rn;
        }
        double ps = 0;
        if (D == 1 && nb >= 0) {
          const int k1 = (int)enr_index(M, ex, S ? (ey + 1 == M.ny ? 0 : ey + 1) : (ey == 0 ? M.ny - 1 : ey - 1), ez);
          if (k1 >= 0)
            ps = psi_face_node<NP, NQ>(M, k1, 2 + (1 - S), a, b) * u[M.enr_off + (int64_t)k1 * 3 + c];
        }
        en[D].wall[S] = nb < 0;
        en[D].v[S] = D == 1 ? v + ps : v;
        vn[D][S] = v;
        en[D].d[S] = d;
        en[D].tau[S] = nb < 0 ? M.pen * M.wall_mult * ih[D] : pen * (rn > ih[D] ? rn : ih[D]);
      }
    }
    double q[NP];
    line(0, x, en[0], vn[0], q);
    double* o = su + c * Sh::SC + Sh::SJ * k;  // line (a, b) along x starts at SJ a + SK b = SJ k
    double* ro = sr + c * Sh::SC + Sh::SJ * k;
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      o[l] = x[l];
      ro[l] = q[l];
    }
  }
  phase();

  if (live) {
    int lb, ls;
    double q[NP];
    NodeLds<NP>::line(1, a, b, lb, ls);
    double* p = su + c * Sh::SC + lb;
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = p[l * ls];
    line(1, x, en[1], vn[1], q);
    p = sr + c * Sh::SC + lb;
#pragma unroll
    for (int l = 0; l < NP; ++l) p[l * ls] += q[l];
    NodeLds<NP>::line(2, a, b, lb, ls);
    p = su + c * Sh::SC + lb;
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = p[l * ls];
    line(2, x, en[2], vn[2], qz);
  }
  phase();

  // cross terms, on the lines of component c along direction c
  if (live) {
    const int d1 = c == 0 ? 1 : 0, d2 = c == 2 ? 1 : 2;  // the tangential directions, d1 along a, d2 along b
    int lb, ls;
    NodeLds<NP>::line(c, a, b, lb, ls);
    const double* w1 = sw + d1 * Sh::SC + lb;
    const double* w2 = sw + d2 * Sh::SC + lb;
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = w1[l * ls] + w2[l * ls];
    const double ihc = c == 0 ? ih[0] : (c == 1 ? ih[1] : ih[2]);
    const double ih1 = c == 0 ? ih[1] : ih[0], ih2 = c == 2 ? ih[1] : ih[2];
    const double* j1 = sj + (c * 2) * 2 * NP2;      // jumps of component d1, then of d2, [side][NP2]
    ip_cross(ops, s_e, theta, ihc, ih1, ih2, a, b, j1, j1 + 2 * NP2, x, sr + c * Sh::SC + lb, ls);
  }
  phase();

  if (live) {  // along z: add the z part; mass matrix
    int lb, ls;
    NodeLds<NP>::line(2, a, b, lb, ls);
    double* p = sr + c * Sh::SC + lb;
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = p[l * ls] + qz[l];
    if (MINV) {
#pragma unroll
      for (int l = 0; l < NP; ++l) p[l * ls] = x[l];
    } else {
      ip_mass(ops, x, p, ls);
    }
  }
  phase();
  if (!MINV) {
    if (live) {
      int lb, ls;
      NodeLds<NP>::line(1, a, b, lb, ls);
      double* p = sr + c * Sh::SC + lb;
#pragma unroll
      for (int l = 0; l < NP; ++l) x[l] = p[l * ls];
      ip_mass(ops, x, p, ls);
    }
    phase();
  }
  if (live) {
    const double* p = sr + c * Sh::SC + Sh::SJ * k;
    double* o = r + ((int64_t)e * 3 + c) * NP3 + NP * k;
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = p[l];
    const double sc = MINV ? M.nu : M.nu / (ih[0] * ih[1] * ih[2]);
    if (MINV) {
#pragma unroll
      for (int l = 0; l < NP; ++l) o[l] = sc * x[l];
    } else {
      ip_mass(ops, x, o, 1, sc);
    }
  }
}

template <int NP, int NQ, bool MINV>
__global__ __launch_bounds__(256) void viscous_regular_kernel(const MeshDev M, int lin_off,
                                                              const double* __restrict__ u, double* __restrict__ r,
                                                              int ncells, int layer_lo, int nlayers) {
  viscous_cells<NP, NQ, MINV>(M, lin_off, u, r, xcd_block(gridDim.x, blockIdx.x) * SepShape<NP>::CB, ncells, layer_lo,
                              nlayers);
}

// Vorticity right-hand side b(v) = (v, curl u)_e in nodal form: curl u is a
// polynomial of the cell's space, so b = |J| (M x M x M) curl u with the nodal
// derivatives Dn u / h; MINV stops at M^{-1} b = curl u itself.
// Thread (row r, line) takes d_{d1} u_{d2} of its row along d1, then
// d_{d2} u_{d1} along d2 (d1 < d2 the other two directions) together with
// the first mass sweep.  Bound by the read of u and the write of b: 83 us for
// the 61,440 such cells of the 64 x 32 x 32 mesh, k = 4 (4.4 TB/s; 2713 us with
// direct sums over the basis at the Gauss points).
template <int NP, bool MINV>
__global__ __launch_bounds__(256) void vorticity_regular_kernel(const MeshDev M, int lin_off,
                                                                const double* __restrict__ u, double* __restrict__ out,
                                                                int ncells, int layer_lo, int nlayers) {
  using Sh = SepShape<NP>;
  constexpr int NP2 = Sh::NP2, NP3 = Sh::NP3, CB = Sh::CB;
  constexpr LinOps O = lin_ops(NP);
  __shared__ double s_u[CB * 3 * Sh::SC];
  __shared__ double s_r[CB * 3 * Sh::SC];
  const double* ops = M.tab + lin_off;
  const int tid = threadIdx.x, first = xcd_block(gridDim.x, blockIdx.x) * CB;
  const int cell = tid / Sh::TPC, t = tid - cell * Sh::TPC;
  const int r = t / NP2, k = t - r * NP2;
  const int a = k % NP, b = k / NP;
  const bool live = cell < CB && first + cell < ncells;
  double* su = s_u + cell * 3 * Sh::SC;
  double* sr = s_r + cell * 3 * Sh::SC + r * Sh::SC;
  const int d1 = r == 0 ? 1 : 0, d2 = r == 2 ? 1 : 2;
  // curl_r = sg (d_{d1} u_{d2} - d_{d2} u_{d1}), sg = -1 for r = y
  const double sg = r == 1 ? -1.0 : 1.0;
  double x[NP], ih[3] = {0, 0, 0};
  int64_t e = 0;
  auto load = [&](const double* p, int st) {
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = p[l * st];
  };
  auto dot = [&](int tab, int l) {
    double acc = 0;
#pragma unroll
    for (int m = 0; m < NP; ++m) acc += ops[tab + l * NP + m] * x[m];
    return acc;
  };
  if (live) {
    const int i = first + cell;
    const int ex = i % M.nx, t0 = i / M.nx;
    const int ey = layer_lo + t0 % nlayers, ez = t0 / nlayers;
    e = ex + M.nx * (ey + (int64_t)M.ny * ez);
    ih[0] = M.ihx;
    ih[1] = M.ihy[ey];
    ih[2] = M.ihz;
    load(u + (e * 3 + r) * NP3 + NP * k, 1);
#pragma unroll
    for (int l = 0; l < NP; ++l) su[r * Sh::SC + Sh::SJ * k + l] = x[l];
  }
  __syncthreads();
  const double f1 = sg * (d1 == 0 ? ih[0] : ih[1]), f2 = -sg * (d2 == 1 ? ih[1] : ih[2]);
  int lb1, ls1, lb2, ls2;
  NodeLds<NP>::line(d1, a, b, lb1, ls1);
  NodeLds<NP>::line(d2, a, b, lb2, ls2);
  if (live) {
    load(su + d2 * Sh::SC + lb1, ls1);
#pragma unroll
    for (int l = 0; l < NP; ++l) sr[lb1 + l * ls1] = f1 * dot(O.Dn, l);
  }
  __syncthreads();
  if (live) {
    load(su + d1 * Sh::SC + lb2, ls2);
    double v[NP];
#pragma unroll
    for (int l = 0; l < NP; ++l) v[l] = sr[lb2 + l * ls2] + f2 * dot(O.Dn, l);
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = v[l];
#pragma unroll
    for (int l = 0; l < NP; ++l) sr[lb2 + l * ls2] = MINV ? x[l] : dot(O.M, l);
  }
  __syncthreads();
  if (!MINV) {
    // the other tangential direction: y for rows x and y, z for row z
    int lb, ls;
    NodeLds<NP>::line(r == 2 ? 2 : 1, a, b, lb, ls);
    if (live) {
      load(sr + lb, ls);
#pragma unroll
      for (int l = 0; l < NP; ++l) sr[lb + l * ls] = dot(O.M, l);
    }
    __syncthreads();
  }
  if (live) {
    load(sr + Sh::SJ * k, 1);
    const double vol = 1.0 / (ih[0] * ih[1] * ih[2]);
    double* o = out + (e * 3 + r) * NP3 + NP * k;
#pragma unroll
    for (int l = 0; l < NP; ++l) o[l] = MINV ? x[l] : vol * dot(O.M, l);
  }
}

// Cells of a workgroup of the gradient and divergence kernels.
template <int NU, int NPP>
struct MixShape {
  static constexpr int CB = NU <= 3 ? 8 : (NU <= 5 ? 4 : 2);
};

// Pressure gradient term on cells without enrichment, one component at a time
// separable:  g_c = h_a h_b (G_c x M_a x M_b) p  with the 1-D operators of
// mix_ops; the neighbours' halves of the central averages enter as one more
// value at each end of the lines along c (walls: the cell's own end value).
// The cell's pressure with its six neighbour layers is swept along z (lines
// through the x and y neighbours' layers included), y and x.  Loops run over
// the lines of all cells of the workgroup.  96 us for the 61,440 such cells of
// the 64 x 32 x 32 mesh, k_u = 4, k_p = 3 (373 us by quadrature, 27 barrier
// phases a cell): the write of g and five short phases bound it.
template <int NU, int NPP>
__global__ __launch_bounds__(256) void gradient_regular_kernel(const MeshDev M, int mix_off,
                                                               const double* __restrict__ p, double* __restrict__ out,
                                                               int ncells, int layer_lo, int nlayers) {
  constexpr int CB = MixShape<NU, NPP>::CB, NP2 = NPP * NPP, NP3 = NP2 * NPP, NU2 = NU * NU, NU3 = NU2 * NU;
  constexpr MixOps O = mix_ops(NU, NPP);
  constexpr int LZ = NP2 + 4 * NPP;  // z lines with mass: (a, b), then x- and y-neighbour layers [S][tangential]
  // P: pressure [node], then neighbour layers [D][S][NP2]; A: after z, mass [line][NU]; Gz: after z, gradient
  constexpr int NPV = NP3 + 6 * NP2, NA = LZ * NU, NG = NP2 * NU;
  // after y: x component on x in [-1, NPP] ext, y and z components
  constexpr int NB = (NPP + 2) * NU2, NC = NPP * NU2;
  constexpr int S1 = (NPV > NB + 2 * NC ? NPV : NB + 2 * NC), S2 = NA + NG;
  __shared__ double s1[CB * S1];
  __shared__ double s2[CB * S2];
  __shared__ int s_e[CB * 7];  // cell, then its neighbours (walls: the cell itself, flagged below)
  const double* ops = M.tab + mix_off;
  const int tid = threadIdx.x, first = xcd_block(gridDim.x, blockIdx.x) * CB;
  const int nc = ncells - first < CB ? ncells - first : CB;
  if (tid < nc * 7) {
    const int cell = tid / 7, f = tid - cell * 7 - 1;
    const int i = first + cell;
    const int ex = i % M.nx, t0 = i / M.nx;
    const int ey = layer_lo + t0 % nlayers, ez = t0 / nlayers;
    const int e = ex + M.nx * (ey + M.ny * ez);
    s_e[tid] = f < 0 ? e : cell_nb(M, e, ex, ey, ez, f >> 1, f & 1);
  }
  __syncthreads();
  for (int it = tid; it < nc * NPV; it += 256) {
    const int cell = it / NPV, i = it - cell * NPV;
    double v;
    if (i < NP3) v = p[(int64_t)s_e[cell * 7] * NP3 + i];
    else {
      const int f = (i - NP3) / NP2, l = (i - NP3) - f * NP2, D = f >> 1, S = f & 1;
      const int nb = s_e[cell * 7 + 1 + f];
      // the neighbour's layer at the shared face; the cell's own on a wall
      const int ld = (nb < 0) == (S == 1) ? NPP - 1 : 0;
      const int l1 = l % NPP, l2 = l / NPP;
      const int nd = D == 0 ? ld + NPP * l : (D == 1 ? l1 + NPP * (ld + NPP * l2) : l + NP2 * ld);
      v = p[(int64_t)(nb < 0 ? s_e[cell * 7] : nb) * NP3 + nd];
    }
    s1[cell * S1 + i] = v;
  }
  __syncthreads();
  // z: mass on the lines of the cell and of the x and y neighbour layers, gradient on the cell's
  for (int it = tid; it < nc * (LZ + NP2); it += 256) {
    const int cell = it / (LZ + NP2), i = it - cell * (LZ + NP2);
    const double* P = s1 + cell * S1;
    int base, st;
    const bool grad = i >= LZ;
    if (i < NP2 || grad) {
      base = grad ? i - LZ : i;
      st = NP2;
    } else {  // layer of face (D, S), D = x: [y + NPP z], D = y: [x + NPP z]: tangential index l1, line along z
      const int j = i - NP2, f = j / NPP;
      base = NP3 + f * NP2 + (j - f * NPP);
      st = NPP;
    }
    double x[NPP];
#pragma unroll
    for (int l = 0; l < NPP; ++l) x[l] = P[base + l * st];
    double* o = s2 + cell * S2 + (grad ? NA + (i - LZ) * NU : i * NU);
    if (grad) {
      const double e0 = P[NP3 + 4 * NP2 + (i - LZ)], e1 = P[NP3 + 5 * NP2 + (i - LZ)];
#pragma unroll
      for (int q = 0; q < NU; ++q) {
        double acc = q == 0 ? -0.5 * e0 : (q == NU - 1 ? 0.5 * e1 : 0.0);
#pragma unroll
        for (int l = 0; l < NPP; ++l) acc += ops[O.Gu + q * NPP + l] * x[l];
        o[q] = acc;
      }
    } else {
#pragma unroll
      for (int q = 0; q < NU; ++q) {
        double acc = 0;
#pragma unroll
        for (int l = 0; l < NPP; ++l) acc += ops[O.Mup + q * NPP + l] * x[l];
        o[q] = acc;
      }
    }
  }
  __syncthreads();
  // y: mass for the x component (x neighbours' lines included) and the z component, gradient for the y one
  constexpr int LY = (3 * NPP + 2) * NU;
  for (int it = tid; it < nc * LY; it += 256) {
    const int cell = it / LY, i = it - cell * LY;
    const int line = i / NU, q = i - line * NU;  // q: z index
    const double* A = s2 + cell * S2;
    double* B = s1 + cell * S1;
    double x[NPP];
    if (line < NPP + 2) {
      // x component: x = line, or the layers of the x neighbours (line NPP: S = 0, NPP + 1: S = 1)
#pragma unroll
      for (int l = 0; l < NPP; ++l)
        x[l] = A[(line < NPP ? line + NPP * l : NP2 + (line - NPP) * NPP + l) * NU + q];
#pragma unroll
      for (int j = 0; j < NU; ++j) {
        double acc = 0;
#pragma unroll
        for (int l = 0; l < NPP; ++l) acc += ops[O.Mup + j * NPP + l] * x[l];
        B[line + (NPP + 2) * (j + NU * q)] = acc;
      }
    } else if (line < 2 * NPP + 2) {
      const int xx = line - NPP - 2;
#pragma unroll
      for (int l = 0; l < NPP; ++l) x[l] = A[(xx + NPP * l) * NU + q];
      const double e0 = A[(NP2 + 2 * NPP + xx) * NU + q], e1 = A[(NP2 + 3 * NPP + xx) * NU + q];
#pragma unroll
      for (int j = 0; j < NU; ++j) {
        double acc = j == 0 ? -0.5 * e0 : (j == NU - 1 ? 0.5 * e1 : 0.0);
#pragma unroll
        for (int l = 0; l < NPP; ++l) acc += ops[O.Gu + j * NPP + l] * x[l];
        B[NB + xx + NPP * (j + NU * q)] = acc;
      }
    } else {
      const int xx = line - 2 * NPP - 2;
#pragma unroll
      for (int l = 0; l < NPP; ++l) x[l] = A[NA + (xx + NPP * l) * NU + q];
#pragma unroll
      for (int j = 0; j < NU; ++j) {
        double acc = 0;
#pragma unroll
        for (int l = 0; l < NPP; ++l) acc += ops[O.Mup + j * NPP + l] * x[l];
        B[NB + NC + xx + NPP * (j + NU * q)] = acc;
      }
    }
  }
  __syncthreads();
  // x, and write
  for (int it = tid; it < nc * 3 * NU2; it += 256) {
    const int cell = it / (3 * NU2), i = it - cell * 3 * NU2;
    const int c = i / NU2, k = i - c * NU2;
    const int e = s_e[cell * 7];
    const double hy = M.hy[(e / M.nx) % M.ny];
    const double sc = c == 0 ? hy * M.hz : (c == 1 ? M.hx * M.hz : M.hx * hy);
    const double* B = s1 + cell * S1 + (c == 0 ? (NPP + 2) * k : NB + (c - 1) * NC + NPP * k);
    double x[NPP];
#pragma unroll
    for (int l = 0; l < NPP; ++l) x[l] = B[l];
    const double e0 = c == 0 ? B[NPP] : 0.0, e1 = c == 0 ? B[NPP + 1] : 0.0;
    double* o = out + ((int64_t)e * 3 + c) * NU3 + NU * k;
    const double* tb = ops + (c == 0 ? O.Gu : O.Mup);
#pragma unroll
    for (int q = 0; q < NU; ++q) {
      double acc = q == 0 ? -0.5 * e0 : (q == NU - 1 ? 0.5 * e1 : 0.0);
#pragma unroll
      for (int l = 0; l < NPP; ++l) acc += tb[q * NPP + l] * x[l];
      o[q] = sc * acc;
    }
  }
}

// Velocity divergence term on cells without enrichment whose neighbours have
// none either: the transposed sweeps, c = sum_c h_a h_b (Gp_c x M_a^T x M_b^T) u_c,
// along x, y, z; component c brings the layers of its neighbours along c.
// 116 us for 57,344 cells of the 64 x 32 x 32 mesh (by quadrature 547 us for
// 61,440): the read of u and its neighbour layers bounds it.
template <int NU, int NPP>
__global__ __launch_bounds__(256) void divergence_regular_kernel(const MeshDev M, int mix_off,
                                                                 const double* __restrict__ u,
                                                                 double* __restrict__ out, int ncells, int layer_lo,
                                                                 int nlayers) {
  constexpr int CB = MixShape<NU, NPP>::CB, NP2 = NPP * NPP, NP3 = NP2 * NPP, NU2 = NU * NU, NU3 = NU2 * NU;
  constexpr MixOps O = mix_ops(NU, NPP);
  constexpr int NV = 3 * NU3 + 6 * NU2;  // u, then the neighbours' layers of their normal component [D][S][NU2]
  // after x: u_x [NPP][NU y][NU z]; u_y with its layers [S] behind: lines (y, z), then [S][z]; u_z: (y, z), then [S][y]
  constexpr int LX = 3 * NU2 + 4 * NU, NX = LX * NPP;
  // after y: x and y parts together [NPP x][NPP y][NU z]; z part [NPP][NPP][NU], then [S][NPP][NPP]
  constexpr int NY1 = NP2 * NU, NY2 = NP2 * (NU + 2);
  constexpr int S1 = NV > NY1 + NY2 ? NV : NY1 + NY2;
  __shared__ double s1[CB * S1];
  __shared__ double s2[CB * NX];
  __shared__ int s_e[CB * 7];
  const double* ops = M.tab + mix_off;
  const int tid = threadIdx.x, first = xcd_block(gridDim.x, blockIdx.x) * CB;
  const int nc = ncells - first < CB ? ncells - first : CB;
  if (tid < nc * 7) {
    const int cell = tid / 7, f = tid - cell * 7 - 1;
    const int i = first + cell;
    const int ex = i % M.nx, t0 = i / M.nx;
    const int ey = layer_lo + t0 % nlayers, ez = t0 / nlayers;
    const int e = ex + M.nx * (ey + M.ny * ez);
    s_e[tid] = f < 0 ? e : cell_nb(M, e, ex, ey, ez, f >> 1, f & 1);
  }
  __syncthreads();
  for (int it = tid; it < nc * NV; it += 256) {
    const int cell = it / NV, i = it - cell * NV;
    double v;
    if (i < 3 * NU3) v = u[(int64_t)s_e[cell * 7] * 3 * NU3 + i];
    else {
      const int f = (i - 3 * NU3) / NU2, l = (i - 3 * NU3) - f * NU2, D = f >> 1, S = f & 1;
      const int nb = s_e[cell * 7 + 1 + f];
      const int ld = (nb < 0) == (S == 1) ? NU - 1 : 0;
      const int l1 = l % NU, l2 = l / NU;
      const int nd = D == 0 ? ld + NU * l : (D == 1 ? l1 + NU * (ld + NU * l2) : l + NU2 * ld);
      v = u[((int64_t)(nb < 0 ? s_e[cell * 7] : nb) * 3 + D) * NU3 + nd];
    }
    s1[cell * S1 + i] = v;
  }
  __syncthreads();
  // x lines: gradient table for u_x, mass for u_y and u_z and the layers of the y and z neighbours
  for (int it = tid; it < nc * LX; it += 256) {
    const int cell = it / LX, i = it - cell * LX;
    const double* V = s1 + cell * S1;
    // lines [u_x: NU2 | u_y: NU2, then [S][z] | u_z: NU2, then [S][y]]
    int base;
    if (i < NU2) base = NU * i;
    else if (i < 2 * NU2) base = NU3 + NU * (i - NU2);
    else if (i < 2 * NU2 + 2 * NU) base = 3 * NU3 + 2 * NU2 + NU * (i - 2 * NU2);
    else if (i < 3 * NU2 + 2 * NU) base = 2 * NU3 + NU * (i - 2 * NU2 - 2 * NU);
    else base = 3 * NU3 + 4 * NU2 + NU * (i - 3 * NU2 - 2 * NU);
    double x[NU];
#pragma unroll
    for (int l = 0; l < NU; ++l) x[l] = V[base + l];
    double* o = s2 + cell * NX + i * NPP;
    if (i < NU2) {
      const double e0 = V[3 * NU3 + i], e1 = V[3 * NU3 + NU2 + i];
#pragma unroll
      for (int q = 0; q < NPP; ++q) {
        double acc = q == 0 ? -0.5 * e0 : (q == NPP - 1 ? 0.5 * e1 : 0.0);
#pragma unroll
        for (int l = 0; l < NU; ++l) acc += ops[O.Gp + q * NU + l] * x[l];
        o[q] = acc;
      }
    } else {
#pragma unroll
      for (int q = 0; q < NPP; ++q) {
        double acc = 0;
#pragma unroll
        for (int l = 0; l < NU; ++l) acc += ops[O.Mup + l * NPP + q] * x[l];
        o[q] = acc;
      }
    }
  }
  __syncthreads();
  // y lines
  constexpr int LY = NPP * NU + NPP * (NU + 2);
  for (int it = tid; it < nc * LY; it += 256) {
    const int cell = it / LY, i = it - cell * LY;
    const double* X = s2 + cell * NX;
    double* Y = s1 + cell * S1;
    const int e = s_e[cell * 7];
    const double hy = M.hy[(e / M.nx) % M.ny];
    const int line = i / NPP, q = i - line * NPP;  // q: x index
    double x[NU];
    if (line < NU) {  // z = line: u_x with mass, u_y with the gradient table, their areas
      const double* p = X + NU * line * NPP + q;
      const double* py = X + (NU2 + NU * line) * NPP + q;
      const double* pe = X + (2 * NU2 + line) * NPP + q;
      double y[NU];
#pragma unroll
      for (int l = 0; l < NU; ++l) {
        x[l] = hy * M.hz * p[l * NPP];
        y[l] = M.hx * M.hz * py[l * NPP];
      }
      const double e0 = M.hx * M.hz * pe[0], e1 = M.hx * M.hz * pe[NU * NPP];
#pragma unroll
      for (int j = 0; j < NPP; ++j) {
        double acc = j == 0 ? -0.5 * e0 : (j == NPP - 1 ? 0.5 * e1 : 0.0);
#pragma unroll
        for (int l = 0; l < NU; ++l) acc += ops[O.Mup + l * NPP + j] * x[l] + ops[O.Gp + j * NU + l] * y[l];
        Y[q + NPP * (j + NPP * line)] = acc;
      }
    } else {
      const int z = line - NU;  // < NU: the cell's z, else the z neighbours' layers
      const double* p = X + (2 * NU2 + 2 * NU + NU * z) * NPP + q;
#pragma unroll
      for (int l = 0; l < NU; ++l) x[l] = M.hx * hy * p[l * NPP];
#pragma unroll
      for (int j = 0; j < NPP; ++j) {
        double acc = 0;
#pragma unroll
        for (int l = 0; l < NU; ++l) acc += ops[O.Mup + l * NPP + j] * x[l];
        Y[NY1 + q + NPP * (j + NPP * z)] = acc;
      }
    }
  }
  __syncthreads();
  // z lines, and write
  for (int it = tid; it < nc * NP2; it += 256) {
    const int cell = it / NP2, k = it - cell * NP2;
    const double* Y = s1 + cell * S1 + k;
    double x[NU], y[NU];
#pragma unroll
    for (int l = 0; l < NU; ++l) {
      x[l] = Y[NP2 * l];
      y[l] = Y[NY1 + NP2 * l];
    }
    const double e0 = Y[NY1 + NP2 * NU], e1 = Y[NY1 + NP2 * (NU + 1)];
    double* o = out + (int64_t)s_e[cell * 7] * NP3 + k;
#pragma unroll
    for (int q = 0; q < NPP; ++q) {
      double acc = q == 0 ? -0.5 * e0 : (q == NPP - 1 ? 0.5 * e1 : 0.0);
#pragma unroll
      for (int l = 0; l < NU; ++l) acc += ops[O.Mup + l * NPP + q] * x[l] + ops[O.Gp + q * NU + l] * y[l];
      o[q * NP2] = acc;
    }
  }
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

// A launch of its own for the cells away from the enriched layers costs 5 us or more.  While the general kernel's
// workgroups (one a cell) of all regular cells are resident at once, they take no longer than those of the interface
// cells alone, so `resident` is 256 CUs times the kernel's workgroups a CU.
RegularLayers split_layers(const dg_mesh* m, int64_t resident) {
  RegularLayers L = regular_layers(m);
  if (L.xnl > 0 && L.inl > 0 && (int64_t)m->P.nx * L.nl * m->P.nz <= resident) {
    L.inl = 0;
    L.xlo = L.lo;
    L.xnl = L.nl;
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
#define X(p, q)                                                                                                     \
  if (m->np_u == p && m->P.nq_u == q) {                                                                             \
    const unsigned nb = (unsigned)((nc + SepShape<p>::CB - 1) / SepShape<p>::CB);                                   \
    if (inverse_mass)                                                                                               \
      hipLaunchKernelGGL((viscous_regular_kernel<p, q, true>), dim3(nb), dim3(256), 0, s, M, off, u, out, (int)nc,  \
                         lo, nl);                                                                                   \
    else                                                                                                            \
      hipLaunchKernelGGL((viscous_regular_kernel<p, q, false>), dim3(nb), dim3(256), 0, s, M, off, u, out, (int)nc, \
                         lo, nl);                                                                                   \
    return check_hip(hipGetLastError(), "viscous kernel launch");                                                   \
  }
  X(3, 4) X(4, 4) X(4, 5) X(5, 7) X(6, 8)
#undef X
  return set_error(DG_ERR_UNSUPPORTED, "viscous operator: degree not compiled");
}

int launch_vorticity_regular(const dg_mesh* m, const double* u, double* b, int lo, int nl, bool inverse_mass,
                             hipStream_t s) {
  if (nl <= 0) return DG_OK;
  const MeshDev M = velocity_meshdev(m);
  const int off = lin_offset(m->np_u, m->P.nq_u, m->P.nq_wn);
  const int64_t nc = (int64_t)m->P.nx * nl * m->P.nz;
#define X(p)                                                                                                        \
  if (m->np_u == p) {                                                                                               \
    const unsigned nb = (unsigned)((nc + SepShape<p>::CB - 1) / SepShape<p>::CB);                                   \
    if (inverse_mass)                                                                                               \
      hipLaunchKernelGGL((vorticity_regular_kernel<p, true>), dim3(nb), dim3(256), 0, s, M, off, u, b, (int)nc, lo,  \
                         nl);                                                                                       \
    else                                                                                                            \
      hipLaunchKernelGGL((vorticity_regular_kernel<p, false>), dim3(nb), dim3(256), 0, s, M, off, u, b, (int)nc, lo, \
                         nl);                                                                                       \
    return check_hip(hipGetLastError(), "vorticity kernel launch");                                                 \
  }
  X(3) X(4) X(5) X(6)
#undef X
  return set_error(DG_ERR_UNSUPPORTED, "vorticity: degree not compiled");
}

int launch_divgrad_regular(const dg_mesh* m, bool divergence, const double* in, double* out, int lo, int nl,
                           hipStream_t s) {
  if (nl <= 0) return DG_OK;
  const MeshDev M = velocity_meshdev(m);
  const int off = mix_offset(m->np_u, m->P.nq_u, m->P.nq_wn);
  const int64_t nc = (int64_t)m->P.nx * nl * m->P.nz;
#define X(p, q)                                                                                                      \
  if (m->np_u == p && m->np_p == q) {                                                                                \
    const unsigned nb = (unsigned)((nc + MixShape<p, q>::CB - 1) / MixShape<p, q>::CB);                              \
    if (divergence)                                                                                                  \
      hipLaunchKernelGGL((divergence_regular_kernel<p, q>), dim3(nb), dim3(256), 0, s, M, off, in, out, (int)nc, lo, \
                         nl);                                                                                        \
    else                                                                                                             \
      hipLaunchKernelGGL((gradient_regular_kernel<p, q>), dim3(nb), dim3(256), 0, s, M, off, in, out, (int)nc, lo,   \
                         nl);                                                                                        \
    return check_hip(hipGetLastError(), "divergence/gradient kernel launch");                                       \
  }
  X(3, 2) X(4, 3) X(5, 4) X(6, 5)
#undef X
  return set_error(DG_ERR_UNSUPPORTED, "pressure gradient / velocity divergence: degrees not compiled");
}

}  // namespace dgwm
