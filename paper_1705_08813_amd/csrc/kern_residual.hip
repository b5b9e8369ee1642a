// Velocity residual of cells without enrichment (arXiv 1705.08813, Sec. 4.2)
// on box meshes.
//
// Convective terms: volume and faces by the velocity rule.  Their integrands
// need only u at the points and only value tests on the faces, so a line of
// points is interpolated, multiplied and integrated back in the registers of
// one thread; derivatives are taken at the nodes, where
//   int d_d phi f = Dn_d^T (S x S x S)^T w f   (phi' is in the span of the basis).
// Viscous terms: linear with constant nu, so they separate exactly into 1-D
// operators (ip_line.h); only an enriched neighbour's psi u~ enters the flux by
// quadrature.
//
// 64 x 32 x 32 mesh, k = 4, 61,440 cells: 680 us in FP64 and 415 us in FP32, where
// the collocation-gradient kernel took 1,224 us and 770 us.  It is bound by the
// vector unit (some 5,000 instructions a cell, 72% busy) and the eight
// barriers of a cell; memory would allow 110 us (0.55 GB).
#include "batch.h"
#include "ip_line.h"
#include "velocity.h"

namespace dgwm {

namespace {

// Cells of a workgroup: small degrees share one, so that the point lines of
// its cells fill wavefronts.
template <int NP>
struct ResCells {
  static constexpr int CB = NP <= 4 ? 2 : 1;
};

template <int NP, int NQ, bool VISC>
struct ResShape {
  using L = NodeLds<NP>;
  static constexpr int NP2 = NP * NP, NP3 = NP2 * NP, NQ2 = NQ * NQ;
  static constexpr int U = 3 * L::SC;            // nodal values
  static constexpr int NB = 18 * NP2;            // neighbour layers [face][c][NP2]
  static constexpr int A = 3 * NQ * NP2;         // after the x sweep
  static constexpr int B = 3 * NQ2 * NP;         // after the y sweep
  static constexpr int T1 = 2 * 18 * NQ * NP;    // face traces swept along t1 [side][face][c][q1][i2]
  static constexpr int Z = 6 * NQ2 * NP;         // products u_c u_d integrated along z
  static constexpr int Y = 6 * NQ * NP2;         // ... and along y
  static constexpr int P = 6 * L::SC;            // ... and along x: nodal
  static constexpr int FB = 18 * NP2;            // face value tests [face][c][NP2]
  static constexpr int J = VISC ? 12 * NP2 : 0;  // tangential jumps [D][2][side][NP2]
  static constexpr int W = VISC ? U : 0, R = VISC ? U : 0;
  // region 1: U, neighbour values, neighbour derivatives, A; later Z; later P
  static constexpr int R1a = U + NB + (VISC ? NB : 0) + A, R1b = R1a > Z ? R1a : Z, R1 = R1b > P ? R1b : P;
  // region 2: B, W, J; later Y; later the nodal convective rows along z and along y
  static constexpr int R2a = B + W + J, R2b = R2a > Y ? R2a : Y, R2 = R2b > 2 * U ? R2b : 2 * U;
  // region 3: T1; the integrated face fluxes replace the own side, the face tests the neighbour's
  static constexpr int R3 = T1;
  static constexpr int CELL = R1 + R2 + R3 + R;
  static_assert(FB <= T1 / 2, "face tests fit the neighbour's half of the traces");
};

// What the threads of a workgroup need to know about one of its cells.
template <typename T>
struct CellInfo {
  int e, nb[6];      // cell and neighbours (-1: wall)
  int enr[2];        // enriched index of the neighbours across y = 0 and y = 1, or -1
  T h[3], ih[3];     // sizes and their reciprocals
  T ihn[2];          // reciprocal heights of the y neighbours
};

template <typename T, int NP, int NQ, bool VISC>
__device__ __forceinline__ void residual_cells(const MeshDev& M, const T* __restrict__ u, T* __restrict__ r, int first,
                                               int ncells, int layer_lo, int nlayers) {
  using Sh = ResShape<NP, NQ, VISC>;
  using L = NodeLds<NP>;
  constexpr int CB = ResCells<NP>::CB, NP2 = Sh::NP2, NP3 = Sh::NP3, NQ2 = Sh::NQ2, TPC = 3 * NP2, NT = 256;
  static_assert(CB * TPC <= 128, "the lines of the workgroup's cells fit two wavefronts");
  static_assert(CB * 2 * NP2 <= NT, "one thread per node of the y faces");
  static_assert(CB * 12 * NQ <= 128 && CB * 2 * NQ2 <= 128, "half lines of points fit two wavefronts each");
  constexpr int HQ = (NQ + 1) / 2, HP = (NP + 1) / 2;
  constexpr LinOps O = lin_ops(NP);
  constexpr auto& tb = ct::tab<NP, NQ>;
  constexpr bool F64 = sizeof(T) == 8;
  __shared__ T s_mem[CB * Sh::CELL];
  __shared__ CellInfo<T> s_ci[CB];
  __shared__ T s_psi[CB * 2 * NP2];  // enriched y neighbours: psi projected on the face basis
  __shared__ T s_ut[CB * 6];         // their coefficients
  __shared__ T s_e[NP2], s_w[NQ];
  const int tid = threadIdx.x;
  // coefficients come as wide scalar loads from the mesh's tables
  const double* const ops_at = M.tab + M.lin_off + (F64 ? 0 : O.f32);
  const double* const S_at = M.tab + (F64 ? 0 : M.proj_off + NP * NQ);
  ConstTab<T> ops = const_tab<T>(ops_at), tabS = const_tab<T>(S_at);
  auto phase = [&]() __attribute__((always_inline)) {  // (see const_tab)
    __syncthreads();
    ops = const_tab<T>(ops_at);
    tabS = const_tab<T>(S_at);
  };
  auto S = [&](int q, int i) { return tabS[q * NP + i]; };
  const int nc = CB == 1 ? 1 : (ncells - first < CB ? ncells - first : CB);

  if (tid < nc) {
    CellInfo<T>& I = s_ci[tid];
    const int i = first + tid;
    const int ex = i % M.nx, t0 = i / M.nx;
    const int ey = layer_lo + t0 % nlayers, ez = t0 / nlayers;
    const int e = ex + M.nx * (ey + M.ny * ez);
    I.e = e;
#pragma unroll
    for (int f = 0; f < 6; ++f) I.nb[f] = cell_nb(M, e, ex, ey, ez, f >> 1, f & 1);
    const int y0 = ey == 0 ? M.ny - 1 : ey - 1, y1 = ey + 1 == M.ny ? 0 : ey + 1;
    I.enr[0] = I.nb[2] < 0 ? -1 : (int)enr_index(M, ex, y0, ez);
    I.enr[1] = I.nb[3] < 0 ? -1 : (int)enr_index(M, ex, y1, ez);
    I.h[0] = T(M.hx);
    I.h[1] = T(M.hy[ey]);
    I.h[2] = T(M.hz);
    I.ih[0] = T(M.ihx);
    I.ih[1] = T(M.ihy[ey]);
    I.ih[2] = T(M.ihz);
    I.ihn[0] = T(M.ihy[y0]);
    I.ihn[1] = T(M.ihy[y1]);
  }
  if (tid < NP2) s_e[tid] = ops[O.E + tid];
  if (tid >= 64 && tid < 64 + NQ) s_w[tid - 64] = T(M.tab[tab_layout(NP, NQ, NQ).w + tid - 64]);
  __syncthreads();

  // load, one thread per (side, component, line): the cells' values along x,
  // and on the neighbours' lines along x, y, z the value and (viscous terms)
  // the normal derivative on the shared face
  if ((tid & 127) < nc * TPC) {
    const int s = __builtin_amdgcn_readfirstlane(tid >> 7);
    const int cell = (tid & 127) / TPC, ck = (tid & 127) - cell * TPC;
    const int cc = ck / NP2, kk = ck - cc * NP2;
    const CellInfo<T>& I = s_ci[cell];
    T* m = s_mem + cell * Sh::CELL;
    T own[NP], y[3][VISC ? NP : 1];
    if (s == 0) {
      const T* p = u + ((int64_t)I.e * 3 + cc) * NP3 + NP * kk;
#pragma unroll
      for (int l = 0; l < NP; ++l) own[l] = p[l];
    }
#pragma unroll
    for (int D = 0; D < 3; ++D) {
      const int nb = I.nb[2 * D + s];
      int base, st;
      vec_line<NP>(D, kk % NP, kk / NP, base, st);
      const T* p = u + ((int64_t)(nb < 0 ? I.e : nb) * 3 + cc) * NP3 + base;
      if constexpr (VISC) {
#pragma unroll
        for (int l = 0; l < NP; ++l) y[D][l] = p[l * st];
      } else {
        y[D][0] = p[(s ? 0 : NP - 1) * st];
      }
    }
    if (s == 0) {
      T* o = m + cc * L::SC + L::SJ * kk;
#pragma unroll
      for (int l = 0; l < NP; ++l) o[l] = own[l];
    }
#pragma unroll
    for (int D = 0; D < 3; ++D) {
      T* o = m + Sh::U + ((2 * D + s) * 3 + cc) * NP2 + kk;
      if constexpr (VISC) {
        // the neighbour below (s = 0) meets the cell at its xi_D = 1
        T d = 0;
#pragma unroll
        for (int l = 0; l < NP; ++l) d += ops[(s ? O.nd0 : O.nd1) + l] * y[D][l];
        o[0] = s ? y[D][0] : y[D][NP - 1];
        o[Sh::NB] = d * (D == 1 ? I.ihn[s] : I.ih[D]);
      } else {
        o[0] = y[D][0];
      }
    }
  }
  // an enriched neighbour across a y face: its coefficients, and the face
  // projection of its psi (the viscous jump terms test it with polynomials)
  if (tid < nc * 6) {
    const int cell = tid / 6, i = tid - cell * 6;
    const int en = s_ci[cell].enr[i / 3];
    if (en >= 0) s_ut[tid] = u[M.enr_off + (int64_t)en * 3 + i % 3];
  }
  if constexpr (VISC) {
    const int cell = tid / (2 * NP2), i = tid - cell * 2 * NP2;
    const int s = i / NP2, k = i - s * NP2;
    const int en = cell < nc ? s_ci[cell].enr[s] : -1;
    if (en >= 0) s_psi[tid] = T(psi_face_node<NP, NQ>(M, en, 2 + (1 - s), k % NP, k / NP));
  }
  phase();

  // the viscous line of this thread: (cell, component, tangential indices); the
  // first two wavefronts take the x and y lines, the others the z lines
  const bool upper = __builtin_amdgcn_readfirstlane(tid >> 7);
  const int vcell = (tid & 127) / TPC, vt = (tid & 127) - vcell * TPC;
  const int c = vt / NP2, k = vt - c * NP2, a = k % NP, b = k / NP;
  const bool vlive = VISC && vcell < nc;
  T* vm = s_mem + (vlive ? vcell : 0) * Sh::CELL;
  T* vu = vm;
  T* vw = vm + Sh::R1 + Sh::B;
  T* vj = vw + Sh::W;
  T* vr = vm + Sh::R1 + Sh::R2 + Sh::R3 + c * L::SC;
  const CellInfo<T>& VI = s_ci[vlive ? vcell : 0];
  const T theta = T(M.theta);
  T x[NP], qz[NP];
  // the scalar interior-penalty operator of component c along D on one line,
  // and its jumps for the cross terms (D != c); an enriched neighbour's psi u~
  // enters the adjoint terms here and the flux at the points below
  auto line = [&](int D, const T (&p)[NP], T (&q)[NP]) __attribute__((always_inline)) {
    IpEnds<T> n;
    const T rd = D == 0 ? VI.ih[0] : (D == 1 ? VI.ih[1] : VI.ih[2]);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const T* o = vm + Sh::U + ((2 * D + s) * 3 + c) * NP2 + k;
      n.v[s] = o[0];
      n.d[s] = o[Sh::NB];
      n.wall[s] = VI.nb[2 * D + s] < 0;
      const T rn = D == 1 && VI.ihn[s] > rd ? VI.ihn[s] : rd;
      n.tau[s] = n.wall[s] ? T(M.pen * M.wall_mult) * rd : T(M.pen) * rn;
    }
    T J[2];
    ip_line(ops, c == D, rd, theta, n, p, q, J, [&](T (&j)[2]) __attribute__((always_inline)) {
      if (D == 1) {
        const T* ps = s_psi + vcell * 2 * NP2 + k;
        if (VI.enr[0] >= 0) j[0] -= ps[0] * s_ut[vcell * 6 + c];
        if (VI.enr[1] >= 0) j[1] -= ps[NP2] * s_ut[vcell * 6 + 3 + c];
      }
    });
    if (c != D) {
      T* o = vj + (D * 2 + (c < D ? c : c - 1)) * 2 * NP2 + k;
      o[0] = J[0];
      o[NP2] = J[1];
    }
  };
  // W_c: the weak derivative of component c along direction c
  auto weak = [&]() __attribute__((always_inline)) {
    int lb, ls;
    L::line(c, a, b, lb, ls);
    const T* p = vu + c * L::SC + lb;
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = p[l * ls];
    const T* o = vm + Sh::U + 7 * c * NP2 + k;  // face 2 c, component c
    ip_weak(ops, VI.ih[c], VI.nb[2 * c] < 0, VI.nb[2 * c + 1] < 0, o[0], o[3 * NP2], x, vw + c * L::SC + lb, ls);
  };
  auto mass = [&](int D) __attribute__((always_inline)) {  // M along D on this thread's line of the viscous rows
    int lb, ls;
    L::line(D, a, b, lb, ls);
    T* p = vr + lb;
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = p[l * ls];
    if (D == 2) {
#pragma unroll
      for (int l = 0; l < NP; ++l) x[l] += qz[l];
    }
    ip_mass(ops, x, p, ls);
  };
  const int wt = (tid + 128) & 255;  // items of the point phases start at the third wavefront

  // 1: viscous x lines | interpolation along x, face layers along t1
  if (vlive && !upper) {
    T q[NP];
    int lb, ls;
    L::line(0, a, b, lb, ls);
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = vu[c * L::SC + lb + l];
    line(0, x, q);
#pragma unroll
    for (int l = 0; l < NP; ++l) vr[lb + l] = q[l];
    weak();
  }
  for (int it = wt; it < nc * 3 * NP2; it += NT) {
    const int cell = it / (3 * NP2), i = it - cell * 3 * NP2;
    T* m = s_mem + cell * Sh::CELL;
    const int cc = i / NP2, jm = i - cc * NP2;
    const T* p = m + cc * L::SC + L::SJ * jm;
    T* o = m + (VISC ? 2 : 1) * Sh::NB + Sh::U + NQ * i;
    T y[NP];
#pragma unroll
    for (int l = 0; l < NP; ++l) y[l] = p[l];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      T acc = 0;
#pragma unroll
      for (int l = 0; l < NP; ++l) acc += S(q, l) * y[l];
      o[q] = acc;
    }
  }
  for (int it = VISC ? wt : tid; it < nc * 36 * NP; it += VISC ? 128 : NT) {
    if (VISC && wt >= 128) break;
    const int cell = it / (36 * NP), i = it - cell * 36 * NP;
    T* m = s_mem + cell * Sh::CELL;
    const int side = i / (18 * NP), fi = i - side * 18 * NP;      // fi = (face * 3 + c) * NP + i2
    const int fc = fi / NP, i2 = fi - fc * NP, f = fc / 3, cc = fc - 3 * f;
    const int D = f >> 1, s = f & 1;
    T y[NP];
    if (side == 0) {
      // the layer of face (D, s): t1 runs along x (D != 0) or y
      const int t1 = D == 0 ? L::SJ : 1, t2 = D == 2 ? L::SJ : L::SK;
      const T* p = m + cc * L::SC + (s ? (NP - 1) * (D == 0 ? 1 : (D == 1 ? L::SJ : L::SK)) : 0) + t2 * i2;
#pragma unroll
      for (int l = 0; l < NP; ++l) y[l] = p[l * t1];
    } else {
      const T* p = m + Sh::U + fc * NP2 + NP * i2;
#pragma unroll
      for (int l = 0; l < NP; ++l) y[l] = p[l];
    }
    T* o = m + Sh::R1 + Sh::R2 + side * 18 * NQ * NP + fc * NQ * NP + i2;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      T acc = 0;
#pragma unroll
      for (int l = 0; l < NP; ++l) acc += S(q, l) * y[l];
      o[q * NP] = acc;
    }
  }
  phase();

  // 2: viscous y lines | viscous z lines, interpolation along y
  if (vlive && !upper) {
    T q[NP];
    int lb, ls;
    L::line(1, a, b, lb, ls);
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = vu[c * L::SC + lb + l * ls];
    line(1, x, q);
#pragma unroll
    for (int l = 0; l < NP; ++l) vr[lb + l * ls] += q[l];
  }
  if (vlive && upper) {
    int lb, ls;
    L::line(2, a, b, lb, ls);
#pragma unroll
    for (int l = 0; l < NP; ++l) x[l] = vu[c * L::SC + lb + l * ls];
    line(2, x, qz);
  }
  for (int it = wt; it < nc * 3 * NQ * NP; it += NT) {
    const int cell = it / (3 * NQ * NP), i = it - cell * 3 * NQ * NP;
    T* m = s_mem + cell * Sh::CELL;
    const int cc = i / (NQ * NP), qm = i - cc * NQ * NP, mm = qm / NQ, q0 = qm - mm * NQ;
    const T* p = m + (VISC ? 2 : 1) * Sh::NB + Sh::U + cc * NQ * NP2 + q0 + NQ * NP * mm;
    T* o = m + Sh::R1 + cc * NQ2 * NP + q0 + NQ2 * mm;
    T y[NP];
#pragma unroll
    for (int l = 0; l < NP; ++l) y[l] = p[l * NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      T acc = 0;
#pragma unroll
      for (int l = 0; l < NP; ++l) acc += S(q, l) * y[l];
      o[q * NQ] = acc;
    }
  }
  phase();

  // 3: numerical flux on the lines of face points | products on the z lines of
  // volume points | viscous cross terms
  // A pair of lanes shares a line: lane h = 0 takes its points q = 0, 1, ... from
  // one end, lane h = 1 from the other.  The rule and the basis are symmetric,
  // S[n_q-1-q][k-l] = S[q][l], so the second lane reads the line's nodes in
  // reverse and both use the same coefficients; the middle point of an odd rule
  // belongs to the first.  Each lane integrates its points and the pair adds up.
  if (tid < nc * 12 * NQ) {
    const int h = tid & 1, ln = tid >> 1;
    const int cell = ln / (6 * NQ), i = ln - cell * 6 * NQ;
    const int f = i / NQ, q1 = i - f * NQ, D = f >> 1, s = f & 1;
    const CellInfo<T>& I = s_ci[cell];
    T* t0 = s_mem + cell * Sh::CELL + Sh::R1 + Sh::R2 + f * 3 * NQ * NP + q1 * NP;
    const int nb0 = h ? NP - 1 : 0, nst = h ? -1 : 1;
    const T sg = s ? T(1) : T(-1);
    const T w1 = s_w[q1] * (D == 0 ? I.h[1] * I.h[2] : (D == 1 ? I.h[0] * I.h[2] : I.h[0] * I.h[1]));
    // components in the order normal, t1, t2
    const int comp[3] = {D, D == 0 ? 1 : 0, D == 2 ? 1 : 2};
    T um[3][HQ], up[3][HQ];
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
      const T* tc = t0 + comp[cc] * NQ * NP + nb0;
      T y[NP], z[NP];
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        y[l] = tc[nst * l];
        z[l] = tc[18 * NQ * NP + nst * l];
      }
#pragma unroll
      for (int q = 0; q < HQ; ++q) {
        T am = 0, ap = 0;
#pragma unroll
        for (int l = 0; l < NP; ++l) {
          am += S(q, l) * y[l];
          ap += S(q, l) * z[l];
        }
        um[cc][q] = am;
        up[cc][q] = ap;
      }
    }
    if (I.nb[f] < 0) {  // mirror state on a wall
#pragma unroll
      for (int cc = 0; cc < 3; ++cc)
#pragma unroll
        for (int q = 0; q < HQ; ++q) up[cc][q] = -um[cc][q];
    }
    const int en = D == 1 ? I.enr[s] : -1;
    const double* ps = en >= 0 ? M.psi + ((size_t)en * M.psi_pts + M.psi_off[1 + 2 + (1 - s)] + q1 + (h ? NQ * (NQ - 1) : 0)) * 4
                               : nullptr;
    const int pst = h ? -4 * NQ : 4 * NQ;
    const T* ut = s_ut + cell * 6 + 3 * s;
    if (en >= 0) {  // u+ takes psi u~ (a y face: normal component 1)
#pragma unroll
      for (int q = 0; q < HQ; ++q) {
        const T pv = T(ps[pst * q]);
        up[0][q] += pv * ut[1];
        up[1][q] += pv * ut[0];
        up[2][q] += pv * ut[2];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int q = 0; q < HQ; ++q) {
      const T w = w1 * (2 * q + 1 == NQ && h ? T(0) : T(tb.w[q]));
      const T wm = w * um[0][q], wp = w * up[0][q];
      const T am = wm < 0 ? -wm : wm, ap = wp < 0 ? -wp : wp;
      const T lam = am > ap ? am : ap;  // w Lambda / 2
      const T hm = T(0.5) * sg * wm, hp = T(0.5) * sg * wp;
#pragma unroll
      for (int cc = 0; cc < 3; ++cc)
        um[cc][q] = um[cc][q] * hm + up[cc][q] * hp + lam * (um[cc][q] - up[cc][q]);
    }
    if (VISC && en >= 0) {  // the viscous flux takes its gradient and its jump
      const T hn = -T(0.5) * T(M.nu) * sg;
      const T taun = T(M.nu) * T(M.pen) * (I.ihn[s] > I.ih[1] ? I.ihn[s] : I.ih[1]);
#pragma unroll
      for (int q = 0; q < HQ; ++q) {
        const T pv = T(ps[pst * q]), g0 = T(ps[pst * q + 1]), g1 = T(ps[pst * q + 2]), g2 = T(ps[pst * q + 3]);
        const T w = w1 * (2 * q + 1 == NQ && h ? T(0) : T(tb.w[q]));
        um[0][q] += w * (hn * (T(2) * ut[1] * g1) - taun * pv * ut[1]);
        um[1][q] += w * (hn * (ut[0] * g1 + ut[1] * g0) - taun * pv * ut[0]);
        um[2][q] += w * (hn * (ut[2] * g1 + ut[1] * g2) - taun * pv * ut[2]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
      T* tc = t0 + comp[cc] * NQ * NP + nb0;
      T o[NP];
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        T acc = 0;
#pragma unroll
        for (int q = 0; q < HQ; ++q) acc += S(q, l) * um[cc][q];
        o[l] = acc;
      }
#pragma unroll
      for (int l = 0; l < HP; ++l) tc[nst * l] = o[l] + pair_swap(o[NP - 1 - l]);
    }
  }
  if (tid >= 128 && tid - 128 < nc * 2 * NQ2) {
    const int h = tid & 1, ln = (tid - 128) >> 1;
    const int cell = ln / NQ2, pq = ln - cell * NQ2;
    T* m = s_mem + cell * Sh::CELL;
    const int nb0 = h ? NQ2 * (NP - 1) : 0, nst = h ? -NQ2 : NQ2;
    const T* p = m + Sh::R1 + pq + nb0;
    T v[3][HQ];
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
      T y[NP];
#pragma unroll
      for (int l = 0; l < NP; ++l) y[l] = p[cc * NQ2 * NP + nst * l];
#pragma unroll
      for (int q = 0; q < HQ; ++q) {
        T acc = 0;
#pragma unroll
        for (int l = 0; l < NP; ++l) acc += S(q, l) * y[l];
        v[cc][q] = acc;
      }
    }
    const T wxy = s_w[pq % NQ] * s_w[pq / NQ];
    T* o = m + pq + nb0;
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
      T wv[HQ];
#pragma unroll
      for (int q = 0; q < HQ; ++q) wv[q] = wxy * (2 * q + 1 == NQ && h ? T(0) : T(tb.w[q])) * v[cc][q];
#pragma unroll
      for (int d = cc; d < 3; ++d) {
        const int pr = cc == 0 ? d : (cc == 1 ? 2 + d : 5);  // pairs 00 01 02 11 12 22
        T z[NP];
#pragma unroll
        for (int l = 0; l < NP; ++l) {
          T acc = 0;
#pragma unroll
          for (int q = 0; q < HQ; ++q) acc += S(q, l) * (wv[q] * v[d][q]);
          z[l] = acc;
        }
#pragma unroll
        for (int l = 0; l < HP; ++l) o[pr * NQ2 * NP + nst * l] = z[l] + pair_swap(z[NP - 1 - l]);
      }
    }
  }
  if constexpr (VISC) {
    const int t = tid ^ 128;  // with the volume points, whose lines are shorter
    if (t < nc * TPC) {
      const int cell = t / TPC, i = t - cell * TPC;
      const int cc = i / NP2, kk = i - cc * NP2, aa = kk % NP, bb = kk / NP;
      T* m = s_mem + cell * Sh::CELL;
      const CellInfo<T>& I = s_ci[cell];
      const int d1 = cc == 0 ? 1 : 0, d2 = cc == 2 ? 1 : 2;
      int lb, ls;
      L::line(cc, aa, bb, lb, ls);
      const T* w1 = m + Sh::R1 + Sh::B + d1 * L::SC + lb;
      const T* w2 = m + Sh::R1 + Sh::B + d2 * L::SC + lb;
      T y[NP];
#pragma unroll
      for (int l = 0; l < NP; ++l) y[l] = w1[l * ls] + w2[l * ls];
      const T ihc = cc == 0 ? I.ih[0] : (cc == 1 ? I.ih[1] : I.ih[2]);
      const T ih1 = cc == 0 ? I.ih[1] : I.ih[0], ih2 = cc == 2 ? I.ih[1] : I.ih[2];
      const T* j1 = m + Sh::R1 + Sh::B + Sh::W + (cc * 2) * 2 * NP2;
      ip_cross(ops, s_e, theta, ihc, ih1, ih2, aa, bb, j1, j1 + 2 * NP2, y, m + Sh::R1 + Sh::R2 + Sh::R3 + cc * L::SC + lb,
               ls);
    }
  }
  phase();

  // 4: viscous rows: mass along z | products along y | face fluxes along t1
  if (vlive && upper) mass(2);
  for (int it = tid; it < nc * 6 * NQ * NP; it += NT) {
    const int cell = it / (6 * NQ * NP), i = it - cell * 6 * NQ * NP;
    T* m = s_mem + cell * Sh::CELL;
    const int pr = i / (NQ * NP), qm = i - pr * NQ * NP, mm = qm / NQ, q0 = qm - mm * NQ;
    const T* p = m + pr * NQ2 * NP + q0 + NQ2 * mm;
    T* o = m + Sh::R1 + pr * NQ * NP2 + q0 + NQ * NP * mm;
    T y[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) y[q] = p[q * NQ];
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      T acc = 0;
#pragma unroll
      for (int q = 0; q < NQ; ++q) acc += S(q, l) * y[q];
      o[l * NQ] = acc;
    }
  }
  for (int it = tid; it < nc * 18 * NP; it += NT) {
    const int cell = it / (18 * NP), i = it - cell * 18 * NP;
    T* m = s_mem + cell * Sh::CELL + Sh::R1 + Sh::R2;
    const int fc = i / NP, i2 = i - fc * NP;
    const T* p = m + fc * NQ * NP + i2;
    T* o = m + 18 * NQ * NP + fc * NP2 + NP * i2;
    T y[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) y[q] = p[q * NP];
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      T acc = 0;
#pragma unroll
      for (int q = 0; q < NQ; ++q) acc += S(q, l) * y[q];
      o[l] = acc;
    }
  }
  phase();

  // 5: mass along y | products along x
  if (vlive && !upper) mass(1);
  for (int it = wt; it < nc * 6 * NP2; it += NT) {
    const int cell = it / (6 * NP2), i = it - cell * 6 * NP2;
    T* m = s_mem + cell * Sh::CELL;
    const int pr = i / NP2, jm = i - pr * NP2;
    const T* p = m + Sh::R1 + NQ * i;
    T* o = m + pr * L::SC + L::SJ * jm;
    T y[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) y[q] = p[q];
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      T acc = 0;
#pragma unroll
      for (int q = 0; q < NQ; ++q) acc += S(q, l) * y[q];
      o[l] = acc;
    }
  }
  phase();

  // 6: convective rows, derivative tests along z and along y with the face tests of those directions
  for (int it = tid; it < nc * 2 * TPC; it += NT) {
    const int cell = it / (2 * TPC), j = it - cell * 2 * TPC;
    const int D = j < TPC ? 2 : 1, i = j < TPC ? j : j - TPC;
    const int cc = i / NP2, kk = i - cc * NP2;
    T* m = s_mem + cell * Sh::CELL;
    const CellInfo<T>& I = s_ci[cell];
    int lb, ls;
    L::line(D, kk % NP, kk / NP, lb, ls);
    const int lo = cc < D ? cc : D, hi = cc < D ? D : cc;
    const T* p = m + (lo == 0 ? hi : (lo == 1 ? 2 + hi : 5)) * L::SC + lb;
    T y[NP];
#pragma unroll
    for (int l = 0; l < NP; ++l) y[l] = p[l * ls];
    // -|J| / h_D
    const T sc = -I.h[0] * (D == 2 ? I.h[1] : I.h[2]);
    const T* fb = m + Sh::R1 + Sh::R2 + 18 * NQ * NP + (2 * D * 3 + cc) * NP2 + kk;
    T* o = m + Sh::R1 + (D == 2 ? 0 : Sh::U) + cc * L::SC + lb;
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      T acc = 0;
#pragma unroll
      for (int n = 0; n < NP; ++n) acc += ops[O.Dn + n * NP + l] * y[n];
      acc *= sc;
      if (l == 0) acc += fb[0];
      if (l == NP - 1) acc += fb[3 * NP2];
      o[l * ls] = acc;
    }
  }
  phase();

  // 7: along x: the last derivative tests, mass of the viscous rows; write
  for (int it = tid; it < nc * TPC; it += NT) {
    const int cell = it / TPC, i = it - cell * TPC;
    const int cc = i / NP2, kk = i - cc * NP2;
    T* m = s_mem + cell * Sh::CELL;
    const CellInfo<T>& I = s_ci[cell];
    const int lb = L::SJ * kk;
    const T* p = m + cc * L::SC + lb;                   // pairs 00, 01, 02
    const T* pz = m + Sh::R1 + cc * L::SC + lb;
    const T* pr = m + Sh::R1 + Sh::R2 + Sh::R3 + cc * L::SC + lb;
    T y[NP], v[NP];
#pragma unroll
    for (int l = 0; l < NP; ++l) y[l] = p[l];
    if (VISC) {
#pragma unroll
      for (int l = 0; l < NP; ++l) v[l] = pr[l];
    }
    const T sc = -I.h[1] * I.h[2];
    const T vs = T(M.nu) * (I.h[0] * I.h[1] * I.h[2]);
    const T* fb = m + Sh::R1 + Sh::R2 + 18 * NQ * NP + cc * NP2 + kk;
    T* o = r + ((int64_t)I.e * 3 + cc) * NP3 + NP * kk;
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      T acc = 0;
#pragma unroll
      for (int n = 0; n < NP; ++n) acc += ops[O.Dn + n * NP + l] * y[n];
      acc = sc * acc + (pz[l] + pz[Sh::U + l]);
      if (VISC) {
        T w = 0;
#pragma unroll
        for (int n = 0; n < NP; ++n) w += ops[O.M + l * NP + n] * v[n];
        acc += vs * w;
      }
      if (l == 0) acc += fb[0];
      if (l == NP - 1) acc += fb[3 * NP2];
      o[l] = acc;
    }
  }
}

// Workgroups per CU the launch bounds plan for: as many as the LDS holds, up
// to the register budget that keeps the flux lines out of scratch (128 at four).
template <typename T, int NP>
__host__ __device__ constexpr int res_wg_per_cu() {
  return NP == 6 ? (sizeof(T) == 8 ? 2 : 3) : 4;
}

template <typename T, int NP, int NQ, bool VISC>
__global__ __launch_bounds__(256, (res_wg_per_cu<T, NP>())) void residual_kernel(const MeshDev M, const T* __restrict__ u, T* __restrict__ r,
                                                       int ncells, int layer_lo, int nlayers) {
  residual_cells<T, NP, NQ, VISC>(M, u, r, xcd_block(gridDim.x, blockIdx.x) * ResCells<NP>::CB, ncells, layer_lo,
                                  nlayers);
}

// Cells of many meshes in one launch (see vel_kernel_batched); a workgroup
// holds cells of one mesh.
template <typename T, int NP, int NQ>
__global__ __launch_bounds__(256, (res_wg_per_cu<T, NP>())) void residual_kernel_batched(const VelBatchItem* __restrict__ items,
                                                               const int64_t* __restrict__ prefix, int nitems) {
  const int lo = batch_item(prefix, nitems);
  const VelBatchItem& it = items[lo];
  residual_cells<T, NP, NQ, true>(it.M, static_cast<const T*>(it.u), static_cast<T*>(it.r),
                                  (int)(blockIdx.x - prefix[lo]) * ResCells<NP>::CB, it.ncells, it.layer_lo,
                                  it.nlayers);
}

}  // namespace

#define DG_RES_COMBOS(X) X(3, 4) X(4, 4) X(4, 5) X(5, 7) X(6, 8)

int residual_cells_per_block(int np) {
  switch (np) {
    case 3: return ResCells<3>::CB;
    case 4: return ResCells<4>::CB;
    case 5: return ResCells<5>::CB;
    case 6: return ResCells<6>::CB;
  }
  return 0;
}

template <typename T>
int launch_residual_regular(const dg_mesh* m, const T* u, T* r, int lo, int nl, bool viscous, hipStream_t s) {
  if (nl <= 0) return DG_OK;
  const MeshDev M = velocity_meshdev(m);
  const int64_t nc = (int64_t)m->P.nx * nl * m->P.nz;
#define X(p, q)                                                                                                \
  if (m->np_u == p && m->P.nq_u == q) {                                                                        \
    const unsigned nb = (unsigned)((nc + ResCells<p>::CB - 1) / ResCells<p>::CB);                              \
    if (viscous)                                                                                               \
      hipLaunchKernelGGL((residual_kernel<T, p, q, true>), dim3(nb), dim3(256), 0, s, M, u, r, (int)nc, lo, nl); \
    else                                                                                                       \
      hipLaunchKernelGGL((residual_kernel<T, p, q, false>), dim3(nb), dim3(256), 0, s, M, u, r, (int)nc, lo, nl); \
    return check_hip(hipGetLastError(), "residual kernel launch");                                             \
  }
  DG_RES_COMBOS(X)
#undef X
  return set_error(DG_ERR_UNSUPPORTED, "velocity degree/quadrature combination not compiled");
}
template int launch_residual_regular<double>(const dg_mesh*, const double*, double*, int, int, bool, hipStream_t);
template int launch_residual_regular<float>(const dg_mesh*, const float*, float*, int, int, bool, hipStream_t);

template <typename T>
int launch_residual_regular_batched(int np, int nq, const VelBatchItem* items, const int64_t* prefix, int n,
                                    int64_t blocks, hipStream_t s) {
  if (n <= 0 || blocks <= 0) return DG_OK;
#define X(p, q)                                                                                                     \
  if (np == p && nq == q) {                                                                                         \
    hipLaunchKernelGGL((residual_kernel_batched<T, p, q>), dim3((unsigned)blocks), dim3(256), 0, s, items, prefix, n); \
    return check_hip(hipGetLastError(), "batched residual kernel launch");                                          \
  }
  DG_RES_COMBOS(X)
#undef X
  return set_error(DG_ERR_UNSUPPORTED, "velocity combination not compiled");
}
template int launch_residual_regular_batched<double>(int, int, const VelBatchItem*, const int64_t*, int, int64_t,
                                                     hipStream_t);
template int launch_residual_regular_batched<float>(int, int, const VelBatchItem*, const int64_t*, int, int64_t,
                                                    hipStream_t);

}  // namespace dgwm
