// The viscous interior-penalty operator of a box cell in nodal form, one line
// of nodes at a time: what the residual (kern_residual.hip) and the multiscale
// viscous operator (kern_linear.hip) evaluate alike.
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
// `ops` holds the 1-D operators of lin_ops.
#pragma once

#include "kern_common.h"

namespace dgwm {

// What a cell's line along D meets at its two ends: the neighbours' values (as
// the jumps see them) and normal derivatives, the penalties, and walls.
template <typename T>
struct IpEnds {
  T v[2], d[2], tau[2];
  bool wall[2];
};

// q = Q_D p on a line of component c (own: c = D), and its two jumps J.
// `adjoint` may add to the jumps what only the adjoint terms see.
template <typename T, int NP, typename F>
__device__ __forceinline__ void ip_line(ConstTab<T> ops, bool own, T rd, T theta, const IpEnds<T>& n, const T (&p)[NP],
                                        T (&q)[NP], T (&J)[2], F&& adjoint) {
  constexpr LinOps O = lin_ops(NP);
  const T kap = own ? T(2) : T(1);
  T d0 = 0, d1 = 0;
#pragma unroll
  for (int l = 0; l < NP; ++l) {
    d0 += ops[O.nd0 + l] * p[l];
    d1 += ops[O.nd1 + l] * p[l];
  }
  d0 *= rd;
  d1 *= rd;
  // mirror states on a wall: u+ = -u-, grad u+ = grad u-
  J[0] = p[0] - (n.wall[0] ? -p[0] : n.v[0]);
  J[1] = p[NP - 1] - (n.wall[1] ? -p[NP - 1] : n.v[1]);
  const T s0 = d0 + (n.wall[0] ? d0 : n.d[0]), s1 = d1 + (n.wall[1] ? d1 : n.d[1]);
  const T G0 = rd * (T(0.5) * kap * s0 + n.tau[0] * J[0]), G1 = rd * (n.tau[1] * J[1] - T(0.5) * kap * s1);
  adjoint(J);
  const T r2 = kap * rd * rd, H0 = T(0.5) * theta * r2 * J[0], H1 = -T(0.5) * theta * r2 * J[1];
#pragma unroll
  for (int l = 0; l < NP; ++l) {
    T acc = 0;
#pragma unroll
    for (int m = 0; m < NP; ++m) acc += ops[O.A + l * NP + m] * p[m];
    q[l] = r2 * acc + ops[O.l0 + l] * G0 + ops[O.l1 + l] * G1 + ops[O.g0 + l] * H0 + ops[O.g1 + l] * H1;
  }
}

// w = W_d on a line along d, w at stride ws; v: the neighbours' values at its ends.
template <typename T, int NP>
__device__ __forceinline__ void ip_weak(ConstTab<T> ops, T rd, bool wall0, bool wall1, T v0, T v1, const T (&p)[NP], T* w,
                                        int ws) {
  constexpr LinOps O = lin_ops(NP);
  const T a0 = T(0.5) * (p[0] + (wall0 ? p[0] : v0)), a1 = T(0.5) * (p[NP - 1] + (wall1 ? p[NP - 1] : v1));
#pragma unroll
  for (int l = 0; l < NP; ++l) {
    T acc = ops[O.l0 + l] * a0 - ops[O.l1 + l] * a1;
#pragma unroll
    for (int m = 0; m < NP; ++m) acc += ops[O.E + l * NP + m] * p[m];
    w[l * ws] = rd * acc;
  }
}

// Cross terms on the line (a, b) of component c along c: x = W_{d1} + W_{d2} on it, j1 and j2 the jumps of the components
// d1 (along a) and d2 (along b) on the faces normal to c, [side][NP2]; E in LDS; added to p at stride ps.
template <typename T, int NP>
__device__ __forceinline__ void ip_cross(ConstTab<T> ops, const T* E, T theta, T ihc, T ih1, T ih2, int a, int b,
                                         const T* j1, const T* j2, const T (&x)[NP], T* p, int ps) {
  constexpr LinOps O = lin_ops(NP);
  constexpr int NP2 = NP * NP;
  T y[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    T s1 = 0, s2 = 0;
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      s1 += E[a * NP + j] * j1[s * NP2 + j + NP * b];
      s2 += E[b * NP + j] * j2[s * NP2 + a + NP * j];
    }
    y[s] = (s ? -T(0.5) : T(0.5)) * theta * ihc * (ih1 * s1 + ih2 * s2);
  }
#pragma unroll
  for (int l = 0; l < NP; ++l) {
    T acc = 0;
#pragma unroll
    for (int m = 0; m < NP; ++m) acc += ops[O.Dn + l * NP + m] * x[m];
    p[l * ps] += ihc * acc + ops[O.l0 + l] * y[0] + ops[O.l1 + l] * y[1];
  }
}

// y = f M x along a line, y at stride ys.
template <typename T, int NP>
__device__ __forceinline__ void ip_mass(ConstTab<T> ops, const T (&x)[NP], T* y, int ys, T f = T(1)) {
  constexpr LinOps O = lin_ops(NP);
#pragma unroll
  for (int l = 0; l < NP; ++l) {
    T acc = 0;
#pragma unroll
    for (int m = 0; m < NP; ++m) acc += ops[O.M + l * NP + m] * x[m];
    y[l * ys] = f * acc;
  }
}

}  // namespace dgwm
