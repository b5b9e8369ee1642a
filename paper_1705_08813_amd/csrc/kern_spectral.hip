// Direct solve of the element-wise projection step (arXiv 1705.08813, Sec.
// 4.2, eq. projectionspat) in cells without enrichment, FP64.
//
// In a cell of height h_y (flat mesh, affine cell) the system is
//   (M_e + D_e) x = M_e u_hat - s g,   M_e = |J| Mh,   D_e = |J| tau_D,e Dh,
// with Mh the reference mass (the tensor product K (x) K (x) K of the 1-D
// mass K of the velocity rule, per component) and Dh the div-div form with
// physical derivatives and reference weights; Mh and Dh depend on the layer
// only, tau_D,e on the cell.  With the Cholesky factor K = C C^T and
// L = C (x) C (x) C (Mh = L L^T), and the eigendecomposition of the
// whitened form  L^{-1} Dh L^{-T} = Z diag(lambda) Z^T  (once per distinct
// layer height, on the host, by the cyclic Jacobi method),
//   x = L^{-T} Z diag(1 / (1 + tau_D,e lambda)) Z^T L^T (u_hat - (s/|J|) Mh^{-1} g).
// Mh^{-1} is a sweep with 1-D matrices; L^T and L^{-T} are folded into the
// layer's tables (L Z)^T and L^{-T} Z.  The cell is symmetric under reflection
// in each direction, so in even/odd coordinates both tables fall into eight
// diagonal blocks (Parity in kern_tile.h); the change of coordinates is sums
// and differences along the three directions.  A workgroup takes a tile of 16
// cells of one layer and runs both block products out of LDS on the FP64
// matrix cores.  The result is exact up to rounding: no iteration, every cell
// the same work.
// Measured (64 x 32 x 32 cells, k = 4, 61,440 cells here): 305 us, 0.55 GB at
// 1.8 TB/s; with the dense 375 x 375 tables it was 1,196 us, bound by their
// products.  What is left is the LDS passes between barriers and, at the FP64
// matrix rate, 80 us of products.  Eight wavefronts on a tile instead of four
// fill the wait of one phase with another tile's work at the same LDS.
#include <algorithm>
#include <thread>
#include <vector>

#include "kern_common.h"
#include "kern_tile.h"
#include "symeig.h"

namespace dgwm {

namespace {


struct SpecArgs {
  int nx, ny, layer_lo, tiles, nblocks;  // tiles per layer; blocks in the launch
  int64_t ncol;                          // cells per layer (nx * nz)
  double hx, hz;
  const double* hy;     // [ny] cell heights
  const double* mats;   // [np][np]: K^{-1} (row-major, out_a = sum_i M[a][i] in_i)
  const double* slots;  // [slot]: first product, second product (operand order of BlockGemm), lambda (class order)
  const int32_t* map;   // [ny] slot of each layer
  const double* tau_d;
  const double* u_hat;
  const double* g;
  double scale;
  double* x;
};

template <int NP>
__global__ __launch_bounds__(tile_threads(NP), tile_waves(NP)) void spectral_step_kernel(const SpecArgs A) {
  constexpr int NP2 = NP * NP, NP3 = NP2 * NP, N = 3 * NP3, NC = kTileCols, LD = kTileLD, NT = tile_threads(NP);
  constexpr int PL = (NC * N + NT - 1) / NT;  // values of the tile per thread
  constexpr auto& P = parity<NP>;
  using Gemm = BlockGemm<NP, NT / 64>;
  __shared__ double T[Parity<NP>::ROWS * LD];
  __shared__ double Mt[NP2];
  __shared__ double tauc[NC];
  __shared__ int64_t base[NC];
  __shared__ short cls[N];
  // consecutive logical blocks (tiles of one layer) on one XCD: hardware
  // block b runs on XCD b % 8
  const int per = (A.nblocks + 7) / 8;
  const int lb = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
  if (lb >= A.nblocks) return;
  const int tid = threadIdx.x;
  const int layer = A.layer_lo + lb / A.tiles;
  const int64_t j0 = (int64_t)(lb % A.tiles) * NC;
  const int nc = A.ncol - j0 < NC ? (int)(A.ncol - j0) : NC;
  if (tid < NC) {
    const int64_t j = j0 + (tid < nc ? tid : 0);
    const int64_t e = j % A.nx + (int64_t)A.nx * layer + (int64_t)A.nx * A.ny * (j / A.nx);
    base[tid] = e * N;
    tauc[tid] = tid < nc ? A.tau_d[e] : 0.0;
  }
  for (int i = tid; i < NP2; i += NT) Mt[i] = A.mats[i];
  for (int i = tid; i < (Parity<NP>::ROWS - N) * LD; i += NT) T[N * LD + i] = 0.0;
  for (int i = tid; i < N; i += NT) cls[P.pos[i]] = (short)i;
  __syncthreads();
  double u[PL];
  auto fetch = [&](const double* __restrict__ src) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PL; ++i) {
      const int idx = tid + i * NT, c = idx / N;
      u[i] = c < nc ? src[base[c] + (idx - c * N)] : 0.0;
    }
  };
  fetch(A.g);
#pragma unroll
  for (int i = 0; i < PL; ++i) {
    const int idx = tid + i * NT, c = idx / N;
    if (idx < NC * N) T[(idx - c * N) * LD + c] = u[i];
  }
  fetch(A.u_hat);  // in flight over the sweeps
  __syncthreads();
  // Mh^{-1} g
  tile_sweep<NP, NT, 0>(T, Mt, tid);
  __syncthreads();
  tile_sweep<NP, NT, 1>(T, Mt, tid);
  __syncthreads();
  tile_sweep<NP, NT, 2>(T, Mt, tid);
  __syncthreads();
  const double f = A.scale / (A.hx * A.hy[layer] * A.hz);
#pragma unroll
  for (int i = 0; i < PL; ++i) {
    const int idx = tid + i * NT, c = idx / N;
    if (idx < NC * N) T[(idx - c * N) * LD + c] = u[i] - f * T[(idx - c * N) * LD + c];
  }
  __syncthreads();
  // (the factors L^T before and L^{-T} after the products are folded into the tables)
  const double* Z1 = A.slots + (size_t)A.map[layer] * (2 * (size_t)Parity<NP>::ZN + N);
  const double* Z2 = Z1 + Parity<NP>::ZN;
  const double* lam = Z2 + Parity<NP>::ZN;
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), col = lane & 15;
  tile_parity<NP, NT, false>(T, cls, tid);
  Gemm gemm;
  dgwm_d4 acc[Gemm::RT];
  gemm.load(Z1, lane, wv);
  gemm.run(T, Z1, acc, lane, wv);
  gemm.load(Z2, lane, wv);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < Gemm::RT; ++q)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = Gemm::row(q, j, lane, wv);
      if (row >= 0) T[row * LD + col] = acc[q][j] / (1.0 + tauc[col] * lam[row]);
    }
  __syncthreads();
  gemm.run(T, Z2, acc, lane, wv);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < Gemm::RT; ++q)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = Gemm::row(q, j, lane, wv);
      if (row >= 0) T[row * LD + col] = acc[q][j];
    }
  __syncthreads();
  tile_parity<NP, NT, true>(T, cls, tid);
  int id = tid;
  asm("" : "+v"(id));
#pragma unroll
  for (int i = 0; i < PL; ++i) {
    const int idx = id + i * NT, c = idx / N;
    if (c < nc) A.x[base[c] + (idx - c * N)] = T[(idx - c * N) * LD + c];
  }
}

// Lower Cholesky factor of the symmetric positive definite n x n matrix a.
void cholesky(int n, const std::vector<double>& a, std::vector<double>& c) {
  c.assign((size_t)n * n, 0.0);
  for (int j = 0; j < n; ++j) {
    double d = a[j * n + j];
    for (int k = 0; k < j; ++k) d -= c[j * n + k] * c[j * n + k];
    c[j * n + j] = std::sqrt(d);
    for (int i = j + 1; i < n; ++i) {
      double s = a[i * n + j];
      for (int k = 0; k < j; ++k) s -= c[i * n + k] * c[j * n + k];
      c[i * n + j] = s / c[j * n + j];
    }
  }
}

// Inverse of a lower triangular matrix (forward substitution per column).
void lower_inverse(int n, const std::vector<double>& c, std::vector<double>& ci) {
  ci.assign((size_t)n * n, 0.0);
  for (int col = 0; col < n; ++col) {
    for (int i = col; i < n; ++i) {
      double s = i == col ? 1.0 : 0.0;
      for (int k = col; k < i; ++k) s -= c[i * n + k] * ci[k * n + col];
      ci[i * n + col] = s / c[i * n + i];
    }
  }
}

}  // namespace

int spectral_layers(const dg_mesh& m, std::vector<int>* map, std::vector<double>* heights) {
  const dg_mesh_params& P = m.P;
  if (m.curved) return 0;
  const int lo = 0, hi = P.ny - 1;  // every layer (enriched cells share their polynomial block)
  std::vector<double> hs;
  if (map) map->assign(P.ny, 0);
  for (int j = lo; j <= hi; ++j) {
    const double t0 = 2.0 * j / P.ny - 1.0, t1 = 2.0 * (j + 1) / P.ny - 1.0;
    const double h = P.gamma > 0 ? std::tanh(P.gamma * t1) / std::tanh(P.gamma) - std::tanh(P.gamma * t0) / std::tanh(P.gamma)
                                 : t1 - t0;
    int s = -1;
    for (size_t q = 0; q < hs.size(); ++q)
      if (hs[q] == h) s = (int)q;
    if (s < 0) {
      s = (int)hs.size();
      hs.push_back(h);
    }
    if (map) (*map)[j] = s;
  }
  if (heights) *heights = hs;
  return (int)hs.size();
}

namespace {

// Reflection classes for a run-time np (host side of Parity).
struct Classes {
  int n[8], tiles[8], steps, zn;  // sizes, row tiles; steps of a tile, entries of a product
  std::vector<int> pos;
};
template <int NP>
Classes classes_of() {
  Classes c;
  for (int p = 0; p < 8; ++p) {
    c.n[p] = parity<NP>.n[p];
    c.tiles[p] = (c.n[p] + 15) / 16;
  }
  c.steps = Parity<NP>::KS;
  c.zn = Parity<NP>::ZN;
  c.pos.assign(parity<NP>.pos, parity<NP>.pos + Parity<NP>::N);
  return c;
}
bool spectral_classes(int np, Classes* c) {
  switch (np) {
    case 3: *c = classes_of<3>(); return true;
    case 4: *c = classes_of<4>(); return true;
    case 5: *c = classes_of<5>(); return true;
    case 6: *c = classes_of<6>(); return true;
  }
  return false;
}
// table entries of the two products of one layer
size_t block_entries(int np) {
  switch (np) {
    case 3: return Parity<3>::ZN;
    case 4: return Parity<4>::ZN;
    case 5: return Parity<5>::ZN;
    case 6: return Parity<6>::ZN;
  }
  return 0;
}

}  // namespace

// K^{-1}, per layer slot the blocks and eigenvalues, the int32 layer map.
static size_t table_doubles(const dg_mesh& m, int ns) {
  const size_t n = 3 * (size_t)m.np_u * m.np_u * m.np_u;
  return (size_t)m.np_u * m.np_u + (size_t)ns * (2 * block_entries(m.np_u) + n) + (m.P.ny + 1) / 2;
}

// Doubles reserved in the mesh workspace: the tables, and at least the size of
// one layer's dense n x n pair, which callers who leave the step tables out
// count on saving.  What is beyond the tables is neither formed nor written.
size_t spectral_table_doubles(const dg_mesh& m) {
  const int ns = spectral_layers(m, nullptr, nullptr);
  if (ns == 0) return 0;
  const size_t n = 3 * (size_t)m.np_u * m.np_u * m.np_u;
  return std::max(table_doubles(m, ns), 2 * n * n + n);
}

// Host: 1-D factors, whitened div-div forms, their eigendecompositions; copies
// everything into m->spec (synchronous on s).
static int build_spectral_tables(const dg_mesh* m, hipStream_t s) {
  const dg_mesh_params& P = m->P;
  const int np = m->np_u, nq = P.nq_u, np3 = np * np * np, n = 3 * np3, npt = nq * nq * nq;
  std::vector<int> map;
  std::vector<double> heights;
  const int ns = spectral_layers(*m, &map, &heights);
  if (ns == 0) return DG_OK;
  const TabLayout Lu = tab_layout(np, nq, P.nq_wn);
  std::vector<double> tu(Lu.size);
  fill_tables(np, nq, P.nq_wn, tu.data());
  const double* S = tu.data() + Lu.S;
  const double* Sd = tu.data() + Lu.Sd;
  const double* w = tu.data() + Lu.w;
  std::vector<double> K((size_t)np * np), C, Ci;
  for (int i = 0; i < np; ++i)
    for (int j = 0; j < np; ++j) {
      double v = 0.0;
      for (int q = 0; q < nq; ++q) v += w[q] * S[q * np + i] * S[q * np + j];
      K[i * np + j] = v;
    }
  Classes cl;
  if (!spectral_classes(np, &cl)) return set_error(DG_ERR_UNSUPPORTED, "projection step: degree not compiled");
  // K^{-1} in nodal coordinates
  cholesky(np, K, C);
  lower_inverse(np, C, Ci);
  const size_t nz = (size_t)cl.zn, head = (size_t)np * np, per = 2 * nz + n;
  std::vector<double> host(table_doubles(*m, ns), 0.0);
  double* Kinv = host.data();
  for (int a = 0; a < np; ++a)
    for (int i = 0; i < np; ++i) {
      double v = 0.0;  // K^{-1} = C^{-T} C^{-1}
      for (int k = 0; k < np; ++k) v += Ci[k * np + a] * Ci[k * np + i];
      Kinv[a * np + i] = v;
    }
  // orthonormal even/odd coordinates Pm v (1 / sqrt 2 (v_i +- v_{np-1-i}), the middle node as it is); the device's
  // sums and differences are these times dsc, which the tables divide out.  K in them is block diagonal, and its
  // Cholesky factor with it.
  const int ne = (np + 1) / 2, no = np / 2;
  std::vector<double> Pm((size_t)np * np, 0.0), dsc(np, 1.0);
  for (int i = 0; i < no; ++i) {
    const double q = std::sqrt(0.5);
    Pm[i * np + i] = Pm[i * np + np - 1 - i] = q;
    Pm[(ne + i) * np + i] = q;
    Pm[(ne + i) * np + np - 1 - i] = -q;
    dsc[i] = dsc[ne + i] = std::sqrt(2.0);
  }
  if (np % 2) Pm[(ne - 1) * np + no] = 1.0;
  std::vector<double> Kp((size_t)np * np, 0.0), Sp((size_t)nq * np, 0.0), Sdp((size_t)nq * np, 0.0);
  for (int a = 0; a < np; ++a)
    for (int b = 0; b < np; ++b) {
      if ((a < ne) != (b < ne)) continue;
      double v = 0.0;
      for (int i = 0; i < np; ++i)
        for (int j = 0; j < np; ++j) v += Pm[a * np + i] * K[i * np + j] * Pm[b * np + j];
      Kp[a * np + b] = v;
    }
  for (int q = 0; q < nq; ++q)
    for (int a = 0; a < np; ++a)
      for (int i = 0; i < np; ++i) {
        Sp[q * np + a] += S[q * np + i] * Pm[a * np + i];
        Sdp[q * np + a] += Sd[q * np + i] * Pm[a * np + i];
      }
  cholesky(np, Kp, C);
  lower_inverse(np, C, Ci);
  // whitened 1-D tables: St = Sp C^{-T}, Sdt = Sdp C^{-T}
  std::vector<double> St((size_t)nq * np, 0.0), Sdt((size_t)nq * np, 0.0);
  for (int q = 0; q < nq; ++q)
    for (int a = 0; a < np; ++a)
      for (int i = 0; i < np; ++i) {
        St[q * np + a] += Sp[q * np + i] * Ci[a * np + i];
        Sdt[q * np + a] += Sdp[q * np + i] * Ci[a * np + i];
      }
  std::vector<int> sweeps(ns, 0);
  auto work = [&](int slot) {
    const double h[3] = {m->hx, heights[slot], m->hz};
    // G[q][I] = sqrt(w_q) div of whitened basis function I at point q
    std::vector<double> G((size_t)npt * n);
    for (int qz = 0; qz < nq; ++qz)
      for (int qy = 0; qy < nq; ++qy)
        for (int qx = 0; qx < nq; ++qx) {
          const int q = qx + nq * (qy + nq * qz);
          const double sw = std::sqrt(w[qx] * w[qy] * w[qz]);
          for (int iz = 0; iz < np; ++iz)
            for (int iy = 0; iy < np; ++iy)
              for (int ix = 0; ix < np; ++ix) {
                const int B = ix + np * (iy + np * iz);
                const double sx = St[qx * np + ix], sy = St[qy * np + iy], sz = St[qz * np + iz];
                G[(size_t)q * n + B] = sw * Sdt[qx * np + ix] * sy * sz / h[0];
                G[(size_t)q * n + np3 + B] = sw * sx * Sdt[qy * np + iy] * sz / h[1];
                G[(size_t)q * n + 2 * np3 + B] = sw * sx * sy * Sdt[qz * np + iz] / h[2];
              }
        }
    std::vector<double> Bm, lam, vt, v((size_t)n), w((size_t)n);
    auto along = [&](const std::vector<double>& M, bool transpose, std::vector<double>& x) {
      for (int dir = 0; dir < 3; ++dir) {
        const int sd = dir == 0 ? 1 : (dir == 1 ? np : np * np);
        for (int c = 0; c < 3; ++c)
          for (int l = 0; l < np * np; ++l) {
            const int base = c * np3 + (dir == 0 ? l * np : (dir == 1 ? (l % np) + (l / np) * np * np : l));
            double in[8], out[8];
            for (int i = 0; i < np; ++i) in[i] = x[base + i * sd];
            for (int a = 0; a < np; ++a) {
              double t = 0.0;
              for (int i = 0; i < np; ++i) t += (transpose ? M[i * np + a] : M[a * np + i]) * in[i];
              out[a] = t;
            }
            for (int a = 0; a < np; ++a) x[base + a * sd] = out[a];
          }
      }
    };
    // scale of a 3-D coordinate (product over its directions)
    auto scale = [&](int at) {
      const int B = at % np3;
      return dsc[B % np] * dsc[(B / np) % np] * dsc[B / (np * np)];
    };
    // per class: first product (L Z)^T, entry (k, r) = (L z_r)[k]; second L^{-T} Z, entry (k, r) = (L^{-T} z_k)[r]
    // (z_r eigenvector r; L and L^{-T} as 1-D factors along each direction of each component)
    double* A1 = host.data() + head + slot * per;
    double* A2 = A1 + nz;
    double* L = A2 + nz;
    for (int p = 0, o = 0, t = 0; p < 8; o += cl.n[p], t += cl.tiles[p], ++p) {
      const int np_ = cl.n[p];
      const int* at = cl.pos.data() + o;
      Bm.assign((size_t)np_ * np_, 0.0);
      for (int q = 0; q < npt; ++q) {
        const double* gq = &G[(size_t)q * n];
        for (int I = 0; I < np_; ++I) {
          const double gi = gq[at[I]];
          double* row = &Bm[(size_t)I * np_];
          for (int J = 0; J < np_; ++J) row[J] += gi * gq[at[J]];
        }
      }
      const int sw = sym_eig_jacobi(np_, Bm, lam, vt);
      sweeps[slot] = sw < 0 ? sw : (sweeps[slot] < 0 ? sweeps[slot] : sw);
      // entry (k, r) of the class: tile r / 16, step k / 4, lane (k % 4, r % 16)
      auto entry = [&](int k, int r) {
        return ((size_t)(t + r / 16) * cl.steps + k / 4) * 64 + (k % 4) * 16 + r % 16;
      };
      for (int r = 0; r < np_; ++r) {
        std::fill(v.begin(), v.end(), 0.0);
        for (int k = 0; k < np_; ++k) v[at[k]] = vt[(size_t)r * np_ + k];
        w = v;
        along(C, false, v);   // L z_r
        along(Ci, true, w);   // L^{-T} z_r
        for (int k = 0; k < np_; ++k) {
          const double is = 1.0 / scale(at[k]);
          A1[entry(k, r)] = v[at[k]] * is;
          A2[entry(r, k)] = w[at[k]] * is;
        }
        L[o + r] = std::max(lam[r], 0.0);  // positive semidefinite form
      }
    }
  };
  // slots t, t + nth, ... per worker; an allocation failure marks the slot (-2) instead of escaping the thread,
  // and workers that cannot be started run on this thread
  auto run = [&](int t, int nth) {
    for (int slot = t; slot < ns; slot += nth) {
      try {
        work(slot);
      } catch (...) {
        sweeps[slot] = -2;
      }
    }
  };
  const int nth = std::max(1, std::min<int>(ns, std::min(16u, std::max(1u, std::thread::hardware_concurrency()))));
  std::vector<std::thread> pool;
  int started = 0;
  try {
    pool.reserve(nth);
    for (; started < nth; ++started) pool.emplace_back(run, started, nth);
  } catch (...) {
  }
  for (int t = started; t < nth; ++t) run(t, nth);
  for (auto& th : pool) th.join();
  for (int slot = 0; slot < ns; ++slot) {
    if (sweeps[slot] == -2) return set_error(DG_ERR_ARG, "projection step: host memory for the layer tables refused");
    if (sweeps[slot] < 0) return set_error(DG_ERR_NOT_CONVERGED, "projection step: eigendecomposition did not converge");
  }
  int32_t* mp = reinterpret_cast<int32_t*>(host.data() + head + ns * per);
  for (int j = 0; j < P.ny; ++j) mp[j] = map[j];
  int rc = check_hip(hipMemcpyAsync(m->spec, host.data(), sizeof(double) * host.size(), hipMemcpyHostToDevice, s),
                     "copy");
  if (!rc) rc = check_hip(hipStreamSynchronize(s), "projection step tables");
  if (!rc) m->spec_ok = 1;
  return rc;
}

int ensure_spectral_tables(const dg_mesh* m, hipStream_t s) {
  if (m->spec_ok) return DG_OK;
  try {
    return build_spectral_tables(m, s);
  } catch (...) {  // host allocations: no exception crosses the C ABI
    return set_error(DG_ERR_ARG, "projection step: host memory for the layer tables refused");
  }
}

void spectral_pointers(const dg_mesh* m, const double** mats, const double** slots, const int32_t** map) {
  const int np = m->np_u;
  const size_t n = 3 * (size_t)np * np * np;
  const int ns = spectral_layers(*m, nullptr, nullptr);
  *mats = m->spec;
  *slots = m->spec + np * np;
  *map = reinterpret_cast<const int32_t*>(m->spec + np * np + (size_t)ns * (2 * block_entries(np) + n));
}

int launch_spectral_step(const dg_mesh* m, const double* tau_d, const double* u_hat, const double* g, double scale,
                         double* x, hipStream_t s) {
  const dg_mesh_params& P = m->P;
  const int lo = (P.fully_periodic || m->lower_slot < 0) ? 0 : 1;
  const int hi = (P.fully_periodic || m->upper_slot < 0) ? P.ny - 1 : P.ny - 2;
  const int nl = hi - lo + 1;
  if (nl <= 0) return DG_OK;
  const int np = m->np_u;
  SpecArgs A;
  A.nx = P.nx;
  A.ny = P.ny;
  A.layer_lo = lo;
  A.ncol = (int64_t)P.nx * P.nz;
  A.hx = m->hx;
  A.hz = m->hz;
  A.hy = m->hy;
  spectral_pointers(m, &A.mats, &A.slots, &A.map);
  A.tau_d = tau_d;
  A.u_hat = u_hat;
  A.g = g;
  A.scale = scale;
  A.x = x;
#define X(p)                                                                                                \
  if (np == p) {                                                                                            \
    const int64_t tiles = (A.ncol + kTileCols - 1) / kTileCols;                                             \
    const int64_t nb = tiles * nl;                                                                          \
    if (nb > INT32_MAX / 2) return set_error(DG_ERR_ARG, "projection step: mesh too large");                \
    A.tiles = (int)tiles;                                                                                   \
    A.nblocks = (int)nb;                                                                                    \
    const int grid = ((A.nblocks + 7) / 8) * 8;                                                             \
    hipLaunchKernelGGL(spectral_step_kernel<p>, dim3((unsigned)grid), dim3(tile_threads(p)), 0, s, A);      \
    return check_hip(hipGetLastError(), "projection step kernel launch");                                   \
  }
  X(3) X(4) X(5) X(6)
#undef X
  return set_error(DG_ERR_UNSUPPORTED, "projection step: degree not compiled");
}

}  // namespace dgwm
