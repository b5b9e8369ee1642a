// The coarse end of the multigrid V-cycle in one workgroup (preconditioner of
// the Poisson solve): from the first level whose vectors fit in one CU's LDS
// down to the coarsest and back.
//
// On these levels a launch costs more than its work: a smoothing step of 16
// cells is 0.1 MFLOP and 4 us of launch, load and drain, and a cycle over two
// such levels with its transfers and coarsest solve takes 17 of them in a row.
// Here every level's right-hand side, iterate and inverse diagonal stay in
// LDS, the iterate of a level also in the registers of the thread that owns
// its x pencil, and a step is four barriers.  One workgroup holds one mesh, so
// a batch of meshes is one launch.  The arithmetic of an entry is that of the
// separate kernels (kern_poisson.hip, kern_mg.hip): operator by 1-D operators
// in z, y, x sweeps, Chebyshev recurrence, transfers direction by direction,
// dense inverse on the coarsest level.
//
// Used from the first level whose x pencils fit 1,024 threads, whose vectors
// fit the LDS below and whose coarsest level, if solved densely, has at most
// 256 unknowns (a CU alone reads the n^2 entries of a larger one slower than
// the launches cost).  16 x 8 x 8 cells, k = 3: the levels of 16 and 2 cells and
// the coarsest solve 26 us, 80 us as 17 launches; 1.2 us a step, the latency of
// its LDS passes, and 11 us around them.  A solve 2.9 -> 2.5 ms; eight solves
// of 16 x 16 x 16 cells, k = 2, 10.0 -> 8.3 ms (single runs of either spread by 5%).
#include <algorithm>
#include <vector>

#include "batch.h"

namespace dgwm {

namespace {

constexpr int kTailThreads = 1024;  // most x pencils of the first level
constexpr int kTailSteps = 64;      // most smoothing steps on a level
constexpr int kTailDense = 256;     // largest dense coarsest level: one CU reads its n^2 entries

// LDS entries: 80 KB in FP32, 144 KB in FP64
template <typename T>
constexpr int tail_cap() {
  return sizeof(T) == 4 ? 20480 : 18432;
}

// LDS layout of one cell's scratch (PoiLds of kern_poisson.hip)
template <int NP>
struct TailLds {
  static constexpr int SJ = NP, SK = NP * NP + (NP == 4 ? 1 : 0), SC = NP == 4 ? 76 : NP * NP * NP;
  static __device__ __forceinline__ int base(int D, int a, int b) {
    return D == 0 ? SJ * a + SK * b : (D == 1 ? a + SK * b : a + SJ * b);
  }
  static __device__ __forceinline__ constexpr int stride(int D) { return D == 0 ? 1 : (D == 1 ? SJ : SK); }
};

// Place of the image's entries behind its segment.
template <typename T>
__host__ __device__ __forceinline__ T* tail_entries(void* img) {
  return reinterpret_cast<T*>(static_cast<char*>(img) + kTailHead);
}

// The constant part of the LDS layout, formed once per solve: transfer table
// of halved directions, per level the Chebyshev coefficients (c1, c2) of every
// step, heights and their reciprocals, y transfer table and inverse diagonal,
// then the dense inverse where it fits.
template <typename T, int NP>
__global__ __launch_bounds__(256) void mg_tail_image_kernel(const TailArr<T> A) {
  constexpr int NP2 = NP * NP;
  const TailSeg<T>& S = A.s[blockIdx.x];
  const int tid = threadIdx.x, NT = blockDim.x;
  T* const img = tail_entries<T>(S.img);
  // the segment itself in front of the image: the cycle takes two pointers and this block
  for (int t = tid; t < (int)(sizeof(TailSeg<T>) / 4); t += NT)
    reinterpret_cast<uint32_t*>(S.img)[t] = reinterpret_cast<const uint32_t*>(&S)[t];
  for (int t = tid; t < 2 * NP2; t += NT) {  // [child][l][i]: N_i((child + x_l) / 2)
    const int i = t % NP, l = (t / NP) % NP, ch = t / NP2;
    img[t] = T(lobatto_basis<NP>(i, 0.5 * (ch + ct::lobatto<NP>.x[l])));
  }
  if (tid < S.nlev) {
    const TailLevel<T>& L = S.lv[tid];
    T* co = img + L.oco;
    const double sigma = L.theta / L.delta;
    double rho = 1.0 / sigma;
    for (int k = 0; k < L.deg; ++k) {
      const double rn = 1.0 / (2.0 * sigma - rho);
      co[2 * k] = k == 0 ? T(0) : T(rn * rho);
      co[2 * k + 1] = k == 0 ? T(1.0 / L.theta) : T(2.0 * rn / L.delta);
      if (k > 0) rho = rn;
    }
  }
  for (int j = 0; j < S.nlev; ++j) {
    const TailLevel<T>& L = S.lv[j];
    for (int i = tid; i < 2 * L.ny; i += NT) img[L.ohy + i] = T(L.hy[i]);
    for (int i = tid; i < L.n; i += NT) img[L.od + i] = L.dinv[i];
    if (j + 1 < S.nlev && L.cy)
      for (int t = tid; t < S.lv[j + 1].ny * 2 * NP2; t += NT) {
        const int i = t % NP, l = (t / NP) % NP, ch = (t / NP2) % 2, Y = t / (2 * NP2);
        const double h0 = L.hy[2 * Y], r = h0 / (h0 + L.hy[2 * Y + 1]), xl = ct::lobatto<NP>.x[l];
        img[L.opy + t] = T(lobatto_basis<NP>(i, ch == 0 ? r * xl : r + (1.0 - r) * xl));
      }
  }
  if (S.odense >= 0)
    for (int i = tid; i < S.ndense * S.ndense; i += NT) img[S.odense + i] = S.B[i];
}

// c / n for c < 2^8 cells and inv = ceil(2^16 / n)
__device__ __forceinline__ int tail_div(int c, int inv) { return (c * inv) >> 16; }

// A cell's code is executed a few times at most, so that its instructions come
// from memory: one loop over the visits of the levels keeps a single copy of
// smoothing and transfers.
//
// G = 3 threads share a pencil index where they fit in a workgroup: thread
// group g takes the direction-g part of the operator and its share of the
// sweeps, group 0 the iterate.  G = 1: every thread does all three.
template <typename T, int NP, int G>
__global__ __launch_bounds__(kTailThreads) void mg_tail_kernel(const TailRuns<T> A) {
  constexpr int NP2 = NP * NP, NP3 = NP2 * NP;
  using LD = TailLds<NP>;
  const T* const rhs = A.r[blockIdx.x].b;
  T* const sol = A.r[blockIdx.x].x;
  const auto& S = *(const __attribute__((address_space(4))) TailSeg<T>*)(uintptr_t)A.r[blockIdx.x].img;
  __shared__ __align__(16) T buf[tail_cap<T>()];
  const int tid = threadIdx.x, NT = blockDim.x;
  const int nl = S.nlev;
  T* const sP = buf + S.oscr;
  T* const sX = sP + S.nscr;
  T* const sY = sX + S.nscr;
  T* const sZ = sY + S.nscr;
  const T* const half = buf;
  {
    // the image, eight 16-byte loads a thread in flight, and the right-hand side
    typedef T V __attribute__((ext_vector_type(16 / sizeof(T))));
    const V* src = reinterpret_cast<const V*>(tail_entries<const T>(A.r[blockIdx.x].img));
    V* dst = reinterpret_cast<V*>(buf);
    const int nv = S.nimg / (int)(16 / sizeof(T)), n0 = S.lv[0].n;  // (nimg is a multiple of 4)
    T* b0 = buf + S.lv[0].ob;
    T vb[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) vb[k] = rhs[tid + k * NT < n0 ? tid + k * NT : 0];
    for (int i0 = 0; i0 < nv; i0 += 8 * NT) {
      V v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int i = i0 + tid + k * NT;
        v[k] = src[i < nv ? i : 0];
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int i = i0 + tid + k * NT;
        if (i < nv) dst[i] = v[k];
      }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (tid + k * NT < n0) b0[tid + k * NT] = vb[k];
    for (int i = tid + 2 * NT; i < n0; i += NT) b0[i] = rhs[i];
  }
  __syncthreads();

  constexpr PoiOps O = poi_ops(NP);
  const ConstTab<T> ops = (ConstTab<T>)(uintptr_t)(S.tab + (sizeof(T) == 8 ? 0 : O.f32));
  const ConstTab<T> Mm = ops + O.M, Km = ops + O.K, nd0 = ops + O.nd0, nd1 = ops + O.nd1;
  const T pen = S.pen;
  constexpr int ND = G == 3 ? 1 : 3;
  const int grp = G == 3 ? __builtin_amdgcn_readfirstlane(tid / S.p0) : 0;  // (p0 is a multiple of 64)
  const int pt = tid - grp * S.p0;
  const int c = pt / NP2, t2 = pt - c * NP2, pa = t2 % NP, pb = t2 / NP;

  // smoothing on level j: steps k0 .. deg - 1 from the iterate px (zero start: k0 = 1 and px the first iterate);
  // leaves the last iterate in px and, with `resid`, b - A px in the place of sP (plain layout)
  T px[NP];
  auto smooth = [&](const auto& L, bool zero, bool resid) __attribute__((always_inline)) {
    const int cells = L.nx * L.ny * L.nz;
    const bool in = grp < 3 && c < cells, own = in && grp == 0;
    const T* co = buf + L.oco;
    const T* hy = buf + L.ohy;
    T eb[NP], ei[NP], pm[NP];
    // per direction of this thread: pencil, its neighbours' first entries, walls, 1 / h, areas
    int bD[ND], sD[ND], nb[ND][2];
    bool wall[ND][2];
    T rd[ND], area[ND], rn[ND][2];
    if (in) {
      const int eyz = tail_div(c, L.ix), ex = c - eyz * L.nx, ez = tail_div(eyz, L.iy), ey = eyz - ez * L.ny;
      const T h0 = T(L.hx), h1 = hy[ey], h2 = T(L.hz);
#pragma unroll
      for (int d = 0; d < ND; ++d) {
        const int D = G == 3 ? grp : d;
        const int i = D == 0 ? ex : (D == 1 ? ey : ez), n = D == 0 ? L.nx : (D == 1 ? L.ny : L.nz);
        const int st = D == 0 ? 1 : (D == 1 ? L.nx : L.nx * L.ny);
        const int lo = i == 0 ? c + (n - 1) * st : c - st, hi = i == n - 1 ? c - (n - 1) * st : c + st;
        const bool walls = D == 1 && !S.periodic;
        wall[d][0] = walls && i == 0;
        wall[d][1] = walls && i == n - 1;
        bD[d] = LD::base(D, pa, pb);
        sD[d] = D == 0 ? 1 : (D == 1 ? LD::SJ : LD::SK);
        nb[d][0] = lo * LD::SC + bD[d];
        nb[d][1] = hi * LD::SC + bD[d];
        rd[d] = D == 0 ? T(1.0 / L.hx) : (D == 1 ? hy[L.ny + ey] : T(1.0 / L.hz));
        area[d] = D == 0 ? h1 * h2 : (D == 1 ? h0 * h2 : h0 * h1);
        rn[d][0] = D == 1 ? hy[L.ny + (ey == 0 ? L.ny - 1 : ey - 1)] : rd[d];
        rn[d][1] = D == 1 ? hy[L.ny + (ey + 1 == L.ny ? 0 : ey + 1)] : rd[d];
      }
    }
    if (own) {
      const T* vb = buf + L.ob + c * NP3 + t2 * NP;
      const T* vd = buf + L.od + c * NP3 + t2 * NP;
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        eb[l] = vb[l];
        ei[l] = vd[l];
        pm[l] = T(0);
        if (zero) px[l] = co[1] * ei[l] * eb[l];
      }
    }
    const int last = L.deg + (resid ? 1 : 0);
    for (int k = zero ? 1 : 0; k < last; ++k) {
      if (own)
#pragma unroll
        for (int l = 0; l < NP; ++l) sP[c * LD::SC + LD::base(0, pa, pb) + l] = px[l];
      __syncthreads();
      // Q_D on the thread's pencils
      if (in) {
#pragma unroll
        for (int d = 0; d < ND; ++d) {
          const int s = G == 3 ? sD[d] : LD::stride(d);
          T x[NP];
#pragma unroll
          for (int l = 0; l < NP; ++l) x[l] = G == 1 && d == 0 ? px[l] : sP[c * LD::SC + bD[d] + l * s];
          T J[2], Gf[2];
#pragma unroll
          for (int F = 0; F < 2; ++F) {
            const T* pn = sP + nb[d][F];
            T dn = 0, dx = 0, vn = 0;
#pragma unroll
            for (int l = 0; l < NP; ++l) {
              const T q = pn[l * s];
              dn += (F ? nd0 : nd1)[l] * q;
              dx += (F ? nd1 : nd0)[l] * x[l];
              if (l == (F ? 0 : NP - 1)) vn = q;
            }
            const T tau = pen * (rd[d] > rn[d][F] ? rd[d] : rn[d][F]);
            const T jump = x[F ? NP - 1 : 0] - vn, avg = T(0.5) * (dx * rd[d] + dn * rn[d][F]);
            J[F] = wall[d][F] ? T(0) : jump;
            Gf[F] = wall[d][F] ? T(0) : (F ? tau * jump - avg : tau * jump + avg);
          }
          const T cv = area[d] * rd[d];
          const int D = G == 3 ? grp : d;
          T* dst = (D == 0 ? sX : (D == 1 ? sY : sZ)) + c * LD::SC + bD[d];
#pragma unroll
          for (int l = 0; l < NP; ++l) {
            T kx = 0;
#pragma unroll
            for (int m = 0; m < NP; ++m) kx += Km[l * NP + m] * x[m];
            T q = cv * (kx + T(0.5) * nd0[l] * J[0] - T(0.5) * nd1[l] * J[1]);
            if (l == 0) q += area[d] * Gf[0];
            if (l == NP - 1) q += area[d] * Gf[1];
            dst[l * s] = q;
          }
        }
      }
      __syncthreads();
      // z sweeps: X <- Mz Qx (group 0), Y <- Mz Qy (group 1)
#pragma unroll
      for (int d = 0; d < (G == 3 ? 1 : 2); ++d)
        if (in && grp < 2) {
          T* y = ((G == 3 ? grp : d) ? sY : sX) + c * LD::SC + LD::base(2, pa, pb);
          T u[NP];
#pragma unroll
          for (int l = 0; l < NP; ++l) u[l] = y[l * LD::SK];
#pragma unroll
          for (int l = 0; l < NP; ++l) {
            T v = 0;
#pragma unroll
            for (int m = 0; m < NP; ++m) v += Mm[l * NP + m] * u[m];
            y[l * LD::SK] = v;
          }
        }
      __syncthreads();
      // y sweeps: X <- My X (group 0), Z <- My Qz + Y (group 1)
#pragma unroll
      for (int d = 0; d < (G == 3 ? 1 : 2); ++d)
        if (in && grp < 2) {
          const bool z = (G == 3 ? grp : d) != 0;
          T* y = (z ? sZ : sX) + c * LD::SC + LD::base(1, pa, pb);
          const T* a = sY + c * LD::SC + LD::base(1, pa, pb);
          T u[NP], v[NP];
#pragma unroll
          for (int l = 0; l < NP; ++l) {
            u[l] = y[l * LD::SJ];
            const T al = a[l * LD::SJ];
            v[l] = z ? al : T(0);
          }
#pragma unroll
          for (int l = 0; l < NP; ++l) {
#pragma unroll
            for (int m = 0; m < NP; ++m) v[l] += Mm[l * NP + m] * u[m];
            y[l * LD::SJ] = v[l];
          }
        }
      __syncthreads();
      if (own) {  // x sweep: A p = Mx Z + X on the thread's x pencil, then the step
        const T* z = sZ + c * LD::SC + LD::base(0, pa, pb);
        const T* x = sX + c * LD::SC + LD::base(0, pa, pb);
        T u[NP];
#pragma unroll
        for (int l = 0; l < NP; ++l) u[l] = z[l];
        T r[NP];
#pragma unroll
        for (int l = 0; l < NP; ++l) {
          T v = x[l];
#pragma unroll
          for (int m = 0; m < NP; ++m) v += Mm[l * NP + m] * u[m];
          r[l] = eb[l] - v;
        }
        if (k == L.deg) {
#pragma unroll
          for (int l = 0; l < NP; ++l) sP[c * NP3 + t2 * NP + l] = r[l];
        } else {
          const T c1 = co[2 * k], c2 = co[2 * k + 1];  // (c1 = 0 in the first step)
#pragma unroll
          for (int l = 0; l < NP; ++l) {
            const T v = c2 * ei[l] * r[l] + c1 * (px[l] - pm[l]);
            pm[l] = px[l];
            px[l] += v;
          }
        }
      }
    }
    __syncthreads();
  };

  for (int visit = 0; visit < 2 * nl - 1; ++visit) {
    const bool up = visit >= nl;
    const int j = up ? 2 * nl - 2 - visit : visit;
    const bool last = j == nl - 1;
    const auto& L = S.lv[j];
    const auto& C = S.lv[last ? j : j + 1];  // the next coarser level
    T* const vb = buf + L.ob;
    T* const vx = vb + L.n;
    const int ncx = C.nx, ncxy = C.nx * C.ny;
    const T* const py = buf + L.opy;
    if (last && S.ndense > 0) {
      // x = B b, B symmetric: thread (i, q) adds the entries m = q, q + nq, ... of column i (nq by the mesh's own
      // threads, so that the sums do not depend on the launch)
      const int n = S.ndense, nq = S.threads / n, q = tid / n, i = tid - q * n;
      T v = 0;
      if (q < nq) {
        const T* B = S.odense >= 0 ? buf + S.odense : S.B;
#pragma unroll 8
        for (int m = q; m < n; m += nq) v += B[m * n + i] * vb[m];
        sX[q * n + i] = v;
      }
      __syncthreads();
      if (tid < n) {
        T x = 0;
        for (int k = 0; k < nq; ++k) x += sX[k * n + tid];
        vx[tid] = x;
      }
      __syncthreads();
      continue;
    }
    if (up) {  // x += P x_{j+1}: along z into sX, y into sY, x
      const T* cx = buf + C.ob + C.n;
      for (int t = tid; t < ncxy * L.nz * NP3; t += NT) {
        const int node = t % NP3, cell = t / NP3, fz = tail_div(cell, C.ixy), XY = cell - fz * ncxy;
        const int ji = node % NP2, n = node / NP2;
        T v = 0;
        if (L.cz) {
#pragma unroll
          for (int m = 0; m < NP; ++m)
            v += half[((fz & 1) * NP + n) * NP + m] * cx[(XY + ncxy * (fz >> 1)) * NP3 + m * NP2 + ji];
        } else {
          v = cx[t];
        }
        sX[t] = v;
      }
      __syncthreads();
      for (int t = tid; t < ncx * L.ny * L.nz * NP3; t += NT) {
        const int node = t % NP3, cell = t / NP3, yz = tail_div(cell, C.ix), X = cell - yz * ncx;
        const int fz = tail_div(yz, L.iy), fy = yz - fz * L.ny;
        const int i = node % NP, m = (node / NP) % NP, n = node / NP2;
        T v = 0;
        if (L.cy) {
#pragma unroll
          for (int q = 0; q < NP; ++q)
            v += py[(fy >> 1) * 2 * NP2 + ((fy & 1) * NP + m) * NP + q] *
                 sX[(X + ncx * ((fy >> 1) + C.ny * fz)) * NP3 + n * NP2 + q * NP + i];
        } else {
          v = sX[t];
        }
        sY[t] = v;
      }
      __syncthreads();
      for (int t = tid; t < L.n; t += NT) {
        const int node = t % NP3, cell = t / NP3, yz = tail_div(cell, L.ix), fx = cell - yz * L.nx;
        const int l = node % NP, nm = node / NP;
        T v = 0;
        if (L.cx) {
#pragma unroll
          for (int i = 0; i < NP; ++i)
            v += half[((fx & 1) * NP + l) * NP + i] * sY[((fx >> 1) + ncx * yz) * NP3 + nm * NP + i];
        } else {
          v = sY[t];
        }
        vx[t] += v;
      }
      __syncthreads();
    }
    const bool live = grp == 0 && c < L.nx * L.ny * L.nz;
    if (up && live)
#pragma unroll
      for (int l = 0; l < NP; ++l) px[l] = vx[c * NP3 + t2 * NP + l];
    smooth(L, !up, !up && !last);
    if (live) {
      T* out = up && j == 0 ? sol : vx;
#pragma unroll
      for (int l = 0; l < NP; ++l) out[c * NP3 + t2 * NP + l] = px[l];
    }
    if (!up && !last) {  // b_{j+1} = P^T r, r in sP: along x into sX, y into sY, z
      for (int t = tid; t < ncx * L.ny * L.nz * NP3; t += NT) {
        const int node = t % NP3, cell = t / NP3, yz = tail_div(cell, C.ix), X = cell - yz * ncx;
        const int i = node % NP, kj = node / NP;
        T v = 0;
        if (L.cx) {
#pragma unroll
          for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int l = 0; l < NP; ++l)
              v += half[(a * NP + l) * NP + i] * sP[(2 * X + a + L.nx * yz) * NP3 + kj * NP + l];
        } else {
          v = sP[t];
        }
        sX[t] = v;
      }
      __syncthreads();
      for (int t = tid; t < ncxy * L.nz * NP3; t += NT) {
        const int node = t % NP3, cell = t / NP3, fz = tail_div(cell, C.ixy), XY = cell - fz * ncxy;
        const int Y = tail_div(XY, C.ix), X = XY - Y * ncx;
        const int i = node % NP, jc = (node / NP) % NP, k = node / NP2;
        T v = 0;
        if (L.cy) {
#pragma unroll
          for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int m = 0; m < NP; ++m)
              v += py[Y * 2 * NP2 + (b * NP + m) * NP + jc] *
                   sX[(X + ncx * (2 * Y + b + L.ny * fz)) * NP3 + k * NP2 + m * NP + i];
        } else {
          v = sX[t];
        }
        sY[t] = v;
      }
      __syncthreads();
      T* const cb = buf + C.ob;
      for (int t = tid; t < C.n; t += NT) {
        const int node = t % NP3, cell = t / NP3, Z = tail_div(cell, C.ixy), XY = cell - Z * ncxy;
        const int ji = node % NP2, kc = node / NP2;
        T v = 0;
        if (L.cz) {
#pragma unroll
          for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int m = 0; m < NP; ++m)
              v += half[(b * NP + m) * NP + kc] * sY[(XY + ncxy * (2 * Z + b)) * NP3 + m * NP2 + ji];
        } else {
          v = sY[t];
        }
        cb[t] = v;
      }
    }
    __syncthreads();
  }
}

}  // namespace

#define DG_TAIL_NP(X) X(2) X(3) X(4) X(5) X(6)

// The levels [l, nlev) of mesh m as a tail segment; false if they do not fit.
template <typename T>
bool mg_tail_segment(const dg_mesh* m, int l, int nlev, int deg0, int degc, double range, size_t img_bytes,
                     TailSeg<T>* S) {
  if (img_bytes < kTailHead) return false;
  const int64_t cap = std::min<int64_t>(kTailImage, (int64_t)((img_bytes - kTailHead) / sizeof(T)) / 4 * 4);
  const int np = m->np_p, np2 = np * np, np3 = np2 * np, nl = nlev - l;
  if (nl < 2 || nl > kTailLevels || deg0 < 1 || degc < 1) return false;
  const int sc = np == 4 ? 76 : np3;
  const int64_t cells0 = l > 0 ? m->mg[l].ncell : m->ncell;
  if (cells0 * np2 > kTailThreads) return false;
  *S = TailSeg<T>{};
  S->nlev = nl;
  S->periodic = m->P.fully_periodic ? 1 : 0;
  int64_t off = 2 * np2;
  for (int j = 0; j < nl; ++j) {
    const MeshDev M = poisson_meshdev(m, l + j);
    TailLevel<T>& L = S->lv[j];
    L.nx = M.nx;
    L.ny = M.ny;
    L.nz = M.nz;
    L.n = (M.nx * M.ny * M.nz * np3);
    L.ix = (65536 + M.nx - 1) / M.nx;
    L.iy = (65536 + M.ny - 1) / M.ny;
    L.ixy = (65536 + M.nx * M.ny - 1) / (M.nx * M.ny);
    L.hx = M.hx;
    L.hz = M.hz;
    L.hy = M.hy;
    const bool last = j == nl - 1;
    const double lam = m->mg[l + j].lam;
    const double lmin = last ? lam / 200.0 : lam / range, lmax = 1.1 * lam;
    L.theta = 0.5 * (lmax + lmin);
    L.delta = 0.5 * (lmax - lmin);
    const int64_t deg = last ? 4 * (int64_t)deg0 : (l + j == 0 ? deg0 : degc);
    const bool dense = last && m->coarse_inv;
    if (!dense && deg > kTailSteps) return false;
    L.deg = (dense ? 0 : deg);
    L.oco = off;
    off += 2 * L.deg;
    L.ohy = off;
    off += 2 * M.ny;
    L.opy = off;
    if (!last) {
      const MgLevel& C = m->mg[l + j + 1];
      L.cx = C.cx;
      L.cy = C.cy;
      L.cz = C.cz;
      if (C.cy) off += C.ny * 2 * np2;
    }
    L.od = off;
    off += L.n;
    if (off > cap) return false;
  }
  S->odense = -1;
  if (m->coarse_inv) {
    const int64_t n = m->mg[nlev - 1].n;
    if (n > kTailDense) return false;
    S->ndense = n;
    S->B = reinterpret_cast<const T*>(sizeof(T) == 8 ? (const void*)m->coarse_inv : (const void*)m->coarse_inv32);
    if (off + n * n <= cap) {
      S->odense = (int)off;
      off += n * n;
    }
  }
  off = (off + 3) / 4 * 4;
  S->nimg = (int)off;
  for (int j = 0; j < nl; ++j) {
    S->lv[j].ob = off;
    off += 2 * S->lv[j].n;
    if (off > tail_cap<T>()) return false;
  }
  S->oscr = off;
  S->nscr = std::max<int64_t>({cells0 * sc, S->lv[0].n, kTailThreads});
  off += 4 * S->nscr;
  if (off > tail_cap<T>()) return false;
  const MeshDev M = poisson_meshdev(m, l);
  S->tab = M.tab + M.ops_off;
  S->pen = T(M.pen);
  S->p0 = ((S->lv[0].n / np + 63) / 64 * 64);
  S->groups = 3 * S->p0 <= kTailThreads ? 3 : 1;
  S->threads = std::max(S->groups * S->p0, (S->ndense + 63) / 64 * 64);
  return true;
}

template bool mg_tail_segment<double>(const dg_mesh*, int, int, int, int, double, size_t, TailSeg<double>*);
template bool mg_tail_segment<float>(const dg_mesh*, int, int, int, int, double, size_t, TailSeg<float>*);

// One workgroup per segment.
template <typename T>
int launch_mg_tail_image(int np, const TailSeg<T>* segs, int nseg, hipStream_t s) {
  for (int c0 = 0; c0 < nseg; c0 += kTailSegs) {
    TailArr<T> a{};
    const int n = std::min(kTailSegs, nseg - c0);
    for (int i = 0; i < n; ++i) a.s[i] = segs[c0 + i];
    bool done = false;
#define X(q)                                                                                     \
    if (np == q) {                                                                               \
      done = true;                                                                               \
      hipLaunchKernelGGL((mg_tail_image_kernel<T, q>), dim3((unsigned)n), dim3(256), 0, s, a);   \
    }
    DG_TAIL_NP(X)
#undef X
    if (!done) return set_error(DG_ERR_UNSUPPORTED, "multigrid degree not compiled");
    if (int rc = check_hip(hipGetLastError(), "coarse cycle tables launch")) return rc;
  }
  return DG_OK;
}
template <typename T>
int launch_mg_tail(int np, const TailRun<T>* runs, int nrun, hipStream_t s) {
  for (int groups = 1; groups <= 3; groups += 2)
    for (int c0 = 0; c0 < nrun;) {
      TailRuns<T> a{};
      int n = 0, threads = 64;
      for (; c0 < nrun && n < kTailRuns; ++c0)
        if (runs[c0].groups == groups) {
          a.r[n++] = runs[c0];
          threads = std::max(threads, runs[c0].threads);
        }
      if (n == 0) break;
      bool done = false;
#define X(q)                                                                                                  \
      if (np == q) {                                                                                          \
        done = true;                                                                                          \
        if (groups == 3)                                                                                      \
          hipLaunchKernelGGL((mg_tail_kernel<T, q, 3>), dim3((unsigned)n), dim3((unsigned)threads), 0, s, a); \
        else                                                                                                  \
          hipLaunchKernelGGL((mg_tail_kernel<T, q, 1>), dim3((unsigned)n), dim3((unsigned)threads), 0, s, a); \
      }
      DG_TAIL_NP(X)
#undef X
      if (!done) return set_error(DG_ERR_UNSUPPORTED, "multigrid degree not compiled");
      if (int rc = check_hip(hipGetLastError(), "coarse cycle launch")) return rc;
    }
  return DG_OK;
}
template int launch_mg_tail_image<double>(int, const TailSeg<double>*, int, hipStream_t);
template int launch_mg_tail_image<float>(int, const TailSeg<float>*, int, hipStream_t);
template int launch_mg_tail<double>(int, const TailRun<double>*, int, hipStream_t);
template int launch_mg_tail<float>(int, const TailRun<float>*, int, hipStream_t);

}  // namespace dgwm
