// Tile helpers of the direct projection-step solves: a tile holds NC
// columns (cells, or right-hand sides of cells) of 3 NP^3 nodal values,
// T[k * LD + col] with LD = NC + 1 (an odd stride: lanes along k and lanes
// along the columns both spread over the LDS banks), k = component * NP^3 +
// node and node = ix + NP iy + NP^2 iz.  NT threads share the work.
#pragma once

#include <hip/hip_runtime.h>

namespace dgwm {

constexpr int kTileCols = 16;  // cells (or right-hand sides) of a tile: the columns of one matrix-core product
constexpr int kTileLD = kTileCols + 1;
// Threads of a workgroup with a tile in LDS, and the wavefronts per SIMD whose
// registers have to fit: two tiles of k = 4 (55 KB) or one of k = 5 (90 KB)
// share a CU, so eight wavefronts a tile; more of the smaller tiles fit and
// four are enough.
constexpr int tile_threads(int np) { return np >= 5 ? 512 : 256; }
constexpr int tile_waves(int np) { return np == 5 ? 4 : 2; }

// In place along direction DIR of every (cell, component) block of the tile
// T[k * LD + c] (k = component * NP^3 + node, node = ix + NP iy + NP^2 iz).
template <int NP, int NT, int DIR>
__device__ __forceinline__ void tile_sweep(double* T, const double* Mt, int tid) {
  constexpr int NP2 = NP * NP, NP3 = NP2 * NP, NC = kTileCols, LD = kTileLD;
  constexpr int SD = DIR == 0 ? 1 : (DIR == 1 ? NP : NP2);
  for (int it = tid; it < NC * 3 * NP2; it += NT) {
    const int c = it % NC;
    const int rest = it / NC;
    const int comp = rest / NP2, l = rest - comp * NP2;
    const int base = DIR == 0 ? l * NP : (DIR == 1 ? (l % NP) + (l / NP) * NP2 : l);
    const int k0 = comp * NP3 + base;
    double v[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) v[i] = T[(k0 + i * SD) * LD + c];
#pragma unroll
    for (int a = 0; a < NP; ++a) {
      double o = 0.0;
#pragma unroll
      for (int i = 0; i < NP; ++i) o += Mt[a * NP + i] * v[i];
      T[(k0 + a * SD) * LD + c] = o;
    }
  }
}

// Reflection classes of a box cell's velocity space.  Reflecting the cell in
// direction d (and the component along d) maps mass and div-div form onto
// themselves, so in coordinates that are even or odd along every direction
// both fall into eight blocks, one per choice of signs: in class p (bit d: odd
// under reflection d) component c is odd along d when bit d of p, flipped for
// c = d, is set.  Along one direction the even coordinates v_i + v_{n-1-i}
// (and the middle node) come first, then the odd ones v_i - v_{n-1-i}.
// For k = 4 the blocks have 54, 3 x 51, 3 x 44 and 36 unknowns instead of 375
// together: 17,823 products a column instead of 140,625.
template <int NP>
struct Parity {
  static constexpr int NE = (NP + 1) / 2, NO = NP / 2, N = 3 * NP * NP * NP;
  static constexpr int odd(int p, int c, int d) { return ((p >> d) & 1) ^ (c == d ? 1 : 0); }
  static constexpr int count(int p) {
    int n = 0;
    for (int c = 0; c < 3; ++c) {
      int m = 1;
      for (int d = 0; d < 3; ++d) m *= odd(p, c, d) ? NO : NE;
      n += m;
    }
    return n;
  }
  static constexpr int tiles() {
    int t = 0;
    for (int p = 0; p < 8; ++p) t += (count(p) + 15) / 16;
    return t;
  }
  static constexpr int max_count() {
    int m = 0;
    for (int p = 0; p < 8; ++p) m = count(p) > m ? count(p) : m;
    return m;
  }
  static constexpr int TILES = tiles();                       // 16-row tiles
  static constexpr int KS = (max_count() + 3) / 4;  // 4-deep products of a row tile, the same for all classes
  static constexpr int ZN = 64 * KS * TILES;        // table entries of one product (BlockGemm)
  static constexpr int rows() {
    int m = N;
    for (int p = 0, o = 0; p < 8; o += count(p), ++p) m = o + 4 * KS > m ? o + 4 * KS : m;
    return m;
  }
  static constexpr int ROWS = rows();  // rows of a tile: the products of a small class read past its end
  int n[8], off[9];                    // sizes, first row in class order
  int to[TILES], tr[TILES], tn[TILES]; // first row of the class, of the tile in it; rows left in the class
  short pos[N];                // class order -> component * NP^3 + ix + NP iy + NP^2 iz
  constexpr Parity() : n{}, off{}, to{}, tr{}, tn{}, pos{} {
    int t = 0, o = 0;
    for (int p = 0; p < 8; ++p) {
      n[p] = count(p);
      off[p] = o;
      for (int r = 0; r < n[p]; r += 16) {
        to[t] = o;
        tr[t] = r;
        tn[t++] = n[p] - r;
      }
      for (int c = 0; c < 3; ++c) {
        const int x0 = odd(p, c, 0) ? NE : 0, x1 = odd(p, c, 0) ? NP : NE;
        const int y0 = odd(p, c, 1) ? NE : 0, y1 = odd(p, c, 1) ? NP : NE;
        const int z0 = odd(p, c, 2) ? NE : 0, z1 = odd(p, c, 2) ? NP : NE;
        for (int k = z0; k < z1; ++k)
          for (int j = y0; j < y1; ++j)
            for (int i = x0; i < x1; ++i) pos[o++] = (short)(c * NP * NP * NP + i + NP * (j + NP * k));
      }
    }
    off[8] = o;
  }
};
template <int NP>
inline constexpr Parity<NP> parity{};

// Tile from nodal values to even/odd coordinates in class order (sums and
// differences, unscaled) or, with BACK, from them (v_i = e_i + o_i, v_{n-1-i}
// = e_i - o_i); the layer tables carry the scaling.  A work item is the orbit
// of a node under the reflections (8 nodes, fewer on a middle plane), all
// three directions in registers; `cls` maps a coordinate to its row in class
// order.  Columns c = 0, CS, 2 CS, ...; the tile is complete on return.
template <int NP, int NT, bool BACK, int CS = 1>
__device__ __forceinline__ void tile_parity(double* T, const short* cls, int tid) {
  constexpr int NP2 = NP * NP, NP3 = NP2 * NP, LD = kTileLD, NE = (NP + 1) / 2, NCC = kTileCols / CS;
  constexpr int NI = NCC * 3 * NE * NE * NE, R = (NI + NT - 1) / NT;
  asm("" : "+v"(tid));  // addresses are formed here, not kept from one call to the next
  double v[R][8];
  auto each = [&](int r, auto&& fn) __attribute__((always_inline)) {
    const int it = tid + r * NT;
    if (R * NT != NI && it >= NI) return;
    const int c = (it % NCC) * CS, o = it / NCC;
    const int comp = o / (NE * NE * NE), l = o - comp * (NE * NE * NE);
    const int i0 = l % NE, i1 = (l / NE) % NE, i2 = l / (NE * NE);
    const bool d0 = NP % 2 && i0 == NE - 1, d1 = NP % 2 && i1 == NE - 1, d2 = NP % 2 && i2 == NE - 1;  // middle planes
    const int nx[2] = {i0, NP - 1 - i0}, ny[2] = {NP * i1, NP * (NP - 1 - i1)}, nz[2] = {NP2 * i2, NP2 * (NP - 1 - i2)};
    const int cx[2] = {i0, d0 ? i0 : NE + i0}, cy[2] = {NP * i1, NP * (d1 ? i1 : NE + i1)},
              cz[2] = {NP2 * i2, NP2 * (d2 ? i2 : NE + i2)};
    fn(c, comp * NP3, nx, ny, nz, cx, cy, cz, d0, d1, d2);
  };
#pragma unroll
  for (int r = 0; r < R; ++r)
    each(r, [&](int c, int k0, const int* nx, const int* ny, const int* nz, const int* cx, const int* cy, const int* cz,
                bool d0, bool d1, bool d2) __attribute__((always_inline)) {
      double(&w)[8] = v[r];
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const int row = BACK ? cls[k0 + cx[b & 1] + cy[(b >> 1) & 1] + cz[b >> 2]]
                             : k0 + nx[b & 1] + ny[(b >> 1) & 1] + nz[b >> 2];
        w[b] = T[row * LD + c];
      }
#pragma unroll
      for (int b = 0; b < 8; b += 2) {
        const double x = w[b], y = w[b + 1];
        w[b] = d0 ? x : x + y;
        w[b + 1] = d0 ? y : x - y;
      }
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int b = (m & 1) + 4 * (m >> 1);
        const double x = w[b], y = w[b + 2];
        w[b] = d1 ? x : x + y;
        w[b + 2] = d1 ? y : x - y;
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const double x = w[b], y = w[b + 4];
        w[b] = d2 ? x : x + y;
        w[b + 4] = d2 ? y : x - y;
      }
    });
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r)
    each(r, [&](int c, int k0, const int* nx, const int* ny, const int* nz, const int* cx, const int* cy, const int* cz,
                bool, bool, bool) __attribute__((always_inline)) {
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const int row = BACK ? k0 + nx[b & 1] + ny[(b >> 1) & 1] + nz[b >> 2]
                             : cls[k0 + cx[b & 1] + cy[(b >> 1) & 1] + cz[b >> 2]];
        T[row * LD + c] = v[r][b];
      }
    });
  __syncthreads();
}

typedef double dgwm_d4 __attribute__((ext_vector_type(4)));

// Block products on the matrix cores (FP64 MFMA 16 x 16 x 4) of a tile in
// class order, 16 columns: wavefront wv of NW owns the row tiles wv + NW q of
// Parity, D = Z_p^T(rows) T with the block Z_p[k][r] of its class.  Operand
// lanes: A (Z entries) lane l holds row l % 16, k = k0 + l / 16; B (tile) lane
// l holds k = k0 + l / 16, column l % 16; result element j of lane l is row
// 4 j + l / 16 of the tile, column l % 16.  The table holds the A operands in
// that order, 64 entries a step and KS steps a tile, zero beyond the class, so
// a load is one lane address and a constant; what a small class reads past its
// end is multiplied by zero.  The A operands of a step are loaded as soon as
// the same step of the tile before has used its own (those of the first tile
// by the caller, ahead of a barrier).
template <int NP, int NW>
struct BlockGemm {
  using PA = Parity<NP>;
  static constexpr int RT = (PA::TILES + NW - 1) / NW;
  double fa[PA::KS];

  __device__ __forceinline__ void load(const double* __restrict__ Z, int lane, int wv) {
    const double* z = Z + 64 * PA::KS * (wv < PA::TILES ? wv : 0) + lane;
#pragma unroll
    for (int s = 0; s < PA::KS; ++s) fa[s] = z[64 * s];
  }
  __device__ __forceinline__ void run(const double* T, const double* __restrict__ Z, dgwm_d4 (&acc)[RT], int lane,
                                      int wv) {
    constexpr auto& P = parity<NP>;
    const double* tl = T + (lane >> 4) * kTileLD + (lane & 15);
#pragma unroll
    for (int q = 0; q < RT; ++q) {
      acc[q] = dgwm_d4{0.0, 0.0, 0.0, 0.0};
      const int t = wv + NW * q;  // uniform over the wavefront
      if (NW * (q + 1) <= PA::TILES || t < PA::TILES) {
        // next tile (a wavefront without one loads this tile again)
        const double* z = Z + 64 * PA::KS * (t + NW < PA::TILES ? t + NW : t) + lane;
        const double* b = tl + P.to[t] * kTileLD;
        double fb[PA::KS];
#pragma unroll
        for (int s = 0; s < PA::KS; ++s) fb[s] = b[4 * s * kTileLD];
#pragma unroll
        for (int s = 0; s < PA::KS; ++s) {
          acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[s], fb[s], acc[q], 0, 0, 0);
          if (q + 1 < RT) fa[s] = z[64 * s];
        }
      }
    }
  }
  // row in class order of result element j of tile q of this lane, or -1
  __device__ __forceinline__ static int row(int q, int j, int lane, int wv) {
    constexpr auto& P = parity<NP>;
    const int t = wv + NW * q;
    if (NW * (q + 1) > PA::TILES && t >= PA::TILES) return -1;
    const int r = 4 * j + (lane >> 4);
    return r < P.tn[t] ? P.to[t] + P.tr[t] + r : -1;
  }
};

}  // namespace dgwm
