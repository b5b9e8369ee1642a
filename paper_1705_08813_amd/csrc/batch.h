// Batched launches over many independent meshes (the serving path): the
// descriptors of up to K meshes (or mesh levels) travel by value in the
// kernel arguments of one launch, the workgroups of the launch dealt to
// them in order; larger batches take ceil(n / K) launches.  Segment s owns
// the blocks [blk0_s, blk0_{s+1}); blk0_0 = 0.  A mesh's segment runs the
// same compiled code in every launch it appears in, so its results do not
// depend on the other segments of the launch or on the batch.
#pragma once

#include "kern_common.h"

namespace dgwm {

// What the Poisson kernel does with y = A p at each output entry (solver fusion):
//   kPlain: y = A p
//   kResid: r = b - A p
//   kCheb:  v = c1 (p - zprev) + c2 dinv (b - A p), zout = p + v: one step
//           of the Chebyshev recurrence, whose previous iterate zprev is read
//           from zout before it is overwritten (c1 = 0: not read); zout must
//           not alias p
//   kChebFirst: the same step from the first iterate p = c0 dinv b (zprev =
//           0), which the kernel forms from b as it loads it (the input
//           pointer is b); p itself is written to z1 for the next step
enum PoiEpiKind { kPlain = 0, kResid = 1, kCheb = 2, kChebFirst = 3 };
template <typename T>
struct PoiEpi {
  int kind;
  const T* b;
  const T* dinv;
  T* z1;
  T* zout;
  T c1, c2, c0;
};

// N_i(x) of the NP-node Lobatto basis
template <int NP>
struct LobattoDen {  // 1 / prod_{j != i} (x_i - x_j)
  double inv[NP];
  constexpr LobattoDen() : inv{} {
    for (int i = 0; i < NP; ++i) {
      double d = 1.0;
      for (int j = 0; j < NP; ++j)
        if (j != i) d *= ct::lobatto<NP>.x[i] - ct::lobatto<NP>.x[j];
      inv[i] = 1.0 / d;
    }
  }
};
template <int NP>
inline constexpr LobattoDen<NP> lobatto_den{};

template <int NP>
__device__ __forceinline__ double lobatto_basis(int i, double x) {
  constexpr auto& L = ct::lobatto<NP>;
  double v = lobatto_den<NP>.inv[i];
#pragma unroll
  for (int j = 0; j < NP; ++j)
    if (j != i) v *= x - L.x[j];
  return v;
}

// Multigrid transfer geometry between a fine level and the next coarser one.
struct Tr {
  int nfx, nfy, nfz;   // fine level size
  int ncx, ncy, ncz;   // coarse level size
  int cx, cy, cz;
  const double* hyf;   // fine heights
};

// One mesh level of a batched Poisson launch (same degree and epilogue kind
// for every segment of a launch).
template <typename T>
struct PoiSeg {
  MeshDev M;
  const T* p;
  T* y;
  PoiEpi<T> E;
  int64_t ncell;
  int64_t blk0;
};

// One transfer of a batched restriction (out = P^T in) or prolongation
// (out = add + P in).
template <typename T>
struct TrSeg {
  Tr tr;
  const T* in;
  const T* add;
  T* out;
  int64_t ncc;
  int64_t blk0;
};

// x = B b with one mesh's dense coarsest-level inverse (n x n).
template <typename T>
struct DenseSeg {
  const T* B;
  const T* b;
  T* x;
  int64_t n;
  int64_t blk0;
};

// The coarse end of one mesh's V-cycle (kern_mg_tail.hip): its levels, first
// to coarsest, with their places in the workgroup's LDS (entries), and what
// the cycle reads and writes.  c*: coarsened towards the next level.  The first
// nimg entries of the LDS are constant over a solve and kept in memory as img.
constexpr int kTailLevels = 6;
constexpr int kTailImage = 8192;  // most entries of the image
template <typename T>
struct TailLevel {
  int nx, ny, nz, n, deg;
  int ob, od, ohy, oco, opy;    // ob: b, then x, n entries each; od: 1 / diagonal
  int cx, cy, cz;
  int ix, iy, ixy;              // ceil(2^16 / n) of nx, ny, nx ny
  double hx, hz, theta, delta;
  const double* hy;             // heights, then reciprocals
  const T* dinv;
};
template <typename T>
struct TailSeg {
  TailLevel<T> lv[kTailLevels];
  void* img;          // kTailHead bytes that hold this segment, then the image
  const T* B;         // dense inverse of the coarsest level (ndense x ndense), or nullptr
  const double* tab;  // the mesh's 1-D operators (poi_ops)
  T pen;
  int nlev, ndense, periodic, oscr, nscr, p0, groups, threads;
  int nimg, odense;   // odense: place of B in the image, -1: read from memory
};
constexpr size_t kTailHead = 1024;
static_assert(sizeof(TailSeg<double>) <= kTailHead && sizeof(TailSeg<float>) % 4 == 0, "segment in front of the image");
constexpr int kTailSegs = 4;
// One mesh's cycle: x = V-cycle(b) with the tables at img.
template <typename T>
struct TailRun {
  void* img;
  const T* b;
  T* x;
  int threads, groups;
};
constexpr int kTailRuns = 64;
template <typename T>
struct TailRuns {
  TailRun<T> r[kTailRuns];
};
template <typename T>
struct TailArr {
  TailSeg<T> s[kTailSegs];
};
static_assert(sizeof(TailArr<double>) <= 4000, "kernel arguments stay below 4 KiB");

// Segments per launch (kernel arguments stay below 4 KiB).
constexpr int kPoiSegs = 8, kTrSegs = 16, kDenseSegs = 32;
template <typename S, int K>
struct SegArr {
  S s[K];
  int n;
};

// Segment that owns block `bid` (segments sorted by blk0).
template <typename S, int K>
__device__ __forceinline__ int find_seg(const SegArr<S, K>& a, int64_t bid) {
  int lo = 0, hi = a.n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.s[mid].blk0 <= bid) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Host side: descriptors of one mesh level, workgroup counts, batched launchers.
MeshDev poisson_meshdev(const dg_mesh* m, int l);
// mesh arguments of the velocity kernels
MeshDev velocity_meshdev(const dg_mesh* m);
Tr mg_transfer_geometry(const dg_mesh* m, int l);
int poisson_cells_per_block(int np);
// the transfer kernel family a level pair uses and its coarse cells per workgroup
bool mg_full_transfer(const dg_mesh* m, int l);
int mg_cells_per_block(int np, bool full);
int dense_rows_per_block();

// The launchers take host arrays of segments (blk0 is filled in per launch)
// of one degree (and transfer family) and split them into launches of at
// most K segments.
template <typename T>
int launch_poisson_batched(int np, int kind, const PoiSeg<T>* segs, int nseg, hipStream_t s);
template <typename T>
int launch_mg_restrict_batched(int np, bool full, const TrSeg<T>* segs, int nseg, hipStream_t s);
template <typename T>
int launch_mg_prolong_batched(int np, bool full, const TrSeg<T>* segs, int nseg, hipStream_t s);
// Levels [l, nlev) of m as a tail segment (img and dinv left to the caller); false where they do not fit one workgroup.
// Smoothing interval [lam / range, 1.1 lam], degree deg0 on level 0 and degc below it; img_bytes are left for the image.
template <typename T>
bool mg_tail_segment(const dg_mesh* m, int l, int nlev, int deg0, int degc, double range, size_t img_bytes,
                     TailSeg<T>* S);
template <typename T>
int launch_mg_tail_image(int np, const TailSeg<T>* segs, int nseg, hipStream_t s);
template <typename T>
int launch_mg_tail(int np, const TailRun<T>* runs, int nrun, hipStream_t s);
template <typename T>
int launch_dense_batched(const DenseSeg<T>* segs, int nseg, hipStream_t s);

}  // namespace dgwm
