// Barnes-Hut tree code on the GPU (the paper's collisionless method: section
// "Simulating collisionless systems with hierarchical domain-decomposition
// methods", subsection "Implementation"): every part runs on the device --
// Peano-Hilbert keys and the sort along the curve, an octree whose cells cut
// the curve into distinct pieces until a cell holds at most n_crit
// particles, monopole and quadrupole moments, groups of up to 64
// curve-consecutive particles (split while wider than g_max), the walk with
// a geometric opening criterion, and the force evaluation.
//
// Readings shared with the documentation of nb_tree_forces (nbody.h):
//  * box: lo = per-dimension minimum, side = 2^e >= (1 + 2^-10) * largest
//    extent, h = side 2^-21, integer coordinates floor((x - lo)/h) clamped
//  * keys: 63-bit Peano-Hilbert index (Skilling's construction), particles
//    sorted by (key, index) with a stable radix sort
//  * cell (l, p): the particles with key prefix p of 3l bits; split while it
//    holds more than n_crit particles (l < 21); cube corner from the first
//    particle's coordinates with the low 21-l bits cleared, side 2^(21-l) h
//  * a cell other than the root is accepted for a group when
//    theta^2 d^2 > side^2, d the distance between the group's bounding box
//    and the cube; an opened leaf's particles interact directly
//  * accepted cell: a = -M y s^-3/2 + Q y s^-5/2 - (5/2)(y.Qy) y s^-7/2,
//    phi = -M s^-1/2 - (y.Qy)/2 s^-5/2 with y = x - X, s = |y|^2 + eps2,
//    Q = sum m (3 d d^T - |d|^2 I) about the centre of mass X
//
// Structure on the chip: the build is data-parallel -- one thread per
// particle, with the library's own stable radix sort and exclusive scans
// placing the outputs, so every array keeps curve order and the results are
// reproducible run to run.  (Few particles are sorted by counting each key's
// place instead.)  All levels are built at once; the level bounds
// stay in device memory and the buffers are sized from bounds known up front,
// so nothing is read on the host until the forces are written and a whole
// evaluation can be captured in a graph.  The walk and the force evaluation are
// one kernel, as in the paper's GPU tree code: one wavefront per group, or a
// team of eight while groups are few, walks the tree for the group's 64
// particles and evaluates accepted cells and opened leaves 64 at a time from
// LDS as it finds them, so no interaction list is written to memory.  The
// build and the walk are double precision; the force terms are double or
// mixed (float terms from double separations, summed in double per chunk)
// with the context's precision.  The opening test and the cube geometry are
// computed without fused multiply-adds, in the order stated above, so they
// match any implementation that rounds each operation.
#include <string>
#include <type_traits>
#include <vector>

#include "nb_internal.h"
#include "work_queue.h"

namespace nb {
namespace {

constexpr int kBits = 21;
constexpr int kLevels = kBits + 1;  // cell levels 0 .. kBits
constexpr int kTB = 256;   // threads per block of the element-wise kernels
constexpr int kGS = 64;    // particles per group (one wavefront)

inline int blocks_for(int64_t n, int cap = 65535) {
  int64_t g = (n + kTB - 1) / kTB;
  return (int)(g < 1 ? 1 : (g > cap ? cap : g));
}

struct Box {
  double lo[3];
  double side;
  double h;
};

// A particle in curve order.
struct Part {
  double x[3], m;
};

// What the walk reads of a cell.
struct TreeCell {
  int32_t begin, end;      // range of the cell's particles along the curve
  int32_t child0, child1;  // the children are [child0, child1); both -1 for a leaf
  double corner[3];        // cube corner and side
  double side;
};
// What the evaluation reads of it: centre of mass, mass and traceless
// quadrupole (xx, yy, zz, xy, xz, yz).
struct CellMom {
  double X[3], M, Q[6];
};
// The same for the mixed terms: the separation is formed in double, the rest
// is float.
struct CellMomF {
  double X[3];
  float M, Q[6], pad[3];
};

// ---------------------------------------------------------------- box -----
// Minimum and maximum of three components over the kTB threads of a block
// (red is free again after the next barrier).
__device__ __forceinline__ void block_minmax(double* mn, double* mx, double (*red)[6]) {
  constexpr int W = kTB / 64;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      mn[c] = fmin(mn[c], __shfl_xor(mn[c], o, 64));
      mx[c] = fmax(mx[c], __shfl_xor(mx[c], o, 64));
    }
    if ((threadIdx.x & 63) == 0) {
      red[threadIdx.x >> 6][c] = mn[c];
      red[threadIdx.x >> 6][3 + c] = mx[c];
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    mn[c] = red[0][c];
    mx[c] = red[0][3 + c];
#pragma unroll
    for (int w = 1; w < W; ++w) {
      mn[c] = fmin(mn[c], red[w][c]);
      mx[c] = fmax(mx[c], red[w][3 + c]);
    }
  }
}

__global__ __launch_bounds__(kTB) void k_bbox_partial(const double* __restrict__ pos, int64_t n,
                                                      double* __restrict__ part) {
  __shared__ double red[kTB / 64][6];
  double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int64_t i = (int64_t)blockIdx.x * kTB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kTB)
    for (int c = 0; c < 3; ++c) {
      const double x = pos[3 * i + c];
      mn[c] = fmin(mn[c], x);
      mx[c] = fmax(mx[c], x);
    }
  block_minmax(mn, mx, red);
  if (threadIdx.x == 0)
    for (int c = 0; c < 3; ++c) {
      part[6 * (int64_t)blockIdx.x + c] = mn[c];
      part[6 * (int64_t)blockIdx.x + 3 + c] = mx[c];
    }
}

// The box from the partial minima and maxima, by every thread of a block
// alike (each block of the key pass does it for itself: a launch of its own
// costs more).
__device__ __forceinline__ Box box_of(const double* __restrict__ part, int nblk, double (*red)[6]) {
  double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int b = threadIdx.x; b < nblk; b += kTB)
    for (int c = 0; c < 3; ++c) {
      mn[c] = fmin(mn[c], part[6 * b + c]);
      mx[c] = fmax(mx[c], part[6 * b + 3 + c]);
    }
  block_minmax(mn, mx, red);
  double ext = 0.0;
  for (int c = 0; c < 3; ++c) ext = fmax(ext, mx[c] - mn[c]);
  double side = 1.0;
  if (ext > 0.0) {
    int e = 0;
    (void)frexp(ext * (1.0 + 0x1p-10), &e);
    side = ldexp(1.0, e);
  }
  Box bx;
  for (int c = 0; c < 3; ++c) bx.lo[c] = mn[c];
  bx.side = side;
  bx.h = ldexp(side, -kBits);
  return bx;
}

// --------------------------------------------------------------- keys -----
__device__ __forceinline__ void grid_of(const double* x, const Box& b, int32_t* q) {
  for (int c = 0; c < 3; ++c) {
    double v = floor((x[c] - b.lo[c]) / b.h);
    v = v < 0.0 ? 0.0 : (v > (double)((1 << kBits) - 1) ? (double)((1 << kBits) - 1) : v);
    q[c] = (int32_t)v;
  }
}

// Peano-Hilbert index of three 21-bit coordinates: plane by plane from the
// top, an axis whose bit is set flips the lower bits of axis 0, otherwise
// the two trade their lower bits; then Gray coding along the axes and the
// parity mask of the last axis; finally the bits interleaved from the top.
__device__ __forceinline__ uint64_t hilbert63(uint32_t a0, uint32_t a1, uint32_t a2) {
  uint32_t w[3] = {a0, a1, a2};
  for (uint32_t plane = 1u << (kBits - 1); plane > 1u; plane >>= 1) {
    const uint32_t low = plane - 1u;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (w[k] & plane) {
        w[0] ^= low;
      } else {
        const uint32_t d = (w[0] ^ w[k]) & low;
        w[0] ^= d;
        w[k] ^= d;
      }
    }
  }
  w[1] ^= w[0];
  w[2] ^= w[1];
  uint32_t mask = 0;
  for (uint32_t plane = 1u << (kBits - 1); plane > 1u; plane >>= 1)
    if (w[2] & plane) mask ^= plane - 1u;
  w[0] ^= mask; w[1] ^= mask; w[2] ^= mask;
  uint64_t key = 0;
  for (int b = kBits - 1; b >= 0; --b)
#pragma unroll
    for (int k = 0; k < 3; ++k) key = (key << 1) | ((w[k] >> b) & 1u);
  return key;
}

// idx (may be null): the rows, for a sort that carries them along.
__global__ __launch_bounds__(kTB) void k_keys(const double* __restrict__ pos, int64_t n,
                                              const double* __restrict__ part, int nblk, Box* __restrict__ box,
                                              uint64_t* __restrict__ keys, int32_t* __restrict__ idx) {
  __shared__ double red[kTB / 64][6];
  const Box b = box_of(part, nblk, red);
  if (blockIdx.x == 0 && threadIdx.x == 0) *box = b;
  for (int64_t i = (int64_t)blockIdx.x * kTB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kTB) {
    int32_t q[3];
    grid_of(pos + 3 * i, b, q);
    keys[i] = hilbert63((uint32_t)q[0], (uint32_t)q[1], (uint32_t)q[2]);
    if (idx) idx[i] = (int32_t)i;
  }
}

// --------------------------------------------------------------- tree -----
// The whole tree follows from the sorted keys at once, without a pass per
// level.  A cell (l, p) exists when its parent holds more than n_crit
// particles, so particle i has cells on levels 0 .. top(i) = min(e(i) + 1, 21)
// where e(i) is the deepest level whose cell around i holds more than n_crit
// particles; and i is the first particle of its level-l cell for every
// l >= d(i), one more than the levels its key shares with the key before it.
// So i starts exactly the cells of levels d(i) .. top(i).  Three kernels: per
// tile of kTB particles the number of cells starting on each level
// (k_cell_starts), the prefix of those counts over the tiles, one block per
// level (k_level_scan), and the cells at their places (k_write_cells): level
// after level, in curve order within each, children contiguous.  (A pass of
// three kernels per level, 63 launches whatever the depth, took 0.3-0.35 ms
// per evaluation of 10^4 and of 2.6 x 10^5 particles, most of it launches and
// latency; these three take 26 and 40 us.)
__device__ __forceinline__ void set_geometry(TreeCell& c, int level, const int32_t* ijk, const Box& b) {
#pragma clang fp contract(off)
  const int shift = kBits - level;
  for (int k = 0; k < 3; ++k) {
    const int64_t ci = ((int64_t)ijk[k] >> shift) << shift;
    c.corner[k] = b.lo[k] + (double)ci * b.h;
  }
  c.side = ldexp(b.h, shift);
}

constexpr int kCtrWords = 256;      // the walk's counters (kCtrLine words per XCD)
// What the caller's counts are made of, in one block of memory so that one
// copy brings it to the host: the walk's counters, where each level's cells
// start (and the last ends), and the number of groups.
struct Counts {
  unsigned long long ctr[kCtrWords];
  int32_t lvl[kLevels + 1];
  int32_t ngroups;
};
constexpr int kRows = kLevels + 1;  // per-tile counts: cells starting on each level, then groups
constexpr int kMaxWindow = 256;     // n_crit + 1 up to which the window maximum runs in LDS

// leading octal digits two 63-bit keys share (21: equal)
__device__ __forceinline__ int shared_levels(uint64_t a, uint64_t b) {
  const uint64_t x = a ^ b;
  return x ? (__clzll((long long)x) - 1) / 3 : kBits;
}

// first position in [lo, hi) whose key is >= bound (hi if none)
__device__ __forceinline__ int32_t lower_bound_key(const uint64_t* __restrict__ keys, int32_t lo, int32_t hi,
                                                   uint64_t bound) {
  while (lo < hi) {
    const int32_t mid = lo + (hi - lo) / 2;
    if (keys[mid] < bound) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// e(i) for any n_crit: the deepest level (below 22, -1 for none) whose cell
// around i holds more than n_crit particles, by bisection over the levels
__device__ __forceinline__ int deepest_full(const uint64_t* __restrict__ keys, int32_t n, int32_t i, int n_crit) {
  int lo = -1, hi = kBits;
  while (lo < hi) {
    const int l = (lo + hi + 1) >> 1;
    const int sh = 3 * (kBits - l);
    const uint64_t p = keys[i] >> sh;
    const int32_t b = lower_bound_key(keys, 0, i, p << sh);
    const int32_t e = lower_bound_key(keys, i, n, (p + 1) << sh);
    if (e - b > n_crit) lo = l;
    else hi = l - 1;
  }
  return lo;
}

// number of set bits of `mask` below this lane
__device__ __forceinline__ int lane_rank(uint64_t mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// The group that holds this lane's particle: a chunk of m <= 64 particles is
// halved (first half ceil(n/2)) while a piece of more than one particle is
// wider than g_max.  A full chunk is only ever cut at aligned halves, and a
// piece that fits has pieces that fit, so the group is the largest aligned
// piece around the lane that fits: minimum and maximum over the aligned
// pieces of 2, 4, ..., 64 lanes by butterfly shuffles.  In the last, shorter
// chunk every lane follows the halving of its own piece on the positions in
// LDS (one lane doing it for all took 19 us).
struct Piece {
  int begin, end;          // lanes of the group
  double lo[3], hi[3];     // its bounding box
};
__device__ __forceinline__ Piece group_of(int lane, int m, const double* x, double g_max, double (*xs)[3]) {
  Piece p;
  for (int k = 0; k < 3; ++k) p.lo[k] = p.hi[k] = x[k];
  if (m == kGS) {
    double mn[3], mx[3];
    for (int k = 0; k < 3; ++k) mn[k] = mx[k] = x[k];
    int size = 1;
    for (int h = 1; h < kGS; h <<= 1) {
      for (int k = 0; k < 3; ++k) {
        mn[k] = fmin(mn[k], __shfl_xor(mn[k], h, kGS));
        mx[k] = fmax(mx[k], __shfl_xor(mx[k], h, kGS));
      }
      const double ext = fmax(mx[0] - mn[0], fmax(mx[1] - mn[1], mx[2] - mn[2]));
      if (size == h && !(ext > g_max)) {
        size = 2 * h;
        for (int k = 0; k < 3; ++k) {
          p.lo[k] = mn[k];
          p.hi[k] = mx[k];
        }
      }
    }
    p.begin = lane & ~(size - 1);
    p.end = p.begin + size;
    return p;
  }
  for (int k = 0; k < 3; ++k) xs[lane][k] = x[k];
  __builtin_amdgcn_wave_barrier();
  p.begin = 0;
  p.end = m;
  while (lane < m && p.end - p.begin > 1) {
    double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int j = p.begin; j < p.end; ++j)
      for (int k = 0; k < 3; ++k) {
        mn[k] = fmin(mn[k], xs[j][k]);
        mx[k] = fmax(mx[k], xs[j][k]);
      }
    if (!(fmax(mx[0] - mn[0], fmax(mx[1] - mn[1], mx[2] - mn[2])) > g_max)) {
      for (int k = 0; k < 3; ++k) {
        p.lo[k] = mn[k];
        p.hi[k] = mx[k];
      }
      break;
    }
    const int mid = p.begin + (p.end - p.begin + 1) / 2;
    if (lane < mid) p.end = mid;
    else p.begin = mid;
  }
  return p;
}

// Mass, centre of mass X and traceless quadrupole about it of a tile's
// particles.  Without a positive mass (masses of both signs) X is the tile's
// first particle instead and D the first moment about it (otherwise zero).
struct TileMoments {
  double M, X[3], Q[6], D[3];
};

template <int G>
__device__ __forceinline__ double fold_lanes(double v) {
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Q += the traceless quadrupole of mass m at offset e
__device__ __forceinline__ void add_quad(double* Q, double m, double e0, double e1, double e2) {
  const double ee = e0 * e0 + e1 * e1 + e2 * e2;
  Q[0] += m * (3.0 * (e0 * e0) - ee);
  Q[1] += m * (3.0 * (e1 * e1) - ee);
  Q[2] += m * (3.0 * (e2 * e2) - ee);
  Q[3] += m * (3.0 * (e0 * e1));
  Q[4] += m * (3.0 * (e0 * e2));
  Q[5] += m * (3.0 * (e1 * e2));
}

// Q += what a first moment D about X adds to the quadrupole about X - e
__device__ __forceinline__ void add_dipole(double* Q, const double* D, double e0, double e1, double e2) {
  const double de = 2.0 * (D[0] * e0 + D[1] * e1 + D[2] * e2);
  Q[0] += 6.0 * D[0] * e0 - de;
  Q[1] += 6.0 * D[1] * e1 - de;
  Q[2] += 6.0 * D[2] * e2 - de;
  Q[3] += 3.0 * (D[0] * e1 + D[1] * e0);
  Q[4] += 3.0 * (D[0] * e2 + D[2] * e0);
  Q[5] += 3.0 * (D[1] * e2 + D[2] * e1);
}

// Sums of N values over the block's threads, in a fixed order; red is free
// again after the next barrier.
template <int N>
__device__ __forceinline__ void block_fold(double* v, double (*red)[6]) {
  constexpr int W = kTB / kGS;
  for (int k = 0; k < N; ++k) {
    v[k] = fold_lanes<64>(v[k]);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][k] = v[k];
  }
  __syncthreads();
  for (int k = 0; k < N; ++k) {
    v[k] = red[0][k];
    for (int w = 1; w < W; ++w) v[k] += red[w][k];
  }
}

// Per tile: the particles in curve order, d(i) and top(i) of each (span), the
// numbers of cells starting on each level and of groups, and the moments.
__global__ __launch_bounds__(kTB) void k_cell_starts(const uint64_t* __restrict__ keys, const int32_t* __restrict__ idx,
                                                     const double* __restrict__ pos, const double* __restrict__ mass,
                                                     int32_t n, int n_crit, const Box* __restrict__ box, double g_frac,
                                                     Part* __restrict__ part, uint16_t* __restrict__ span,
                                                     int32_t* __restrict__ cnt, int32_t ntile,
                                                     TileMoments* __restrict__ tiles) {
  constexpr int W = kTB / kGS;
  __shared__ double red[2][W][6];
  __shared__ int8_t win[2][kTB + kMaxWindow];
  __shared__ int32_t wcnt[W][kRows];
  __shared__ double xs[W][kGS][3];
  const int t = threadIdx.x, lane = t & (kGS - 1), wave = t / kGS;
  const int32_t tile0 = (int32_t)blockIdx.x * kTB, i = tile0 + t;
  const bool valid = i < n;
  double x[3] = {0.0, 0.0, 0.0}, pm = 0.0;
  if (valid) {
    const int64_t o = idx[i];
    for (int k = 0; k < 3; ++k) x[k] = pos[3 * o + k];
    pm = mass[o];
    part[i] = Part{{x[0], x[1], x[2]}, pm};
  }
  {
    double v[4] = {pm, pm * x[0], pm * x[1], pm * x[2]}, q[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    block_fold<4>(v, red[0]);
    double X[3], D[3] = {0.0, 0.0, 0.0};
    if (v[0] > 0.0) {
      for (int k = 0; k < 3; ++k) X[k] = v[1 + k] / v[0];
    } else {
      const int64_t o = idx[tile0];
      for (int k = 0; k < 3; ++k) {
        X[k] = pos[3 * o + k];
        D[k] = v[1 + k] - v[0] * X[k];
      }
    }
    if (valid) add_quad(q, pm, x[0] - X[0], x[1] - X[1], x[2] - X[2]);
    block_fold<6>(q, red[1]);
    if (t == 0) {
      TileMoments& tm = tiles[blockIdx.x];
      tm.M = v[0];
      for (int k = 0; k < 3; ++k) tm.X[k] = X[k];
      for (int k = 0; k < 6; ++k) tm.Q[k] = q[k];
      for (int k = 0; k < 3; ++k) tm.D[k] = D[k];
    }
  }
  int e = -1;
  if (n_crit < kMaxWindow) {
    // e(i) is the largest number of levels that keys k and k + n_crit share
    // over the windows k <= i <= k + n_crit; maximum by doubling
    const int len = kTB + n_crit;
    for (int q = t; q < len; q += kTB) {
      const int64_t k = (int64_t)tile0 - n_crit + q;
      win[0][q] = (k >= 0 && k + n_crit < n) ? (int8_t)shared_levels(keys[k], keys[k + n_crit]) : (int8_t)-1;
    }
    __syncthreads();
    int p = 1, cur = 0;
    for (; 2 * p <= n_crit + 1; p *= 2, cur ^= 1) {
      for (int q = t; q < len; q += kTB) {
        const int8_t u = win[cur][q], v = q + p < len ? win[cur][q + p] : (int8_t)-1;
        win[cur ^ 1][q] = u > v ? u : v;
      }
      __syncthreads();
    }
    const int8_t u = win[cur][t], v = win[cur][t + n_crit + 1 - p];
    e = u > v ? u : v;
  } else if (valid) {
    e = deepest_full(keys, n, i, n_crit);
  }
  const int top = e + 1 < kBits ? e + 1 : kBits;
  const int d = i == 0 ? 0 : (valid ? shared_levels(keys[i - 1], keys[i]) + 1 : kBits + 1);
  if (valid) span[i] = (uint16_t)(d | (top << 8));
  int32_t mine = 0;
  for (int l = 0; l < kLevels; ++l) {
    const int32_t c = __popcll(__ballot(valid && d <= l && l <= top));
    if (lane == l) mine = c;
  }
  if (lane < kLevels) wcnt[wave][lane] = mine;
  // groups of the wavefront's chunk
  const int32_t left = n - (tile0 + wave * kGS);
  const int m = left < kGS ? (left > 0 ? left : 0) : kGS;
  const double g_max = g_frac > 0.0 ? g_frac * box->side : INFINITY;
  const Piece p = group_of(lane, m, x, g_max, xs[wave]);
  const uint64_t starts = __ballot(lane < m && p.begin == lane);
  if (lane == 0) wcnt[wave][kLevels] = __popcll(starts);
  __syncthreads();
  if (t < kRows) {
    int32_t sum = 0;
    for (int w = 0; w < W; ++w) sum += wcnt[w][t];
    cnt[(int64_t)t * ntile + blockIdx.x] = sum;
  }
}

// Exclusive prefix of one row of tile counts (block r), in place, and its
// total; also zeroes the walk's counters.
__global__ __launch_bounds__(1024) void k_level_scan(int32_t* __restrict__ cnt, int32_t ntile,
                                                     int32_t* __restrict__ total,
                                                     unsigned long long* __restrict__ ctr) {
  constexpr int T = 1024, W = T / 64;
  __shared__ int32_t wsum[2][W];
  int32_t* row = cnt + (int64_t)blockIdx.x * ntile;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int32_t carry = 0;
  int buf = 0;
  for (int32_t base = 0; base < ntile; base += T) {
    const int32_t k = base + t;
    const int32_t v = k < ntile ? row[k] : 0;
    int32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) wsum[buf][wave] = x;
    __syncthreads();  // the totals alternate between two buffers: one barrier per round
    int32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      before += w < wave ? wsum[buf][w] : 0;
      all += wsum[buf][w];
    }
    if (k < ntile) row[k] = carry + before + x - v;
    carry += all;
    buf ^= 1;
  }
  if (t == 0) total[blockIdx.x] = carry;
  if (blockIdx.x == 0 && t < kCtrWords) ctr[t] = 0ull;
}

// Cells and groups at their places.  Thread i writes the cells its particle
// starts (levels d(i) .. top(i)) and closes those that end before it: levels
// d(i) .. top(i - 1), each the last cell starting before i on its level.  The
// first child of a cell starts at the cell's own particle; the last child is
// the cell closed together with it one level deeper.
__global__ __launch_bounds__(kTB) void k_write_cells(TreeCell* __restrict__ cells, const uint16_t* __restrict__ span,
                                                     const int32_t* __restrict__ cnt,
                                                     const int32_t* __restrict__ total, int32_t ntile, int32_t n,
                                                     const Part* __restrict__ part, const Box* __restrict__ box,
                                                     double g_frac, int32_t* __restrict__ lvl,
                                                     int32_t* __restrict__ gb, int32_t* __restrict__ ge,
                                                     double* __restrict__ gbox, int32_t* __restrict__ ng) {
  constexpr int W = kTB / kGS;
  __shared__ int32_t first[W][kRows];  // index of a wavefront's first cell of a level, or group
  __shared__ int32_t wcnt[W][kRows];
  __shared__ double xs[W][kGS][3];
  const int t = threadIdx.x, lane = t & (kGS - 1), wave = t / kGS;
  const int32_t tile0 = (int32_t)blockIdx.x * kTB, i = tile0 + t;
  const bool valid = i < n;
  const Box bx = *box;
  int d = kLevels, top = -1;
  double x[3] = {0.0, 0.0, 0.0};
  if (valid) {
    const int sp = span[i];
    d = sp & 255;
    top = sp >> 8;
    for (int k = 0; k < 3; ++k) x[k] = part[i].x[k];
  }
  int32_t mine = 0;
  for (int l = 0; l < kLevels; ++l) {
    const int32_t c = __popcll(__ballot(d <= l && l <= top));
    if (lane == l) mine = c;
  }
  if (lane < kLevels) wcnt[wave][lane] = mine;
  const int32_t left = n - (tile0 + wave * kGS);
  const int m = left < kGS ? (left > 0 ? left : 0) : kGS;
  const double g_max = g_frac > 0.0 ? g_frac * bx.side : INFINITY;
  const Piece p = group_of(lane, m, x, g_max, xs[wave]);
  const bool gstart = lane < m && p.begin == lane;
  const uint64_t gmask = __ballot(gstart);
  if (lane == 0) wcnt[wave][kLevels] = __popcll(gmask);
  __syncthreads();
  if (t < kRows) {
    int32_t at = cnt[(int64_t)t * ntile + blockIdx.x];
    if (t < kLevels)
      for (int l = 0; l < t; ++l) at += total[l];
    for (int w = 0; w < W; ++w) {
      first[w][t] = at;
      at += wcnt[w][t];
    }
  }
  if (blockIdx.x == 0 && t <= kLevels) {
    int32_t at = 0;
    for (int l = 0; l < t; ++l) at += total[l];
    lvl[t] = at;  // the cells of level l are [lvl[l], lvl[l + 1])
    if (t == kLevels) *ng = total[kLevels];
  }
  __syncthreads();
  if (gstart) {
    const int32_t g = first[wave][kLevels] + lane_rank(gmask);
    gb[g] = i;
    ge[g] = i + (p.end - p.begin);
    for (int k = 0; k < 3; ++k) {
      gbox[6 * (int64_t)g + k] = p.lo[k];
      gbox[6 * (int64_t)g + 3 + k] = p.hi[k];
    }
  }
  int32_t q[3] = {0, 0, 0};
  if (d <= top) grid_of(x, bx, q);
  const int before_top = valid && i > 0 ? span[i - 1] >> 8 : -1;
  const bool last = i == n - 1;
  int32_t above = 0, above_incl = 0;  // one level up: cells before those starting at i; and including them
  for (int l = 0; l < kLevels; ++l) {
    const bool start = d <= l && l <= top;
    const int32_t c = first[wave][l] + lane_rank(__ballot(start));
    const int32_t incl = c + (start ? 1 : 0);
    if (start) {
      TreeCell& cell = cells[c];
      cell.begin = i;
      set_geometry(cell, l, q, bx);
      if (l == top) cell.child0 = cell.child1 = -1;
      if (l > d) cells[above].child0 = c;
    }
    if (l >= d && l <= before_top) {
      cells[c - 1].end = i;
      if (l > d) cells[above - 1].child1 = c;
    }
    if (last && l <= top) {
      cells[incl - 1].end = n;
      if (l > 0) cells[above_incl - 1].child1 = incl;
    }
    above = c;
    above_incl = incl;
  }
}

// ------------------------------------------------------------ moments -----
// Every cell's moments from its particles, or, where a cell holds whole tiles
// of the curve, from those tiles' moments (k_cell_starts computes them), so no
// level waits for the one below and one launch does all.  Cells of up to
// kSmallCell particles take eight lanes, larger ones a wavefront.  Cell c
// belongs to block c mod the grid: the large cells, which come first in the
// level order, go to different blocks.  The root is never accepted and gets
// no moments.  2.6 x 10^5 particles: 38 us (22 launches, one per level,
// summing children: 140 us; without the tile moments: 640 us, spent on the
// largest cells).
constexpr int kSmallCell = 64;
constexpr int kDirectCell = 512;  // up to here a wavefront takes the particles one by one

// The moments of one cell by the G lanes `t`: of its tm0 <= tile < tm1 whole
// tiles and of the particles before and after them.  momf: the float copy of
// the mixed terms, when they are wanted.
template <int G>
__device__ __forceinline__ void moments_of(const TreeCell& c, CellMom* __restrict__ mom, CellMomF* __restrict__ momf,
                                           const Part* __restrict__ part, const TileMoments* __restrict__ tiles,
                                           int32_t tm0, int32_t tm1, int t) {
  const int32_t b = c.begin, e = c.end;
  const int32_t head = tm1 > tm0 ? tm0 * kTB - b : e - b;  // particles before the tiles (all of them without)
  const int32_t skip = (tm1 - tm0) * kTB;
  const int32_t singles = e - b - skip;
  double M = 0.0, S[3] = {0.0, 0.0, 0.0}, Q[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, X[3];
  for (int32_t u = t; u < singles; u += G) {
    const Part p = part[(int64_t)b + u + (u < head ? 0 : skip)];
    M += p.m;
    for (int k = 0; k < 3; ++k) S[k] += p.m * p.x[k];
  }
  for (int32_t u = tm0 + t; u < tm1; u += G) {
    M += tiles[u].M;
    for (int k = 0; k < 3; ++k) S[k] += tiles[u].M * tiles[u].X[k];
    if (!(tiles[u].M > 0.0))
      for (int k = 0; k < 3; ++k) S[k] += tiles[u].D[k];
  }
  M = fold_lanes<G>(M);
  for (int k = 0; k < 3; ++k) {
    S[k] = fold_lanes<G>(S[k]);
    X[k] = M > 0.0 ? S[k] / M : c.corner[k] + 0.5 * c.side;
  }
  for (int32_t u = t; u < singles; u += G) {
    const Part p = part[(int64_t)b + u + (u < head ? 0 : skip)];
    add_quad(Q, p.m, p.x[0] - X[0], p.x[1] - X[1], p.x[2] - X[2]);
  }
  for (int32_t u = tm0 + t; u < tm1; u += G) {
    for (int k = 0; k < 6; ++k) Q[k] += tiles[u].Q[k];
    const double e[3] = {tiles[u].X[0] - X[0], tiles[u].X[1] - X[1], tiles[u].X[2] - X[2]};
    add_quad(Q, tiles[u].M, e[0], e[1], e[2]);
    if (!(tiles[u].M > 0.0)) add_dipole(Q, tiles[u].D, e[0], e[1], e[2]);
  }
  for (int k = 0; k < 6; ++k) Q[k] = fold_lanes<G>(Q[k]);
  if (t != 0) return;
  if (momf) {
    CellMomF f{};
    f.M = (float)M;
    for (int k = 0; k < 3; ++k) f.X[k] = X[k];
    for (int k = 0; k < 6; ++k) f.Q[k] = (float)Q[k];
    *momf = f;
  } else {
    CellMom f;
    f.M = M;
    for (int k = 0; k < 3; ++k) f.X[k] = X[k];
    for (int k = 0; k < 6; ++k) f.Q[k] = Q[k];
    *mom = f;
  }
}

__global__ __launch_bounds__(kTB) void k_cell_moments(const TreeCell* __restrict__ cells, CellMom* __restrict__ mom,
                                                      CellMomF* __restrict__ momf, const int32_t* __restrict__ lvl,
                                                      const Part* __restrict__ part,
                                                      const TileMoments* __restrict__ tiles) {
  const int32_t ncell = lvl[kLevels];
  const int t = threadIdx.x;
  const int32_t nb = gridDim.x;
  for (int64_t c = blockIdx.x + (int64_t)(t >> 3) * nb; c < ncell; c += (int64_t)(kTB / 8) * nb) {
    const int32_t size = cells[c].end - cells[c].begin;
    if (c > 0 && size <= kSmallCell)
      moments_of<8>(cells[c], mom + c, momf ? momf + c : nullptr, part, tiles, 0, 0, t & 7);
  }
  for (int64_t c = blockIdx.x + (int64_t)(t >> 6) * nb; c < ncell; c += (int64_t)(kTB / 64) * nb) {
    const int32_t b = cells[c].begin, e = cells[c].end;
    if (c == 0 || e - b <= kSmallCell) continue;
    int32_t tm0 = 0, tm1 = 0;
    if (e - b > kDirectCell) {  // holds a whole tile: the tiles within [b, e)
      tm0 = (int32_t)(((int64_t)b + kTB - 1) / kTB);
      tm1 = e / kTB;
    }
    moments_of<64>(cells[c], mom + c, momf ? momf + c : nullptr, part, tiles, tm0, tm1, t & 63);
  }
}

// ------------------------------------------------- walk and forces -----
// One kernel does the walk and the force evaluation, as the paper's GPU
// tree code does: a wavefront takes a group (its lanes are the group's
// particles), walks the tree for the whole group, and evaluates the accepted
// cells and the particles of opened leaves as soon as 64 of them are
// pending.  No interaction list goes to memory; the only memory beyond the
// tree is a per-wavefront stack of cells still to be tested.
//
// Walk step: pop up to 64 cells from the top of the stack, one per lane;
// each lane tests its cell and the wavefront appends accepted cells and
// opened leaves to two LDS lists (ballot + rank) and pushes the children of
// opened internal cells, in lane order, onto the stack (prefix sum).
// Bound on the stack: the pushes keep it ordered by level from bottom to
// top (lane order is stack order, children sit one level below their
// parents, and what is left after a pop is no deeper than what was popped).
// Level-l entries are pushed only by a pop that took level-(l-1) entries,
// and such a pop took every entry of level >= l, which lie above them; so
// the level-l entries on the stack always come from one push of at most
// 8 x 64 entries, and the stack holds at most 8 x 64 x 21 entries (levels
// 1 to 21).  It also never holds more entries than there are cells, since
// a cell is pushed at most once per group.  The kernel still checks every
// push against the capacity and reports an overflow instead of writing
// past it.
constexpr int kStackCap = 8 * kGS * kBits;

__device__ __forceinline__ bool accepted(const TreeCell& c, const double* gbox, double theta) {
#pragma clang fp contract(off)
  double d2 = 0.0;
  for (int k = 0; k < 3; ++k) {
    const double a = c.corner[k] - gbox[3 + k];
    const double b = gbox[k] - (c.corner[k] + c.side);
    double gap = a > b ? a : b;
    gap = gap > 0.0 ? gap : 0.0;
    d2 = k == 0 ? gap * gap : d2 + gap * gap;
  }
  return theta * theta * d2 > c.side * c.side;
}

// s^{-1/2}: v_rsq_f64 (about 2^-24 accurate) refined by one third-order
// Newton step y (1 + e/2 + 3e^2/8), e = 1 - s y^2, to double rounding.
__device__ __forceinline__ double rsqrt_tree(double s) {
  const double y = __builtin_amdgcn_rsq(s);
  const double e = fma(-(s * y), y, 1.0);
  return fma(y, e * fma(e, 0.375, 0.5), y);
}


__device__ __forceinline__ int wave_inclusive_sum(int v, int lane) {
  for (int d = 1; d < kGS; d <<= 1) {
    const int t = __shfl_up(v, d, kGS);
    if (lane >= d) v += t;
  }
  return v;
}

// What one lane of a wavefront has written, in LDS or memory, is read by
// others of the same wavefront after this.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
  __builtin_amdgcn_wave_barrier();
}

struct Accum {
  double a0, a1, a2, ph;
};

// One cell on the lane's particle.  In double the sums go straight into A; in
// mixed precision the separation from the centre of mass is formed in double
// and rounded, the rest of the term is float, and the float sums F of one
// chunk (64 cells of the list) are added into A at its end.
__device__ __forceinline__ void cell_term(const CellMomF& c, double x0, double x1, double x2, float e2, float* F) {
  const float y0 = (float)(x0 - c.X[0]), y1 = (float)(x1 - c.X[1]), y2 = (float)(x2 - c.X[2]);
  const float s = fmaf(y2, y2, fmaf(y1, y1, fmaf(y0, y0, e2)));
  const float q = __builtin_amdgcn_rsqf(s);
  const float q2 = q * q;
  const float q3 = q2 * q, q5 = q3 * q2;
  const float Qy0 = c.Q[0] * y0 + c.Q[3] * y1 + c.Q[4] * y2;
  const float Qy1 = c.Q[3] * y0 + c.Q[1] * y1 + c.Q[5] * y2;
  const float Qy2 = c.Q[4] * y0 + c.Q[5] * y1 + c.Q[2] * y2;
  const float w = (y0 * Qy0 + y1 * Qy1 + y2 * Qy2) * q5;  // (y.Qy) s^-5/2
  const float f = fmaf(-2.5f * w, q2, -c.M * q3);         // -M s^-3/2 - (5/2)(y.Qy) s^-7/2
  F[0] = fmaf(Qy0, q5, fmaf(f, y0, F[0]));
  F[1] = fmaf(Qy1, q5, fmaf(f, y1, F[1]));
  F[2] = fmaf(Qy2, q5, fmaf(f, y2, F[2]));
  F[3] = fmaf(-0.5f, w, fmaf(-c.M, q, F[3]));
}
__device__ __forceinline__ void cell_term(const CellMom& c, double x0, double x1, double x2, double e2, double* F) {
  const double y0 = x0 - c.X[0], y1 = x1 - c.X[1], y2 = x2 - c.X[2];
  const double s = fma(y2, y2, fma(y1, y1, fma(y0, y0, e2)));
  const double q = rsqrt_tree(s);
  const double q2 = q * q;
  const double q3 = q2 * q, q5 = q3 * q2;
  const double Qy0 = c.Q[0] * y0 + c.Q[3] * y1 + c.Q[4] * y2;
  const double Qy1 = c.Q[3] * y0 + c.Q[1] * y1 + c.Q[5] * y2;
  const double Qy2 = c.Q[4] * y0 + c.Q[5] * y1 + c.Q[2] * y2;
  const double w = (y0 * Qy0 + y1 * Qy1 + y2 * Qy2) * q5;  // (y.Qy) s^-5/2
  const double f = fma(-2.5 * w, q2, -c.M * q3);          // -M s^-3/2 - (5/2)(y.Qy) s^-7/2
  F[0] = fma(Qy0, q5, fma(f, y0, F[0]));
  F[1] = fma(Qy1, q5, fma(f, y1, F[1]));
  F[2] = fma(Qy2, q5, fma(f, y2, F[2]));
  F[3] = fma(-0.5, w, fma(-c.M, q, F[3]));
}

// One leaf particle on the lane's particle (itself and coincident ones are
// skipped).
__device__ __forceinline__ void part_term(const Part& p, bool self, double x0, double x1, double x2, float e2,
                                          float* F) {
  const float r0 = (float)(p.x[0] - x0), r1 = (float)(p.x[1] - x1), r2 = (float)(p.x[2] - x2);
  const float s = fmaf(r2, r2, fmaf(r1, r1, fmaf(r0, r0, e2)));
  const bool keep = !self && s > 0.0f;
  const float q = keep ? __builtin_amdgcn_rsqf(s) : 0.0f;
  const float mq = (float)p.m * q;
  const float mq3 = mq * q * q;
  F[0] += mq3 * r0;
  F[1] += mq3 * r1;
  F[2] += mq3 * r2;
  F[3] -= mq;
}
__device__ __forceinline__ void part_term(const Part& p, bool self, double x0, double x1, double x2, double e2,
                                          double* F) {
  const double r0 = p.x[0] - x0, r1 = p.x[1] - x1, r2 = p.x[2] - x2;
  const double s = fma(r2, r2, fma(r1, r1, fma(r0, r0, e2)));
  const bool keep = !self && s > 0.0;
  const double q = keep ? rsqrt_tree(s) : 0.0;
  const double mq = p.m * q;
  const double mq3 = mq * q * q;
  F[0] += mq3 * r0;
  F[1] += mq3 * r1;
  F[2] += mq3 * r2;
  F[3] -= mq;
}

template <bool MIXED>
struct Terms {
  using Mom = typename std::conditional<MIXED, CellMomF, CellMom>::type;
  using T = typename std::conditional<MIXED, float, double>::type;
};

// The sums of one chunk: in double the accumulators themselves.
template <bool MIXED>
__device__ __forceinline__ void chunk_open(const Accum& A, typename Terms<MIXED>::T* F) {
  if constexpr (MIXED) {
    F[0] = F[1] = F[2] = F[3] = 0.0f;
  } else {
    F[0] = A.a0; F[1] = A.a1; F[2] = A.a2; F[3] = A.ph;
  }
}
template <bool MIXED>
__device__ __forceinline__ void chunk_close(Accum& A, const typename Terms<MIXED>::T* F) {
  if constexpr (MIXED) {
    A.a0 += (double)F[0]; A.a1 += (double)F[1]; A.a2 += (double)F[2]; A.ph += (double)F[3];
  } else {
    A.a0 = F[0]; A.a1 = F[1]; A.a2 = F[2]; A.ph = F[3];
  }
}

// What a wavefront stages for evaluation: up to 64 cells or 64 leaf
// particles, never both at a time.
template <bool MIXED>
struct Stage {
  struct Parts {
    Part p[kGS];
    int32_t j[kGS];
  };
  union {
    typename Terms<MIXED>::Mom cell[kGS];
    Parts leaf;
  };
  int32_t begin[kGS], incl[kGS];
};

// The cnt (1 to 64) cells of a list: each lane stages one, then every lane
// adds all of them to its particle.
template <bool MIXED>
__device__ __forceinline__ void eval_cells(Stage<MIXED>& st, const int32_t* list, int cnt,
                                           const typename Terms<MIXED>::Mom* __restrict__ mom, double x0, double x1,
                                           double x2, double eps2, Accum& A, int lane) {
  using T = typename Terms<MIXED>::T;
  if (lane < cnt) st.cell[lane] = mom[list[lane]];
  wave_sync();
  const T e2 = (T)eps2;
  T F[4];
  chunk_open<MIXED>(A, F);
  for (int t = 0; t < cnt; ++t) cell_term(st.cell[t], x0, x1, x2, e2, F);
  chunk_close<MIXED>(A, F);
  wave_sync();
}

// The particles of the cnt (<= 64) leaves of a list, one leaf after another,
// in chunks of 64: this call evaluates chunks u0, u0 + ustep, ...  Lane p
// stages particle p of the chunk (found by a binary search over the leaves'
// prefix sums).
template <bool MIXED>
__device__ __forceinline__ void eval_leaves(Stage<MIXED>& st, const int32_t* list, int cnt,
                                            const TreeCell* __restrict__ cells, const Part* __restrict__ part,
                                            int32_t i, double x0, double x1, double x2, double eps2, Accum& A,
                                            int lane, int u0, int ustep) {
  using T = typename Terms<MIXED>::T;
  int size = 0, begin = 0;
  if (lane < cnt) {
    const TreeCell& c = cells[list[lane]];
    begin = c.begin;
    size = c.end - c.begin;
  }
  const int incl = wave_inclusive_sum(size, lane);
  const int total = __builtin_amdgcn_readlane(incl, kGS - 1);
  st.begin[lane] = begin;
  st.incl[lane] = incl;
  wave_sync();
  const T e2 = (T)eps2;
  for (int base = u0 * kGS; base < total; base += ustep * kGS) {
    const int f = base + lane;
    if (f < total) {
      // the first leaf k whose prefix sum exceeds f
      int lo = 0, hi = cnt - 1;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (st.incl[mid] > f) hi = mid;
        else lo = mid + 1;
      }
      const int32_t j = st.begin[lo] + (f - (lo > 0 ? st.incl[lo - 1] : 0));
      st.leaf.p[lane] = part[j];
      st.leaf.j[lane] = j;
    }
    wave_sync();
    const int m = total - base < kGS ? total - base : kGS;
    T F[4];
    chunk_open<MIXED>(A, F);
#pragma unroll 4
    for (int t = 0; t < m; ++t) part_term(st.leaf.p[t], st.leaf.j[t] == i, x0, x1, x2, e2, F);
    chunk_close<MIXED>(A, F);
    wave_sync();
  }
}

// drop the first 64 entries of a list of n (64 <= n < 128)
__device__ __forceinline__ void shift_list(int32_t* list, int n, int lane) {
  const int32_t v = lane + kGS < n ? list[lane + kGS] : 0;
  wave_sync();
  if (lane + kGS < n) list[lane] = v;
  wave_sync();
}

// The stack of a walk: its first LDS entries in LDS, the rest in memory.
template <int LDS>
struct Stack {
  int32_t* near_;
  int32_t* far_;
  __device__ __forceinline__ int32_t get(int k) const {
    if constexpr (LDS > 0) return k < LDS ? near_[k] : far_[k];
    else return far_[k];
  }
  __device__ __forceinline__ void put(int k, int32_t v) const {
    if constexpr (LDS > 0) {
      if (k < LDS) near_[k] = v;
      else far_[k] = v;
    } else {
      far_[k] = v;
    }
  }
};

// One step of a walk by one wavefront.  Returns false when the push does not
// fit the stack.
template <int LDS>
__device__ __forceinline__ bool walk_step(const Stack<LDS>& stack, int& sp, int32_t stack_cap, int32_t* acc_list,
                                          int& n_acc, int32_t* leaf_list, int& n_leaf,
                                          const TreeCell* __restrict__ cells, const double* box, double theta,
                                          int lane) {
  const int k = sp < kGS ? sp : kGS;
  const int base = sp - k;
  int kind = 3, nch = 0, ch0 = 0;
  int32_t cid = 0;
  if (lane < k) {
    cid = stack.get(base + lane);
    const TreeCell c = cells[cid];
    if (accepted(c, box, theta)) {
      kind = 0;
    } else if (c.child0 < 0) {
      kind = 1;
    } else {
      kind = 2;
      ch0 = c.child0;
      nch = c.child1 - ch0;
    }
  }
  sp = base;
  const uint64_t ma = __ballot(kind == 0), ml = __ballot(kind == 1);
  if (kind == 0) acc_list[n_acc + lane_rank(ma)] = cid;
  if (kind == 1) leaf_list[n_leaf + lane_rank(ml)] = cid;
  n_acc += __popcll(ma);
  n_leaf += __popcll(ml);
  // where each lane's children go: the prefix of nch (0 to 8) over the lanes,
  // bit by bit from ballots
  int before = 0, pushed = 0;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const uint64_t m = __ballot((nch >> b) & 1);
    before += lane_rank(m) << b;
    pushed += __popcll(m) << b;
  }
  if (sp + pushed > stack_cap) return false;
  for (int t = 0; t < nch; ++t) stack.put(sp + before + t, ch0 + t);
  sp += pushed;
  wave_sync();
  return true;
}

struct WalkArgs {
  const int32_t* gb;
  const int32_t* ge;
  const int32_t* ngroups;
  const double* gbox;
  const TreeCell* cells;
  const void* mom;            // CellMom or CellMomF [cells]
  const Part* part;
  const int32_t* idx;         // input row of each particle
  double theta, eps2;
  int32_t* stack;             // stack_cap entries per workgroup
  int32_t stack_cap;
  unsigned int* wq;           // work queue (work_queue.h)
  unsigned long long* ctr;    // kCtrLine words per XCD: accepted pairs, opened pairs, stack overflow; null: not counted
  unsigned int* err;
  double* acc;
  double* pot;
};
constexpr int kCtrLine = 32;  // 64-bit words between the XCDs' counters
static_assert(kCtrLine * kXcd == kCtrWords, "counter buffer");

__device__ __forceinline__ void walk_count(const WalkArgs& a, unsigned long long acc, unsigned long long leaf,
                                           bool overflow) {
  if (a.ctr) {
    unsigned long long* c = a.ctr + (blockIdx.x % kXcd) * kCtrLine;
    atomicAdd(&c[0], acc);
    atomicAdd(&c[1], leaf);
    if (overflow) atomicOr(&c[2], 1ull);
  }
  if (overflow && a.err) atomicOr(a.err, kErrTreeStack);
}

// Many groups: one wavefront per workgroup, each walking and evaluating the
// groups it takes from the work queue, dealt to the XCDs in turn along the
// curve (groups in dense regions cost several times the others).
template <bool MIXED>
__global__ __launch_bounds__(kGS) void k_tree_walk_forces(WalkArgs a) {
  __shared__ Stage<MIXED> stage;
  __shared__ int32_t acc_list[2 * kGS], leaf_list[2 * kGS];
  __shared__ unsigned int slot;
  using Mom = typename Terms<MIXED>::Mom;
  const TreeCell* __restrict__ cells = a.cells;
  const Mom* __restrict__ mom = static_cast<const Mom*>(a.mom);
  const Part* __restrict__ part = a.part;
  const int lane = threadIdx.x;
  const int64_t ngroups = *a.ngroups;
  const Stack<0> stack{nullptr, a.stack + (int64_t)blockIdx.x * a.stack_cap};
  const int32_t root_child0 = cells[0].child0, root_nchild = cells[0].child1 - root_child0;
  unsigned long long tot_acc = 0, tot_leaf = 0;
  bool overflow = false;
  if (!queue_member(ngroups)) return;
  int64_t w = queue_first(a.wq, ngroups);
  while (w < ngroups) {
    const int64_t g = interleaved(w, ngroups);
    const int32_t b = a.gb[g], e = a.ge[g];
    const int32_t i = b + lane;
    const bool valid = i < e;
    const int32_t ir = valid ? i : b;
    const double x0 = part[ir].x[0], x1 = part[ir].x[1], x2 = part[ir].x[2];
    double box[6];
    for (int k = 0; k < 6; ++k) box[k] = a.gbox[6 * g + k];
    Accum A{0.0, 0.0, 0.0, 0.0};
    // the root is never accepted: the walk starts from its children, or
    // opens it when it is a leaf
    int sp = 0, n_acc = 0, n_leaf = 0;
    bool fits = true;
    if (root_nchild > 0) {
      if (lane < root_nchild) stack.put(lane, root_child0 + lane);
      sp = root_nchild;
    } else {
      if (lane == 0) leaf_list[0] = 0;
      n_leaf = 1;
    }
    wave_sync();
    while (sp > 0) {
      fits = walk_step<0>(stack, sp, a.stack_cap, acc_list, n_acc, leaf_list, n_leaf, cells, box, a.theta, lane);
      if (!fits) break;
      if (n_acc >= kGS) {
        eval_cells<MIXED>(stage, acc_list, kGS, mom, x0, x1, x2, a.eps2, A, lane);
        shift_list(acc_list, n_acc, lane);
        n_acc -= kGS;
        tot_acc += kGS;
      }
      if (n_leaf >= kGS) {
        eval_leaves<MIXED>(stage, leaf_list, kGS, cells, part, i, x0, x1, x2, a.eps2, A, lane, 0, 1);
        shift_list(leaf_list, n_leaf, lane);
        n_leaf -= kGS;
        tot_leaf += kGS;
      }
    }
    if (fits) {
      if (n_acc > 0) eval_cells<MIXED>(stage, acc_list, n_acc, mom, x0, x1, x2, a.eps2, A, lane);
      if (n_leaf > 0) eval_leaves<MIXED>(stage, leaf_list, n_leaf, cells, part, i, x0, x1, x2, a.eps2, A, lane, 0, 1);
      tot_acc += n_acc;
      tot_leaf += n_leaf;
      if (valid) {
        const int64_t o = a.idx[i];
        a.acc[3 * o] = A.a0;
        a.acc[3 * o + 1] = A.a1;
        a.acc[3 * o + 2] = A.a2;
        a.pot[o] = A.ph;
      }
    }
    overflow |= !fits;
    wave_sync();
    w = queue_next(a.wq, slot, ngroups, w + gridDim.x);
  }
  if (lane == 0 && (a.ctr || overflow)) walk_count(a, tot_acc, tot_leaf, overflow);
  queue_done(a.wq, ngroups);
}

// Few groups (they leave most of the chip idle at one wavefront each): a team
// of kTeam wavefronts per group.  Wavefront 0 walks, with its stack in LDS,
// and fills one of two pairs of lists; the others meanwhile evaluate the pair
// of the round before, the list's chunks dealt to them in turn, each in the
// composition a single wavefront would give it; when the walk has ended all
// evaluate the last pair.  The partial sums are added in wavefront order.
// Up to kTeamChunks chunks of 64 per compute unit (131072 particles on 256):
// whole evaluations in us, one wavefront per group and teams, double / mixed:
// 10007: 562 / 500 and 255 / 219; 65536: 924 / 823 and 734 / 578; 131072: 1366 /
// 1062 and 1251 / 1016; 262144: 2310 / 1625 and 2354 / 1886 (MI355X).
constexpr int kTeamChunks = 8;
constexpr int kTeam = 8;
constexpr int kTeamStack = 2048;                  // stack entries in LDS
constexpr int kTeamCells = 8 * kGS, kTeamLeaves = 2 * kGS;  // list lengths that end a round

template <bool MIXED>
__global__ __launch_bounds__(kTeam * kGS) void k_tree_walk_team(WalkArgs a) {
  __shared__ int32_t near_[kTeamStack];
  __shared__ int32_t acc_list[2][kTeamCells + kGS], leaf_list[2][kTeamLeaves + kGS];
  __shared__ int count[2][2];  // entries to evaluate of each list pair
  __shared__ int done_s[2];
  __shared__ Stage<MIXED> stage[kTeam];
  __shared__ unsigned int slot;
  // the sums of each wavefront, at the end, in the staging space
  static_assert(sizeof(stage) >= kTeam * 4 * kGS * sizeof(double), "partial sums");
  double (*red)[4][kGS] = reinterpret_cast<double (*)[4][kGS]>(&stage);
  using Mom = typename Terms<MIXED>::Mom;
  const TreeCell* __restrict__ cells = a.cells;
  const Mom* __restrict__ mom = static_cast<const Mom*>(a.mom);
  const Part* __restrict__ part = a.part;
  const int lane = threadIdx.x & (kGS - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kGS);
  const int64_t ngroups = *a.ngroups;
  const Stack<kTeamStack> stack{near_, a.stack + (int64_t)blockIdx.x * a.stack_cap};
  const int32_t root_child0 = cells[0].child0, root_nchild = cells[0].child1 - root_child0;
  unsigned long long tot_acc = 0, tot_leaf = 0;
  bool overflow = false;
  if (!queue_member(ngroups)) return;
  if (threadIdx.x < 2) done_s[threadIdx.x] = 0;
  __syncthreads();
  int64_t w = queue_first(a.wq, ngroups);
  while (w < ngroups) {
    const int64_t g = interleaved(w, ngroups);
    const int32_t b = a.gb[g], e = a.ge[g];
    const int32_t i = b + lane;
    const bool valid = i < e;
    const int32_t ir = valid ? i : b;
    const double x0 = part[ir].x[0], x1 = part[ir].x[1], x2 = part[ir].x[2];
    double box[6];
    for (int k = 0; k < 6; ++k) box[k] = a.gbox[6 * g + k];
    Accum A{0.0, 0.0, 0.0, 0.0};
    // the walk's state, kept by wavefront 0: entries carried over from the
    // previous round (its last, partial chunks) come first in the new lists
    int sp = 0, n_acc = 0, n_leaf = 0;
    bool fits = true;
    if (wave == 0) {
      if (root_nchild > 0) {
        if (lane < root_nchild) stack.put(lane, root_child0 + lane);
        sp = root_nchild;
      } else {
        if (lane == 0) leaf_list[0][0] = 0;
        n_leaf = 1;
      }
      wave_sync();
    }
    bool done = false;
    for (int r = 0;; ++r) {
      const int cur = r & 1, prev = cur ^ 1;
      if (!done && wave == 0) {
        int32_t* al = acc_list[cur];
        int32_t* ll = leaf_list[cur];
        while (sp > 0 && n_acc < kTeamCells && n_leaf < kTeamLeaves) {
          fits = walk_step<kTeamStack>(stack, sp, a.stack_cap, al, n_acc, ll, n_leaf, cells, box, a.theta, lane);
          if (!fits) break;
        }
        const bool end = sp == 0 || !fits;
        const int ea = end ? n_acc : n_acc & ~(kGS - 1), el = end ? n_leaf : n_leaf & ~(kGS - 1);
        if (lane == 0) {
          count[cur][0] = ea;
          count[cur][1] = el;
          done_s[cur] = end ? (fits ? 1 : 2) : 0;
        }
        tot_acc += ea;
        tot_leaf += el;
        // the rest goes to the other lists once the team has read them
        n_acc -= ea;
        n_leaf -= el;
      } else if (r > 0) {
        const int first = done ? wave : wave - 1, step = done ? kTeam : kTeam - 1;
        const int ea = count[prev][0], el = count[prev][1];
        for (int u = first; u * kGS < ea; u += step)
          eval_cells<MIXED>(stage[wave], acc_list[prev] + u * kGS, ea - u * kGS < kGS ? ea - u * kGS : kGS, mom, x0, x1, x2,
                            a.eps2, A, lane);
        for (int u = 0; u * kGS < el; ++u)
          eval_leaves<MIXED>(stage[wave], leaf_list[prev] + u * kGS, el - u * kGS < kGS ? el - u * kGS : kGS, cells, part, i, x0,
                             x1, x2, a.eps2, A, lane, first, step);
      }
      __syncthreads();
      if (done) break;
      const int end = done_s[cur];
      done = end != 0;
      if (end == 2) break;  // the stack overflowed: the group is not written
      if (!done && wave == 0) {
        // the team is done with the other lists; entries carry over to them
        const int ea = count[cur][0], el = count[cur][1];
        if (lane < n_acc) acc_list[prev][lane] = acc_list[cur][ea + lane];
        if (lane < n_leaf) leaf_list[prev][lane] = leaf_list[cur][el + lane];
        wave_sync();
      }
    }
    const bool group_fits = done_s[0] != 2 && done_s[1] != 2;
    __syncthreads();  // every wavefront has finished with the staging space
    red[wave][0][lane] = A.a0;
    red[wave][1][lane] = A.a1;
    red[wave][2][lane] = A.a2;
    red[wave][3][lane] = A.ph;
    __syncthreads();
    if (wave < 4 && valid && group_fits) {
      double v = red[0][wave][lane];
      for (int u = 1; u < kTeam; ++u) v += red[u][wave][lane];
      const int64_t o = a.idx[i];
      if (wave < 3) a.acc[3 * o + wave] = v;
      else a.pot[o] = v;
    }
    overflow |= !group_fits;
    if (threadIdx.x < 2) done_s[threadIdx.x] = 0;
    __syncthreads();
    w = queue_next(a.wq, slot, ngroups, w + gridDim.x);
  }
  if (threadIdx.x == 0 && (a.ctr || overflow)) walk_count(a, tot_acc, tot_leaf, overflow);
  queue_done(a.wq, ngroups);
}

// ------------------------------------------------------------ rank sort -----
// Few particles: a key's place is the number of keys before it (smaller, or
// equal with a smaller row), counted directly.  A block counts for 64 keys, one
// per lane; its sixteen wavefronts each compare a sixteenth of all keys, read at a
// wave-uniform index through the scalar cache.  n^2 / 64 wavefront steps of a
// compare and an add-with-carry, one launch: 10007 keys take 21 us, where the
// 24 launches of eight radix passes took 140.  The line lies where the count
// still wins: whole evaluations of 16384 particles (counted) and 16385 (16
// launches of radix passes) take 295 and 342 us in double, 245 and 310 mixed.
constexpr int kRankThreads = 1024;
constexpr int32_t kRankMax = 16384;

using ConstKey = const __attribute__((address_space(4))) uint64_t;  // not written while the kernel runs

// Keys of [lo, hi) below ki, or not above it: sixteen keys are on their way
// while the sixteen before them are compared.
template <bool EQUAL>
__device__ __forceinline__ int32_t count_below(ConstKey* k, int32_t lo, int32_t hi, uint64_t ki) {
  constexpr int B = 16;
  int32_t cnt = 0, j = lo;
  if (hi - lo >= B) {
    uint64_t nxt[B];
#pragma unroll
    for (int u = 0; u < B; ++u) nxt[u] = k[j + u];
    for (; j + B <= hi; j += B) {
      uint64_t cur[B];
      const int32_t jn = j + 2 * B <= hi ? j + B : lo;
#pragma unroll
      for (int u = 0; u < B; ++u) cur[u] = nxt[u];
#pragma unroll
      for (int u = 0; u < B; ++u) nxt[u] = k[jn + u];
#pragma unroll
      for (int u = 0; u < B; ++u) cnt += (EQUAL ? cur[u] <= ki : cur[u] < ki) ? 1 : 0;
    }
  }
  for (; j < hi; ++j) cnt += (EQUAL ? k[j] <= ki : k[j] < ki) ? 1 : 0;
  return cnt;
}

__global__ __launch_bounds__(kRankThreads) void k_rank_sort(const uint64_t* __restrict__ keys, int32_t n,
                                                            uint64_t* __restrict__ keys_s,
                                                            int32_t* __restrict__ idx_s) {
  constexpr int W = kRankThreads / 64;
  __shared__ int32_t before[W][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t i0 = (int32_t)blockIdx.x * 64, i = i0 + lane;
  const uint64_t ki = i < n ? keys[i] : ~0ull;
  ConstKey* k = (ConstKey*)(uintptr_t)keys;
  const int32_t len = (n + W - 1) / W;
  const int32_t lo = wave * len < n ? wave * len : n, hi = n - lo < len ? n : lo + len;
  const int32_t a1 = hi < i0 ? hi : i0;                       // [lo, a1): rows before the block's
  const int32_t b0 = lo > i0 ? lo : i0;                       // [b0, b1): the block's own rows
  const int32_t b1 = hi < i0 + 64 ? hi : i0 + 64;
  const int32_t c0 = lo > i0 + 64 ? lo : i0 + 64;             // [c0, hi): rows after them
  int32_t cnt = count_below<true>(k, lo, a1, ki) + count_below<false>(k, c0, hi, ki);
  for (int32_t j = b0; j < b1; ++j) cnt += (k[j] < ki || (k[j] == ki && j < i)) ? 1 : 0;
  before[wave][lane] = cnt;
  __syncthreads();
  if (wave == 0 && i < n) {
    int32_t r = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) r += before[w][lane];
    keys_s[r] = ki;
    idx_s[r] = i;
  }
}

// ----------------------------------------------------------- radix sort -----
// Stable least-significant-digit radix sort of (key, row) pairs, 8 bits per
// pass.  A pass: each tile of kRsTile keys counts its digits (k_rs_hist); the
// counts of the tiles before it plus the prefix of the digit totals give every
// (digit, tile) its first output slot; each tile then writes its keys there
// (k_rs_scatter), a key's place among the equal digits of its tile being
// the number of such keys before it.  Up to kRsDirect tiles each scatter block
// adds up the other tiles' counts itself (128 tiles: 128 KB from the L2);
// above, a kernel of its own scans each digit's row (k_rs_rowscan, one block
// per digit).  Within a tile, wavefront w takes the w-th eighth in rounds of 64
// consecutive keys; the lanes of a round that share a digit find each other
// with eight ballots (one per digit bit), and a per-wavefront count of each
// digit carries over between rounds, so the order among equal digits is the
// input order.
constexpr int kRsBits = 8;
constexpr int kRsBuckets = 1 << kRsBits;
constexpr int kRsThreads = 512;
constexpr int kRsWaves = kRsThreads / 64;
constexpr int kRsRounds = 4;                          // rounds of 64 keys per wavefront
constexpr int kRsTile = kRsWaves * 64 * kRsRounds;    // 2048 keys per tile
constexpr int32_t kRsDirect = 128;
static_assert(2 * kRsBuckets == kRsThreads, "two threads per digit in the tile tables");

// Counts of tile b: hist[b][digit] (direct) or hist[digit][b] (row scan).
__global__ __launch_bounds__(kRsThreads) void k_rs_hist(const uint64_t* __restrict__ keys, int32_t n, int shift,
                                                        int32_t* __restrict__ hist, int32_t ntile) {
  __shared__ int32_t h[kRsBuckets];
  const int t = threadIdx.x;
  if (t < kRsBuckets) h[t] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kRsTile;
#pragma unroll
  for (int r = 0; r < kRsTile / kRsThreads; ++r) {
    const int64_t i = base + r * kRsThreads + t;
    if (i < n) atomicAdd(&h[(keys[i] >> shift) & (kRsBuckets - 1)], 1);
  }
  __syncthreads();
  if (t < kRsBuckets) {
    if (ntile <= kRsDirect) hist[(int64_t)blockIdx.x * kRsBuckets + t] = h[t];
    else hist[(int64_t)t * ntile + blockIdx.x] = h[t];
  }
}

// Per digit (block d): the exclusive prefix of its row of tile counts, in
// place (the tile's place among the digit's keys), and the row total.
constexpr int kRowThreads = 256;
__global__ __launch_bounds__(kRowThreads) void k_rs_rowscan(int32_t* __restrict__ hist, int32_t ntile,
                                                            int32_t* __restrict__ total) {
  __shared__ int32_t wsum[2][kRowThreads / 64];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int32_t* row = hist + (int64_t)blockIdx.x * ntile;
  int32_t carry = 0;
  int buf = 0;
  for (int64_t c0 = 0; c0 < ntile; c0 += kRowThreads) {
    const int64_t k = c0 + t;
    const int32_t v = k < ntile ? row[k] : 0;
    const int32_t x = wave_inclusive_sum(v, lane);
    if (lane == 63) wsum[buf][wave] = x;
    __syncthreads();  // the totals alternate between two buffers: one barrier per round
    int32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kRowThreads / 64; ++w) {
      before += w < wave ? wsum[buf][w] : 0;
      all += wsum[buf][w];
    }
    if (k < ntile) row[k] = carry + before + x - v;
    carry += all;
    buf ^= 1;
  }
  if (t == 0) total[blockIdx.x] = carry;
}

__global__ __launch_bounds__(kRsThreads) void k_rs_scatter(const uint64_t* __restrict__ kin,
                                                           const int32_t* __restrict__ vin,
                                                           uint64_t* __restrict__ kout, int32_t* __restrict__ vout,
                                                           int32_t n, int shift, const int32_t* __restrict__ hist,
                                                           const int32_t* __restrict__ total, int32_t ntile) {
  __shared__ int32_t first[kRsBuckets];          // the tile's first output slot of each digit
  __shared__ int32_t wcnt[kRsWaves][kRsBuckets];
  __shared__ int32_t half[2][kRsBuckets];        // direct: the second halves' sums
  __shared__ int32_t wsum[kRsBuckets / 64];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  // the keys are on their way while the tables are summed
  const int64_t base = (int64_t)blockIdx.x * kRsTile + (int64_t)w * 64 * kRsRounds;
  uint64_t key[kRsRounds];
  int32_t val[kRsRounds], rank[kRsRounds];
#pragma unroll
  for (int r = 0; r < kRsRounds; ++r) {
    const int64_t i = base + r * 64 + lane;
    key[r] = i < n ? kin[i] : 0ull;
    val[r] = i < n ? vin[i] : 0;
  }
  // keys of digit d in the tiles before this one (pre) and in all (tot)
  const int d = t & (kRsBuckets - 1);
  int32_t pre = 0, tot = 0;
  if (ntile <= kRsDirect) {
    const int h = t / kRsBuckets;
#pragma unroll 16
    for (int32_t q = h; q < ntile; q += 2) {
      const int32_t c = hist[(int64_t)q * kRsBuckets + d];
      tot += c;
      pre += q < (int32_t)blockIdx.x ? c : 0;
    }
    if (h == 1) {
      half[0][d] = pre;
      half[1][d] = tot;
    }
  } else if (t < kRsBuckets) {
    pre = hist[(int64_t)d * ntile + blockIdx.x];
    tot = total[d];
  }
  for (int q = t; q < kRsWaves * kRsBuckets; q += kRsThreads) (&wcnt[0][0])[q] = 0;
  __syncthreads();
  if (ntile <= kRsDirect && t < kRsBuckets) {
    pre += half[0][d];
    tot += half[1][d];
  }
  // where each digit starts: the exclusive prefix of the digit totals
  const int32_t x = wave_inclusive_sum(t < kRsBuckets ? tot : 0, lane);
  if (t < kRsBuckets && lane == 63) wsum[w] = x;
  __syncthreads();
  if (t < kRsBuckets) {
    int32_t at = x - tot;
    for (int q = 0; q < w; ++q) at += wsum[q];
    first[t] = at + pre;
  }
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int r = 0; r < kRsRounds; ++r) {
    const bool valid = base + r * 64 + lane < n;
    const int dig = (int)((key[r] >> shift) & (kRsBuckets - 1));
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < kRsBits; ++b) {
      const bool bit = (dig >> b) & 1;
      const uint64_t m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    const int before = __popcll(peers & below);
    const int run = valid ? wcnt[w][dig] : 0;
    rank[r] = run + before;
    if (valid && before == 0) wcnt[w][dig] = run + __popcll(peers);  // the group's first lane
  }
  __syncthreads();
  // per digit, where each wavefront's keys start within the tile
  if (t < kRsBuckets) {
    int32_t acc = first[t];
#pragma unroll
    for (int q = 0; q < kRsWaves; ++q) {
      const int32_t c = wcnt[q][t];
      wcnt[q][t] = acc;
      acc += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRsRounds; ++r) {
    if (base + r * 64 + lane < n) {
      const int32_t dst = wcnt[w][(key[r] >> shift) & (kRsBuckets - 1)] + rank[r];
      kout[dst] = key[r];
      vout[dst] = val[r];
    }
  }
}

// ------------------------------------------------------- host helpers -----
struct Alloc {
  TreeScratch& s;
  hipStream_t st;
  bool capturing;
  hipError_t err = hipSuccess;
  template <class T>
  T* get(int slot, int64_t count) {
    if (err != hipSuccess) return nullptr;
    const size_t bytes = (size_t)(count > 0 ? count : 1) * sizeof(T);
    if ((int)s.slots.size() <= slot) {
      if (capturing) {
        err = hipErrorStreamCaptureUnsupported;
        return nullptr;
      }
      s.slots.resize(slot + 1, {nullptr, 0});
    }
    auto& sl = s.slots[slot];
    if (sl.second < bytes) {
      if (capturing) {  // no allocation inside a capture: a call outside it sizes the buffers
        err = hipErrorStreamCaptureUnsupported;
        return nullptr;
      }
      if (sl.first) {
        (void)hipStreamSynchronize(st);
        (void)hipFree(sl.first);
        sl.first = nullptr;
        sl.second = 0;
      }
      const size_t cap = bytes + bytes / 4;
      err = hipMalloc(&sl.first, cap);
      if (err != hipSuccess) return nullptr;
      sl.second = cap;
    }
    return static_cast<T*>(sl.first);
  }
};

enum Slot {
  S_BOXPART, S_BOX, S_KEYS, S_KEYS2, S_IDX, S_IDX2, S_PART, S_MOM, S_SPAN, S_CELLS, S_CNT,
  S_GB, S_GE, S_GBOX, S_STACK, S_COUNTS, S_HIST, S_TILE
};

// Sort (keys, idx) by the low `bits` bits of the keys; returns the buffers
// holding the result (the inputs or the alternates, which are overwritten).
hipError_t radix_sort(Alloc& al, uint64_t* keys, int32_t* idx, uint64_t* keys2, int32_t* idx2, int32_t n, int bits,
                      uint64_t** keys_out, int32_t** idx_out) {
  const int32_t ntile = (n + kRsTile - 1) / kRsTile;
  int32_t* hist = al.get<int32_t>(S_HIST, (int64_t)kRsBuckets * ntile + kRsBuckets);
  if (!hist) return al.err != hipSuccess ? al.err : hipErrorOutOfMemory;
  int32_t* total = hist + (int64_t)kRsBuckets * ntile;
  uint64_t *ka = keys, *kb = keys2;
  int32_t *va = idx, *vb = idx2;
  for (int shift = 0; shift < bits; shift += kRsBits) {
    hipLaunchKernelGGL(k_rs_hist, dim3(ntile), dim3(kRsThreads), 0, al.st, ka, n, shift, hist, ntile);
    if (ntile > kRsDirect)
      hipLaunchKernelGGL(k_rs_rowscan, dim3(kRsBuckets), dim3(kRowThreads), 0, al.st, hist, ntile, total);
    hipLaunchKernelGGL(k_rs_scatter, dim3(ntile), dim3(kRsThreads), 0, al.st, ka, va, kb, vb, n, shift, hist, total,
                       ntile);
    std::swap(ka, kb);
    std::swap(va, vb);
  }
  *keys_out = ka;
  *idx_out = va;
  return hipGetLastError();
}

}  // namespace

#define NB_TRY(x)                 \
  do {                            \
    hipError_t e_ = (x);          \
    if (e_ != hipSuccess) {       \
      *msg = #x;                  \
      return e_;                  \
    }                             \
  } while (0)

namespace {

// box, keys, the sort along the curve; sorted keys and rows go to *keys_s, *idx_s
hipError_t keys_and_order(Alloc& al, const double* pos, int32_t n, Box** box_out, uint64_t** keys_s,
                          int32_t** idx_s, const char** msg) {
  auto need = [&](void* p) -> hipError_t { return p ? hipSuccess : (al.err != hipSuccess ? al.err : hipErrorOutOfMemory); };
  const int nbb = blocks_for(n, 1024);
  double* part = al.get<double>(S_BOXPART, 6 * nbb);
  Box* box = al.get<Box>(S_BOX, 1);
  uint64_t* keys = al.get<uint64_t>(S_KEYS, n);
  uint64_t* keys2 = al.get<uint64_t>(S_KEYS2, n);
  int32_t* idx = al.get<int32_t>(S_IDX, n);
  int32_t* idx2 = al.get<int32_t>(S_IDX2, n);
  NB_TRY(need(idx2));
  const bool by_rank = n <= kRankMax;
  hipLaunchKernelGGL(k_bbox_partial, dim3(nbb), dim3(kTB), 0, al.st, pos, (int64_t)n, part);
  hipLaunchKernelGGL(k_keys, dim3(blocks_for(n)), dim3(kTB), 0, al.st, pos, (int64_t)n, part, nbb, box, keys,
                     by_rank ? nullptr : idx);
  NB_TRY(hipGetLastError());
  if (by_rank) {
    hipLaunchKernelGGL(k_rank_sort, dim3((n + 63) / 64), dim3(kRankThreads), 0, al.st, keys, n, keys2, idx2);
    NB_TRY(hipGetLastError());
    *keys_s = keys2;
    *idx_s = idx2;
  } else {
    NB_TRY(radix_sort(al, keys, idx, keys2, idx2, n, 3 * kBits, keys_s, idx_s));
  }
  *box_out = box;
  return hipSuccess;
}

}  // namespace

hipError_t tree_sorted_keys(TreeScratch& s, hipStream_t st, const double* pos, int32_t n, uint64_t* keys_out,
                            int32_t* idx_out, const char** msg) {
  *msg = "";
  Alloc al{s, st, false};
  Box* box = nullptr;
  uint64_t* keys_s = nullptr;
  int32_t* idx_s = nullptr;
  hipError_t e = keys_and_order(al, pos, n, &box, &keys_s, &idx_s, msg);
  if (e != hipSuccess) return e;
  NB_TRY(hipMemcpyAsync(keys_out, keys_s, (size_t)n * sizeof(uint64_t), hipMemcpyDeviceToDevice, st));
  NB_TRY(hipMemcpyAsync(idx_out, idx_s, (size_t)n * sizeof(int32_t), hipMemcpyDeviceToDevice, st));
  return hipSuccess;
}

hipError_t tree_forces_run(TreeScratch& s, hipStream_t st, const double* pos, const double* mass, int32_t n,
                           double eps2, double theta, int n_crit, double g_frac, bool mixed, double* acc,
                           double* pot, TreeStats* stats, bool capturing, unsigned int* wq, unsigned int* err,
                           const char** msg) {
  *msg = "";
  if (!capturing && !s.host) NB_TRY(hipHostMalloc(&s.host, sizeof(Counts), hipHostMallocDefault));
  Alloc al{s, st, capturing};
  auto need = [&](void* p) -> hipError_t { return p ? hipSuccess : (al.err != hipSuccess ? al.err : hipErrorOutOfMemory); };

  // box, keys, sort along the curve
  Box* box = nullptr;
  uint64_t* keys_s = nullptr;
  int32_t* idx_s = nullptr;
  {
    hipError_t e = keys_and_order(al, pos, n, &box, &keys_s, &idx_s, msg);
    if (e != hipSuccess) return e;
  }
  Part* part = al.get<Part>(S_PART, n);
  // cells, sized by a bound: a cell that splits holds more than n_crit
  // particles and the cells of one level are disjoint, so each level has at
  // most n / (n_crit + 1) of them; the leaves hold at least one particle each,
  // so there are at most n.
  const int64_t inner = n / ((int64_t)n_crit + 1);
  const int64_t cap_cells = 1 + (int64_t)kLevels * inner + n;
  TreeCell* cells = al.get<TreeCell>(S_CELLS, cap_cells);
  CellMom* mom = al.get<CellMom>(S_MOM, cap_cells);  // or CellMomF, which is smaller
  CellMomF* momf = mixed ? reinterpret_cast<CellMomF*>(mom) : nullptr;
  uint16_t* span = al.get<uint16_t>(S_SPAN, n);
  const int32_t ntile = (n + kTB - 1) / kTB;
  int32_t* cnt = al.get<int32_t>(S_CNT, (int64_t)kRows * ntile + kRows);
  TileMoments* tiles = al.get<TileMoments>(S_TILE, ntile);
  const int32_t nchunk = (n + kGS - 1) / kGS;
  int32_t* gb = al.get<int32_t>(S_GB, n);
  int32_t* ge = al.get<int32_t>(S_GE, n);
  double* gbox = al.get<double>(S_GBOX, 6 * (int64_t)n);
  Counts* counts = al.get<Counts>(S_COUNTS, 1);
  NB_TRY(need(counts));
  unsigned long long* ctr = counts->ctr;  // device addresses
  int32_t *lvl = counts->lvl, *gn = &counts->ngroups;
  int32_t* total = cnt + (int64_t)kRows * ntile;
  hipLaunchKernelGGL(k_cell_starts, dim3(ntile), dim3(kTB), 0, st, keys_s, idx_s, pos, mass, n, n_crit, box, g_frac,
                     part, span, cnt, ntile, tiles);
  hipLaunchKernelGGL(k_level_scan, dim3(kRows), dim3(1024), 0, st, cnt, ntile, total, ctr);
  hipLaunchKernelGGL(k_write_cells, dim3(ntile), dim3(kTB), 0, st, cells, span, cnt, total, ntile, n, part,
                     box, g_frac, lvl, gb, ge, gbox, gn);
  hipLaunchKernelGGL(k_cell_moments, dim3((unsigned)std::min<int64_t>(1024, cap_cells)), dim3(kTB), 0, st, cells, mom,
                     momf, lvl, part, tiles);
  NB_TRY(hipGetLastError());

  // walk and forces: a team per group while the groups are few, else one
  // wavefront per group
  int dev = 0, num_cus = 0, per_cu = 0;
  NB_TRY(hipGetDevice(&dev));
  NB_TRY(hipDeviceGetAttribute(&num_cus, hipDeviceAttributeMultiprocessorCount, dev));
  if (num_cus < 1) num_cus = 1;
  const bool team = nchunk <= kTeamChunks * num_cus;
  using WalkFn = void (*)(WalkArgs);
  const WalkFn fn = team ? (mixed ? k_tree_walk_team<true> : k_tree_walk_team<false>)
                         : (mixed ? k_tree_walk_forces<true> : k_tree_walk_forces<false>);
  const int wg = team ? kTeam * kGS : kGS;
  NB_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(fn), wg, 0));
  int64_t grid = (int64_t)num_cus * (per_cu > 0 ? per_cu : 1);
  // a chunk of 64 rarely splits into more than two groups, so more workgroups
  // would mostly find none
  if (grid > 2 * (int64_t)nchunk) grid = 2 * (int64_t)nchunk;
  const int32_t cap = (int32_t)(cap_cells < kStackCap ? cap_cells : kStackCap);
  int32_t* stack = al.get<int32_t>(S_STACK, grid * cap);
  NB_TRY(need(stack));
  const WalkArgs wa{gb, ge, gn, gbox, cells, mom, part, idx_s, theta, eps2, stack, cap, wq, stats ? ctr : nullptr,
                    err, acc, pot};
  hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(wg), 0, st, wa);
  NB_TRY(hipGetLastError());
  if (!stats) return hipSuccess;
  // counts for the caller (synchronises)
  Counts* h = static_cast<Counts*>(s.host);
  NB_TRY(hipMemcpyAsync(h, counts, sizeof(Counts), hipMemcpyDeviceToHost, st));
  NB_TRY(hipStreamSynchronize(st));
  unsigned long long c[3] = {0, 0, 0};
  for (int x = 0; x < kXcd; ++x) {
    c[0] += h->ctr[x * kCtrLine];
    c[1] += h->ctr[x * kCtrLine + 1];
    c[2] |= h->ctr[x * kCtrLine + 2];
  }
  if (c[2]) {
    *msg = "tree walk stack exceeded its bound";
    return hipErrorInvalidValue;
  }
  int depth = 0;
  for (int l = 0; l < kLevels; ++l)
    if (h->lvl[l + 1] > h->lvl[l]) depth = l;
  stats->cells = h->lvl[kLevels];
  stats->groups = h->ngroups;
  stats->accepted = (int64_t)c[0];
  stats->opened_leaves = (int64_t)c[1];
  stats->depth = depth;
  return hipSuccess;
}

void tree_scratch_free(TreeScratch& s) {
  for (auto& sl : s.slots)
    if (sl.first) (void)hipFree(sl.first);
  s.slots.clear();
  if (s.host) (void)hipHostFree(s.host);
  s.host = nullptr;
}

}  // namespace nb
