// Force kernel of the sixth-order Hermite scheme (the higher-order Hermite
// integrators that the paper cites for the direct method, section
// "Simulating Collisional systems with direct force evaluation methods"):
// acceleration, jerk, snap and potential of an active i-set in the field of
// all j-particles, each particle moving with its own predicted position,
// velocity and acceleration.  For r = x_j - x_i, u = v_j - v_i,
// w = a_j - a_i, s = |r|^2 + eps2, q = s^{-1/2}:
//   alpha = (r.u) q^2,  beta = (u.u + r.w) q^2 + alpha^2
//   A = m q^3 r,  J = m q^3 u - 3 alpha A,  S = m q^3 w - 6 alpha J - 3 beta A,
//   phi -= m q
// (the recursive form of the successive time derivatives of m r s^{-3/2}).
//
// The kernel forms them without the common factor, U = u - 3 alpha r and
// W = w - 6 alpha U - 3 beta r, and adds m q^3 r, m q^3 U, m q^3 W: the factor
// enters once per component, in the accumulating multiply-add, 55 double
// instructions per pair besides the reciprocal square root instead of 66.
//
// All arithmetic is double precision and the kernel is bound by it: 262144
// all active run at 555 to 563 G pairs/s (474 G with the recursive form).  A
// wavefront issues 56 vector instructions per pair in 61 quad-cycles of its
// SIMD, 91% of them busy (counters, MI355X; 66 and 86% in the recursive form).
// Layout as the LDS path of the fourth-order kernel: j-tiles of kTile
// particles staged in LDS as five double2 streams (x y | z m | vx vy | vz ax |
// ay az), one or four lanes per i-particle, the j-range cut into S chunks over
// a persistent grid fed by the work queue, per-tile
// double sums folded into a compensated (TwoSum) accumulator, and a second
// kernel adding the S partial blocks in a fixed order.  The active count may
// be read from device memory, so a block step can be captured in a graph.
// The self pair is kept in the loop (it adds exactly zero to A, J and S) and
// its potential term is removed with the identical value; with eps2 == 0
// every pair at zero distance is dropped instead.
#include <map>
#include <mutex>

#include "nb_internal.h"
#include "work_queue.h"

namespace nb {
namespace {

constexpr int kWG6 = 256;   // threads per workgroup = i-particles per block
constexpr int kT6 = 256;    // j-particles per staged tile
constexpr int kC6 = 10;     // acc, jerk, snap, pot
// Work items aimed at per resident workgroup: short items even out the last
// round, at the price of more partial sums (20011 all active: 2 per slot 892,
// 4: 821, 8: 785, 12: 840 us; 131072: 31.7, 31.6, 30.5, 30.6 ms).
constexpr int kItems6 = 8;

// v_rsq_f64 is accurate to about 2^-24; one third-order Newton step
// y <- y (1 + e/2 + 3 e^2/8), e = 1 - s y^2, brings it to double rounding.
__device__ __forceinline__ double rsqrt6(double s) {
  const double y = __builtin_amdgcn_rsq(s);
  const double e = fma(-(s * y), y, 1.0);
  return fma(y, e * fma(e, 0.375, 0.5), y);
}

// hi + lo += x without losing the low part (Knuth's TwoSum).
__device__ __forceinline__ void two_sum6(double& hi, double& lo, double x) {
  const double s = hi + x;
  const double bp = s - hi;
  const double err = (hi - (s - bp)) + (x - bp);
  hi = s;
  lo += err;
}

__host__ __device__ inline int64_t chunk6(int64_t n, int S) {
  const int64_t per = (n + S - 1) / S;
  return ((per + kT6 - 1) / kT6) * kT6;
}

// How an active count is cut: L lanes per i-particle (an i-block holds
// kWG6 / L rows) and S j-chunks, about target_items items.  host_split_rows
// with (kWG6, kT6) bounds the partial sums of every count for both L: four
// times the i-blocks of a quarter of the rows, and no split from target_items
// i-blocks on.
struct Split6 {
  int L, S;
};
__host__ __device__ inline Split6 split6(int64_t n_act, int slots, int target_items, int64_t n) {
  Split6 r{1, 1};
  if (n_act <= 0) return r;
  const int64_t max_s = (n + kT6 - 1) / kT6;
  // Four lanes per row while the whole pair matrix, cut into 256 x 256 blocks,
  // leaves most of the chip idle (at most two items per slot even then): a
  // block of 256 pairs per lane takes about 40 us however few there are.
  // 1000 all active: 41.6 us with one lane per row, 18.7 us with four; 4001:
  // 47.2 and 46.4 us; 65536 with 100 active: 46.1 and 28.7 us.  Above the line
  // four lanes only quarter the work per staged tile (8000: 160 and 188 us).
  if ((n_act + kWG6 - 1) / kWG6 * max_s * 4 <= 2 * (int64_t)slots) r.L = 4;
  const int64_t ib = kWG6 / r.L;
  const int64_t n_iblk = (n_act + ib - 1) / ib;
  int64_t s = (target_items + n_iblk - 1) / n_iblk;
  if (s > max_s) s = max_s;
  if (s < 1) s = 1;
  const int64_t c = chunk6(n, (int)s);  // whole tiles, so fewer chunks may cover n
  r.S = (int)((n + c - 1) / c);
  return r;
}

struct Tile6 {
  double2 xy[kT6];
  double2 zm[kT6];
  double2 vxy[kT6];
  double2 vza[kT6];   // vz, ax
  double2 ayz[kT6];   // ay, az
};

template <bool MASK>
__device__ __forceinline__ void pair6(const double* I, double2 xy, double2 zm, double2 vxy, double2 vza,
                                      double2 ayz, double e2, double* T) {
  const double rx = xy.x - I[0], ry = xy.y - I[1], rz = zm.x - I[2];
  const double ux = vxy.x - I[3], uy = vxy.y - I[4], uz = vza.x - I[5];
  const double wx = vza.y - I[6], wy = ayz.x - I[7], wz = ayz.y - I[8];
  const double s = fma(rz, rz, fma(ry, ry, fma(rx, rx, e2)));
  double q = rsqrt6(s);
  if (MASK) q = (s > 0.0) ? q : 0.0;
  const double q2 = q * q;
  const double ru = fma(rz, uz, fma(ry, uy, rx * ux));
  // u.u + r.w in one chain
  const double z = fma(rz, wz, fma(ry, wy, fma(rx, wx, fma(uz, uz, fma(uy, uy, ux * ux)))));
  const double alpha = ru * q2;
  const double beta = fma(alpha, alpha, z * q2);
  const double mq = zm.y * q;
  const double mq3 = mq * q2;
  const double a3 = -3.0 * alpha, a6 = -6.0 * alpha, b3 = -3.0 * beta;
  const double Ux = fma(a3, rx, ux), Uy = fma(a3, ry, uy), Uz = fma(a3, rz, uz);
  T[0] = fma(mq3, rx, T[0]); T[1] = fma(mq3, ry, T[1]); T[2] = fma(mq3, rz, T[2]);
  T[3] = fma(mq3, Ux, T[3]); T[4] = fma(mq3, Uy, T[4]); T[5] = fma(mq3, Uz, T[5]);
  T[6] = fma(mq3, fma(a6, Ux, fma(b3, rx, wx)), T[6]);
  T[7] = fma(mq3, fma(a6, Uy, fma(b3, ry, wy)), T[7]);
  T[8] = fma(mq3, fma(a6, Uz, fma(b3, rz, wz)), T[8]);
  T[9] += mq;
}

// One (i-block, j-chunk) item.  L lanes share an i-particle: lane `sub` takes
// j = sub, sub + L, ... of every tile, and a butterfly folds the L sums.
template <int L, bool MASK>
__device__ __forceinline__ void item6(Tile6& tile, const Force6Args& a, int64_t jbeg, int64_t jend, int64_t n_act,
                                      int64_t k0, bool final_out, double* part) {
  const int t = threadIdx.x;
  const int64_t k = k0 + t / L;
  const int sub = t % L;
  int64_t irow = k < n_act ? (int64_t)a.active[k] : -1;
  if (k < n_act && !row_in_range(irow, 0, a.n)) {  // not a particle: skipped, and reported by nb_sync
    if (a.err) atomicOr(a.err, kErrActiveRange);
    irow = -1;
  }
  const int64_t ir = irow >= 0 ? irow : 0;
  double I[9];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    I[c] = a.pos[3 * ir + c];
    I[3 + c] = a.vel[3 * ir + c];
    I[6 + c] = a.accj[3 * ir + c];
  }
  const double e2 = a.eps2;
  double hi[kC6], lo[kC6], T[kC6];
#pragma unroll
  for (int c = 0; c < kC6; ++c) hi[c] = lo[c] = T[c] = 0.0;

  for (int64_t base = jbeg; base < jend; base += kT6) {
    __syncthreads();  // every lane is done with the previous tile
    {
      const int64_t j = base + t;
      const bool ok = j < jend;
      const int64_t jr = ok ? j : 0;
      tile.xy[t] = ok ? make_double2(a.pos[3 * jr], a.pos[3 * jr + 1]) : make_double2(0.0, 0.0);
      tile.zm[t] = ok ? make_double2(a.pos[3 * jr + 2], a.mass[jr]) : make_double2(0.0, 0.0);
      tile.vxy[t] = ok ? make_double2(a.vel[3 * jr], a.vel[3 * jr + 1]) : make_double2(0.0, 0.0);
      tile.vza[t] = ok ? make_double2(a.vel[3 * jr + 2], a.accj[3 * jr]) : make_double2(0.0, 0.0);
      tile.ayz[t] = ok ? make_double2(a.accj[3 * jr + 1], a.accj[3 * jr + 2]) : make_double2(0.0, 0.0);
    }
    __syncthreads();
#pragma unroll 2
    for (int jj = sub; jj < kT6; jj += L)
      pair6<MASK>(I, tile.xy[jj], tile.zm[jj], tile.vxy[jj], tile.vza[jj], tile.ayz[jj], e2, T);
#pragma unroll
    for (int c = 0; c < kC6; ++c) {
      two_sum6(hi[c], lo[c], T[c]);
      T[c] = 0.0;
    }
  }
  double v[kC6];
#pragma unroll
  for (int c = 0; c < kC6; ++c) v[c] = hi[c] + lo[c];
#pragma unroll
  for (int o = L / 2; o > 0; o >>= 1) {
#pragma unroll
    for (int c = 0; c < kC6; ++c) v[c] += __shfl_xor(v[c], o, 64);
  }
  if (sub != 0 || irow < 0) return;
  if (final_out) {
    const double self = (e2 > 0.0) ? a.mass[irow] * rsqrt6(e2) : 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      a.acc[3 * k + c] = v[c];
      a.jerk[3 * k + c] = v[3 + c];
      a.snap[3 * k + c] = v[6 + c];
    }
    a.pot[k] = -(v[9] - self);
  } else {
#pragma unroll
    for (int c = 0; c < kC6; ++c) part[c * n_act + k] = v[c];
  }
}

// The items of one launch, taken from the work queue until none is left.
template <int L, bool MASK>
__device__ __forceinline__ void run_items6(Tile6& tile, unsigned int& slot, const Force6Args& a, int64_t n_act,
                                           int S) {
  constexpr int IB = kWG6 / L;
  const int64_t n_iblk = (n_act + IB - 1) / IB;
  const int64_t items = n_iblk * S;
  const int64_t clen = chunk6(a.n, S);
  if (!queue_member(items)) return;
  int64_t w = queue_first(a.wq, items);
  while (w < items) {
    const int64_t chunk = w / n_iblk;
    const int64_t iblk = w - chunk * n_iblk;
    const int64_t jb = chunk * clen;
    const int64_t je = jb + clen < a.n ? jb + clen : a.n;
    item6<L, MASK>(tile, a, jb, je, n_act, iblk * IB, S == 1, a.part + chunk * kC6 * n_act);
    w = queue_next(a.wq, slot, items, w + gridDim.x);
  }
  queue_done(a.wq, items);
}

__device__ __forceinline__ int64_t active_count6(const Force6Args& a) {
  int64_t n_act = a.n_active;
  if (a.n_active_dev) {
    const int64_t d = *a.n_active_dev;
    n_act = d < n_act ? (d < 0 ? 0 : d) : n_act;
  }
  return n_act;
}

template <bool MASK>
__global__ __launch_bounds__(kWG6) void k_forces6(Force6Args a) {
  __shared__ Tile6 tile;
  __shared__ unsigned int slot;
  const int64_t n_act = active_count6(a);
  const Split6 sp = split6(n_act, a.slots, a.target_items, a.n);
  if (sp.L == 1) run_items6<1, MASK>(tile, slot, a, n_act, sp.S);
  else run_items6<4, MASK>(tile, slot, a, n_act, sp.S);
}

// Fixed-order sum of the S partial blocks, self-term removal, output.
__global__ __launch_bounds__(256) void k_reduce6(Force6Args a) {
  const int64_t n_act = active_count6(a);
  const int S = split6(n_act, a.slots, a.target_items, a.n).S;
  if (S <= 1) return;
  const int64_t total = kC6 * n_act;
  const int g = chunk_lanes(S);
  const int lg = __builtin_ctz(g);
  const int lane = threadIdx.x & (g - 1);
  for (int64_t idx = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> lg; idx < total;
       idx += ((int64_t)gridDim.x * blockDim.x) >> lg) {
    const int64_t c = idx / n_act;
    const int64_t k = idx - c * n_act;
    const double s = sum_blocks(a.part + c * n_act + k, kC6 * n_act, S, lane, g);
    if (lane != 0) continue;
    if (!row_in_range(a.active[k], 0, a.n)) continue;  // skipped row (flagged by the force pass)
    if (c < 3) {
      a.acc[3 * k + c] = s;
    } else if (c < 6) {
      a.jerk[3 * k + c - 3] = s;
    } else if (c < 9) {
      a.snap[3 * k + c - 6] = s;
    } else {
      const double self = (a.eps2 > 0.0) ? a.mass[a.active[k]] * rsqrt6(a.eps2) : 0.0;
      a.pot[k] = -(s - self);
    }
  }
}

}  // namespace

int forces6_resident_wgs(bool mask) {
  static std::mutex mu;
  static std::map<int, int> cache;
  std::lock_guard<std::mutex> lk(mu);
  auto it = cache.find(mask ? 1 : 0);
  if (it != cache.end()) return it->second;
  int nblk = 0;
  const void* fn = mask ? (const void*)k_forces6<true> : (const void*)k_forces6<false>;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nblk, fn, kWG6, 0) != hipSuccess || nblk < 1) {
    (void)hipGetLastError();
    nblk = 1;
  }
  cache[mask ? 1 : 0] = nblk;
  return nblk;
}

int forces6_target(int slots) { return kItems6 * slots; }

int forces6_split(int64_t n_act, int slots, int target_items, int64_t n) {
  return split6(n_act, slots, target_items, n).S;
}

hipError_t launch_forces6(const Force6Args& a, bool mask, int grid, hipStream_t st) {
  if (grid < 1) grid = 1;
  if (mask)
    hipLaunchKernelGGL(k_forces6<true>, dim3(grid), dim3(kWG6), 0, st, a);
  else
    hipLaunchKernelGGL(k_forces6<false>, dim3(grid), dim3(kWG6), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (!a.n_active_dev && a.S <= 1) return hipSuccess;
  // threads: the outputs times the lanes per output (with the count on the
  // device, as for the fourth-order reduce: up to 1024 blocks, at least the
  // outputs' threads)
  const int64_t outs = kC6 * a.n_active;
  int64_t threads = outs * chunk_lanes(a.S);
  if (a.n_active_dev) {
    threads = outs * 64 < (int64_t)1024 * 256 ? outs * 64 : (int64_t)1024 * 256;
    if (threads < outs) threads = outs;
  }
  int64_t rg = (threads + 255) / 256;
  if (rg > 4096) rg = 4096;
  if (rg < 1) rg = 1;
  hipLaunchKernelGGL(k_reduce6, dim3((int)rg), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace nb
