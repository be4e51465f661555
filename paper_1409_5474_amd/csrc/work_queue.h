// Work queue of the persistent force grids, shared by the force kernels.
//
// The items -- (i-block, j-chunk) pairs in chunk-major order -- are cut into
// kXcd near-equal ranges, one per XCD: the hardware hands workgroups to the
// chip's 8 XCDs round-robin by blockIdx, so range x is worked by the
// workgroups on XCD x, and that XCD's L2 holds only the j-chunks of its own
// range.  Only the first min(items, grid) workgroups take part (the members;
// the rest return at once, so a launch sized for its largest count costs
// little at a small one).  A member's first item is fixed: member w starts
// with item w / kXcd of range w % kXcd, so a launch of no more items than
// workgroups touches no counter at all.  After that the members of a range
// take its remaining items from a counter in device memory, so a faster
// compute unit takes more; once its own range is exhausted, a workgroup
// takes from the other ranges in turn, so the XCDs (whose clocks differ by a
// few percent) also finish together.  Each item is computed the same way
// whichever workgroup takes it: results do not depend on the assignment.
//
// Device-scope atomics on one cache line are carried out one after another,
// about 12 ns each on the MI355X (1024 workgroups, one atomic each: 12.9 us
// for a kernel that takes 3.0 us without; 3.2 us when each XCD's workgroups
// use a line of their own).  So every counter has a line of its own, the
// workgroups that finish are counted per XCD first, and the members' first
// items cost no atomic.  (With the counters in one line and an atomic for
// the first item, a launch of 1008 short items spent about 40 us on them.)
//
// Lines: [0, kXcd) the range counters (items taken beyond the members' first
// ones), [kXcd, 2 kXcd) the finished members of each XCD, 2 kXcd the XCDs
// whose members have all finished, 2 kXcd + 1 the in-flight word.  All are
// zero before a launch, and the last member to finish sets the counters back
// to zero.  Without a queue (wq null) the grid strides over the items in the
// same order.
//
// The in-flight word lets nb_sync see calls that overlapped on the device also
// where their launches touch no counter.  What such calls share is written by
// one kernel and read by the next (the partial sums of a j-split and how many
// there are), so the first steps the word (wrapping increment
// of limit 1: 0 becomes 1, anything else 0) and the last steps it back
// (wrapping decrement: 1 becomes 0, 0 becomes kOverlapped, n becomes n - 1).
// One call after another leaves 0.  Two first steps without a step back
// between them leave a value that no later sequence of calls brings to 0: the
// step back that closes a stretch of overlapping calls finds the word at 0 or
// far above 1, and from there a call leads to 0 and then to kOverlapped.
// Neither step returns a value, and both are made early, by workgroups or
// wavefronts without other work: a wavefront's later loads, and the end of the
// kernel, wait for an atomic's completion (made by a working workgroup they
// cost a launch 0.6 to 1.1 us, MI355X).  The fourth-order force calls step
// it, except those of small systems (k_forces_small), which share nothing; the
// snap forces, whose shortest launches would take 0.5 us longer, do not.
#pragma once
#include "nb_internal.h"

namespace nb {

constexpr int kXcd = 8;
constexpr unsigned int kOverlapped = 0xffff0000u;
static_assert((2 * kXcd + 1) * kQueueLine < kErrorWord, "work queue larger than its buffer");

__device__ __forceinline__ unsigned int* queue_range(unsigned int* wq, int x) { return wq + x * kQueueLine; }

// Range x of `count` things dealt to the kXcd ranges as evenly as blockIdx
// deals workgroups to the XCDs: its length and its start.
__device__ __forceinline__ int64_t range_len(int64_t count, int x) { return count / kXcd + (x < count % kXcd ? 1 : 0); }
__device__ __forceinline__ int64_t range_lo(int64_t count, int x) {
  const int64_t r = count % kXcd;
  return x * (count / kXcd) + (x < r ? x : r);
}
__device__ __forceinline__ int64_t queue_members(int64_t items) {
  return items < (int64_t)gridDim.x ? items : (int64_t)gridDim.x;
}
__device__ __forceinline__ bool queue_member(int64_t items) { return (int64_t)blockIdx.x < items; }

// The steps of the in-flight word, by one thread of a launch.
__device__ __forceinline__ void flight_begin(unsigned int* wq) {
  if (wq) (void)atomicInc(queue_range(wq, 2 * kXcd + 1), 1u);
}
__device__ __forceinline__ void flight_end(unsigned int* wq) {
  if (wq) (void)atomicDec(queue_range(wq, 2 * kXcd + 1), kOverlapped);
}
// The first step for a launch that a second kernel follows, by the first
// workgroup without an item; with as many items as workgroups by workgroup 0,
// and with more by the first one of XCD 0 to finish, which the counters tell
// (queue_done).
__device__ __forceinline__ void flight_begin_beside(unsigned int* wq, int64_t items) {
  if (items <= (int64_t)gridDim.x && (int64_t)blockIdx.x == (items < (int64_t)gridDim.x ? items : 0) &&
      threadIdx.x == 0)
    flight_begin(wq);
}

// The first item of a member (members <= items, so range x has an item for
// each of its members).
__device__ __forceinline__ int64_t queue_first(const unsigned int* wq, int64_t items) {
  if (!wq) return blockIdx.x;
  return range_lo(items, blockIdx.x % kXcd) + blockIdx.x / kXcd;
}

// The k-th entry of range x as entry 8 k + x of a list: an order in which the
// ranges interleave, for items whose cost varies slowly along the list (the
// XCDs then share the expensive stretches).
__device__ __forceinline__ int64_t interleaved(int64_t w, int64_t items) {
  const int64_t q = items / kXcd, cut = (items % kXcd) * (q + 1);
  const int64_t x = w < cut ? w / (q + 1) : (q > 0 ? items % kXcd + (w - cut) / q : 0);
  return (w - range_lo(items, (int)x)) * kXcd + x;
}

// Thread 0 turns an own-range take into an item: `own` is the counter value
// the take returned.  When that range is exhausted it reads every range's
// counter at once (independent loads, one round of latency: device-scope
// atomics cost about a microsecond each, so the ranges are not visited one
// by one) and takes from the first range with items left, in the order
// x0 + 1, x0 + 2, ...  Returns the item, or `items` once all are exhausted.
//
// The compiler computes the ranges' bounds before the item loop and keeps
// them in registers.  With FRESH the number of items is opaque here, so they
// are computed at each pick instead: for the scalar j-path, which runs close
// to its register limit (mixed, K = 2: 92 -> 28 B of scratch per lane; 262144
// all active 39.14 -> 38.85 ms).  The LDS kernels have registers to spare and
// were slower that way (mixed, K = 1, 3899 rows and 1000003 sources: 2651 us,
// FRESH 2714 us).
template <bool FRESH>
__device__ __forceinline__ int64_t queue_pick(unsigned int* wq, int64_t items, unsigned int own) {
  if constexpr (FRESH) {
    unsigned int n = (unsigned int)items;
    asm volatile("" : "+v"(n));
    items = n;
  }
  const int x0 = blockIdx.x % kXcd;
  const int64_t members = queue_members(items);
  const int64_t k0 = range_len(members, x0) + own;
  if (k0 < range_len(items, x0)) return range_lo(items, x0) + k0;
  for (int attempt = 0; attempt < kXcd; ++attempt) {
    unsigned int cnt[kXcd];
#pragma unroll
    for (int x = 0; x < kXcd; ++x)
      cnt[x] = __hip_atomic_load(queue_range(wq, x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int pick = -1, best = kXcd;
#pragma unroll
    for (int x = 0; x < kXcd; ++x) {
      const int order = (x - x0 - 1 + 2 * kXcd) % kXcd;  // 0 for range x0 + 1
      if (range_len(members, x) + cnt[x] < range_len(items, x) && order < best) {
        best = order;
        pick = x;
      }
    }
    if (pick < 0) return items;
    const int64_t k = range_len(members, pick) + atomicAdd(queue_range(wq, pick), 1u);
    if (k < range_len(items, pick)) return range_lo(items, pick) + k;
  }
  return items;
}

// A member's next item (w_stride: its next item without a queue).
template <bool FRESH = false>
__device__ __forceinline__ int64_t queue_next(unsigned int* wq, unsigned int& slot, int64_t items, int64_t w_stride) {
  if (!wq) return w_stride;
  if (items <= (int64_t)gridDim.x) return items;  // every item was some member's first
  __syncthreads();  // every thread has read `slot` before it is replaced
  if (threadIdx.x == 0)
    slot = (unsigned int)queue_pick<FRESH>(wq, items, atomicAdd(queue_range(wq, blockIdx.x % kXcd), 1u));
  __syncthreads();
  // one value for the whole wave: read into a scalar register, so everything
  // derived from the item (chunk bounds, record addresses) stays uniform
  return (int64_t)(unsigned int)__builtin_amdgcn_readfirstlane((int)slot);
}

// Every member calls queue_done once, after its last queue_next; the last
// member of the last XCD resets the queue (each member's own takes are
// complete by then).  flight: the launch steps the in-flight word.
__device__ __forceinline__ void queue_done(unsigned int* wq, int64_t items, bool flight = false) {
  if (!wq || items <= (int64_t)gridDim.x || threadIdx.x != 0) return;
  const int64_t members = gridDim.x;  // fewer than the items
  const int x = blockIdx.x % kXcd;
  const unsigned int before = atomicAdd(queue_range(wq, kXcd + x), 1u);
  if (flight && x == 0 && before == 0) flight_begin(wq);
  if (before != range_len(members, x) - 1) return;
  const unsigned int xcds = members < kXcd ? (unsigned int)members : kXcd;
  if (atomicAdd(queue_range(wq, 2 * kXcd), 1u) != xcds - 1) return;
  for (int k = 0; k <= 2 * kXcd; ++k) atomicExch(queue_range(wq, k), 0u);
}

}  // namespace nb
