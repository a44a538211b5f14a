// History and running state moved between the orders and layouts that the sweep forms hold
// them in (snapshots of another form, a handle planned again with its history).  Both hold
// the same inputs, so the moved handle continues as one that made the whole run itself, once
// its pending sums are formed again.  Rare: copies by gather, one thread per position, plane
// and range of steps.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "step_items.h"

namespace sbim {
namespace {

constexpr int kMoveThreads = 256;
constexpr int kMoveSteps = 32;  // steps per thread

// Complex entry (component 0) of step n: in the ring of block b, or in the recent ring.
template <typename R>
struct Entry {
  R *re, *im;      // component 0
  long long next;  // reals between components
};
template <typename R>
__device__ __forceinline__ Entry<R> ring_entry(const RingSide &a, int np, int p, long long s, long long n) {
  const long long b = s >> 6;
  const int lane = static_cast<int>(s & 63), cap = a.cap[b];
  R *ring = static_cast<R *>(a.ring);
  if (!a.tiled) {
    R *e = ring + (((a.off[b] + n % cap * a.stride[b]) * np + p) * 3 * kLanes + lane) * 2;
    return {e, e + 1, 2 * kLanes};
  }
  constexpr int TS = RingTile<R>::TS;
  const long long slot = (n + ring_shift<R>(b)) % cap;
  R *e = ring + a.off[b] * np * 3 * kLanes * 2 +
         (((slot / TS * np + p) * 3 * kLanes + lane) * 2) * TS + slot % TS;
  return {e, e + TS, 2LL * kLanes * TS};
}
template <typename R>
__device__ __forceinline__ Entry<R> recent_entry(const RingSide &a, int np, int p, long long s, long long n) {
  R *e = static_cast<R *>(a.ring) + a.records * np * 3 * kLanes * 2 +
         (((n % kRecent * a.nblocks + (s >> 6)) * np + p) * 3 * kLanes + (s & 63)) * 2;
  return {e, e + 1, 2 * kLanes};
}

template <typename R>
__global__ __launch_bounds__(kMoveThreads) void relocate_ring_kernel(RingSide from, RingSide to,
                                                                     const int *map, int np, long long step) {
  const long long s = static_cast<long long>(blockIdx.x) * kMoveThreads + threadIdx.x;
  if (s >= to.M || map[s] < 0) return;
  const long long f = map[s];
  const int p = blockIdx.z;
  // (blocks of equal window and more: the entries both hold cover the mode's window)
  const long long held = min(static_cast<long long>(min(from.cap[f >> 6], to.cap[s >> 6])), step);
  const long long a0 = 1 + static_cast<long long>(blockIdx.y) * kMoveSteps;
  for (long long age = a0; age < a0 + kMoveSteps && age <= held; ++age) {
    const long long n = step - age;
    // (the newest steps of the time-tiled form may not be in their tile yet)
    const Entry<R> src = from.tiled && age <= kRecent ? recent_entry<R>(from, np, p, f, n)
                                                      : ring_entry<R>(from, np, p, f, n);
    const Entry<R> dst = ring_entry<R>(to, np, p, s, n);
    const bool recent = to.tiled && age <= kRecent;
    const Entry<R> d2 = recent ? recent_entry<R>(to, np, p, s, n) : dst;
    for (int c = 0; c < 3; ++c) {
      const R re = src.re[c * src.next], im = src.im[c * src.next];
      dst.re[c * dst.next] = re;
      dst.im[c * dst.next] = im;
      if (recent) {
        d2.re[c * d2.next] = re;
        d2.im[c * d2.next] = im;
      }
    }
  }
}

__global__ __launch_bounds__(kMoveThreads) void relocate_state_kernel(const double2 *src, long long src_M,
                                                                      double2 *dst, long long M,
                                                                      const int *map) {
  const long long s = static_cast<long long>(blockIdx.x) * kMoveThreads + threadIdx.x;
  if (s >= M) return;
  const long long r = blockIdx.y;
  dst[r * M + s] = map[s] < 0 ? double2{0.0, 0.0} : src[r * src_M + map[s]];
}

}  // namespace

hipError_t launch_relocate_ring(bool fp64, const RingSide &from, const RingSide &to, const int *map,
                                int np, long long step, int wmax, hipStream_t st) {
  // (a block's capacity: its largest window, rounded up to whole tiles, at least four)
  const long long held = std::min<long long>(step, wmax + 16);
  if (held <= 0 || to.M == 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>((to.M + kMoveThreads - 1) / kMoveThreads),
                  static_cast<unsigned>((held + kMoveSteps - 1) / kMoveSteps), static_cast<unsigned>(np));
  if (fp64)
    relocate_ring_kernel<double><<<grid, kMoveThreads, 0, st>>>(from, to, map, np, step);
  else
    relocate_ring_kernel<float><<<grid, kMoveThreads, 0, st>>>(from, to, map, np, step);
  return hipGetLastError();
}

hipError_t launch_relocate_state(const double *src, long long src_M, double *dst, long long M,
                                 const int *map, int rows, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>((M + kMoveThreads - 1) / kMoveThreads), static_cast<unsigned>(rows));
  relocate_state_kernel<<<grid, kMoveThreads, 0, st>>>(reinterpret_cast<const double2 *>(src), src_M,
                                                       reinterpret_cast<double2 *>(dst), M, map);
  return hipGetLastError();
}

}  // namespace sbim
