// Mode-space kernels of the boundary-integral step on gfx950:
//   step_kernel      two kinds of items in one launch per step:
//                    mode items: the push (rotate the new spectrum into the
//                    wavevector frame, update the float64 running state, store
//                    the history ring slot) and, from the same registers, the
//                    traction of the step (pending history sum plus the newest
//                    lags, damping and instantaneous terms of Eq. SBI, Sec. 2.3,
//                    rotation back to (x1, x2, x3));
//                    sweep items: the truncated history convolution (the
//                    nonlocal term of Eq. SBI), one pass over a block's history
//                    serving the next several steps;
//   tabulate_kernel  float64 quadrature of the per-lag kernel weights.
//
// Layouts (one material group; modes sorted by (W desc, q asc), 64 per block):
//   ring    [record][plane][component L,N,T][64 lanes] complex.  Step n of
//           block b lives in record blk_off[b] + (n mod blk_cap[b]) * blk_stride[b]:
//           consecutive blocks of one sweep phase (b mod depth) with equal
//           capacity form a run laid out slot-major (stride = run length), so
//           one history slot of a run is contiguous;
//   table   class-major rows: entry cls_off[class] + j holds (w11, w12, w22, w33)
//           of lag j, j < W of the class.
#include <algorithm>
#include <cmath>

#include "step_items.h"

namespace sbim {
namespace {

// History entries whose loads the sweep issues together (measured on gfx950,
// 512x512 x 2 planes, W = 1000): float32 at depth 8, float64 and the
// compensated form fit one more wavefront per SIMD with pairs.
template <typename R, int S, bool COMP> constexpr int sweep_group() {
  constexpr int g = (COMP || sizeof(R) == 8 || S >= 8) ? 2 : 4;
  return S % g == 0 ? g : (S % 2 == 0 ? 2 : 1);  // a divisor of the span
}

// Lag chunks per sweep wavefront (measured on gfx950, 512x512 and 1024x1024 x
// 2 planes, W = 1000 and 2000): four for float32 with one lane per mode (16
// modes x 4 chunks, three wavefronts per SIMD), two otherwise (float64 and the
// compensated form: 32 modes x 2 chunks, 256-byte segments of float32 pairs;
// with two lanes per mode 16 modes x 2 x 2 in every form).  Depth 6 is the
// short-window sweep (mean window under 64 lags): one chunk of 64 modes, as
// chunks of whole spans would mostly pass the windows' ends (2048x2048 x 2,
// per-mode windows of mean 18 lags: 0.85 -> 0.80 ms per step).
template <typename R, int S, int T, bool COMP> constexpr int sweep_lag_groups() {
  if (S == 6 && T == 1) return 1;
  return (COMP || sizeof(R) == 8 || T > 1) ? 2 : 4;
}

// Wavefronts of a work-group that share one sweep item of a long block (8: 64^2 35 us a
// step against 31, 16^2 with 1600 lags 29 against 33; float64), and the window from
// which a block is long (256^2 x 2 float64, windows per mode up to 300: 24 52 us, 48 54,
// 96 61).
constexpr int kSplit = 4, kLongWindow = 24;

// Rows k0 .. k0+S-1 of a mode's kernel.  A class's W rows are followed by a
// zero row, so clamping the lag to W gives zero from the window on.
template <typename R, int S>
__device__ __forceinline__ void load_rows(typename W4<R>::T (&w)[S],
                                          const typename W4<R>::T *__restrict__ rowp, int k0,
                                          int wl) {
#pragma unroll
  for (int k = 0; k < S; ++k) w[k] = rowp[min(k0 + k, wl)];
}

// sums[s] += products of S consecutive history entries (lags i .. i+S-1) with
// rows i+s .. i+s+S-1, the rows held as A = rows i .. i+S-1 and
// B = rows i+S .. i+2S-1.  hp / x point at the ring record / slot of lag i
// and are advanced past lag i+S-1.
template <typename R, int S, int G>
__device__ __forceinline__ void sweep_span(R (&sums)[S][kSums], const typename W4<R>::T (&A)[S],
                                           const typename W4<R>::T (&B)[S],
                                           const cplx<R> *__restrict__ &hp, int &x, int cap,
                                           long long dstep, long long dwrap) {
  static_assert(S % G == 0, "load groups must tile the span");
  typedef R nv2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int g0 = 0; g0 < S; g0 += G) {
    cplx<R> u[G][3];
#pragma unroll
    for (int t = 0; t < G; ++t) {
      // the history is read once per sweep: non-temporal loads keep it from
      // displacing the kernel rows in the caches
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const nv2 v = __builtin_nontemporal_load(reinterpret_cast<const nv2 *>(hp + c * kLanes));
        u[t][c] = cplx<R>{v.x, v.y};
      }
      const bool wrap = x == 0;  // next older slot
      hp += wrap ? dwrap - dstep : -dstep;
      x = wrap ? cap - 1 : x - 1;
    }
#pragma unroll
    for (int t = 0; t < G; ++t)
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int k = g0 + t + s;
        fma_lag<R>(sums[s], k < S ? A[k] : B[k - S], u[t]);
      }
  }
}

// History staged through LDS (float32, 6 steps a lane, two lanes and two lag chunks a
// mode): a stage is the two spans of one pass of the sweep's loop, kStageLags lags of each
// chunk.  A (lag, component) of it is 2 chunks x 16 modes x 8 bytes, contiguous per chunk,
// which 16 lanes fetch in 16-byte pieces straight into LDS, so a stage takes 9 loads of
// 1 KB and no registers, where the lanes' own loads took 36 of 512 bytes, half of them
// fetched twice.
constexpr int kStageLags = 12;
constexpr int kStageLoads = kStageLags * 3 / 4;
constexpr int kStageBytes = kStageLoads * 1024;
typedef __attribute__((address_space(3))) void *lds_ptr;

// Fetches a stage into the LDS at `dst`: piece is the byte offset of the lane's 16 bytes
// of component 0 in a slot, x0 the slot of its chunk's first lag (cap >= kStageLags: one
// wrap at most).  Buffer loads: 32-bit offsets from the block's first slot.  (The compiler
// takes the global form for one that may touch LDS through a flat address, and then waits
// for every load in flight wherever it needs one.)
__device__ __forceinline__ void fetch_stage(__amdgpu_buffer_rsrc_t ring, unsigned piece, int x0, int cap,
                                            unsigned slot_bytes, lds_ptr dst) {
  int e = (threadIdx.x & 63) / 16;  // the lane's (lag, component) of the first load
  asm volatile("" : "+v"(e));       // (opaque: not kept per load through the caller's loop)
  int x = x0 - (e == 3), c = e == 3 ? 0 : e;
  x += x < 0 ? cap : 0;
#pragma unroll
  for (int i = 0; i < kStageLoads; ++i) {
    // (non-temporal, as in sweep_span)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        ring, (__attribute__((address_space(3))) char *)dst + i * 1024, 16,
        static_cast<int>(static_cast<unsigned>(x) * slot_bytes + static_cast<unsigned>(c * (kLanes * 8)) + piece),
        0, 0, 2);
    __builtin_amdgcn_sched_barrier(0);  // (one address at a time)
    // four further on: the next lag's next component
    const bool carry = c == 2;
    x -= carry ? 2 : 1;
    x += x < 0 ? cap : 0;
    c = carry ? 0 : c + 1;
  }
}

// Lags L and L + 1 of a stage, all components, of the lane's chunk and mode (at byte `at`
// of the LDS).  WAIT: the stage's loads are complete once no more than kStageLoads
// younger ones are outstanding; the loads of the next stage are issued before this.
template <int L, bool WAIT>
__device__ __forceinline__ void read_stage(float2 (&u)[2][3], unsigned at) {
  if constexpr (WAIT)
    asm volatile("s_waitcnt vmcnt(9)" ::: "memory");
  static_assert(kStageLoads == 9, "the wait above");
  asm volatile("ds_read_b64 %0, %6 offset:%7\n\t"
               "ds_read_b64 %1, %6 offset:%8\n\t"
               "ds_read_b64 %2, %6 offset:%9\n\t"
               "ds_read_b64 %3, %6 offset:%10\n\t"
               "ds_read_b64 %4, %6 offset:%11\n\t"
               "ds_read_b64 %5, %6 offset:%12\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&v"(u[0][0]), "=&v"(u[0][1]), "=&v"(u[0][2]), "=&v"(u[1][0]), "=&v"(u[1][1]),
                 "=&v"(u[1][2])
               : "v"(at), "n"((3 * L) * 256), "n"((3 * L + 1) * 256), "n"((3 * L + 2) * 256),
                 "n"((3 * L + 3) * 256), "n"((3 * L + 4) * 256), "n"((3 * L + 5) * 256)
               : "memory");
}

// sweep_span (S = 6) on a staged history: H = 0, 1 the first or second span of the stage.
template <int H>
__device__ __forceinline__ void sweep_span_staged(float (&sums)[6][kSums], const float4 (&A)[6],
                                                  const float4 (&B)[6], unsigned at) {
  static_for<3>([&](auto gc) {
    constexpr int g0 = 2 * decltype(gc)::value;
    float2 u[2][3];
    read_stage<6 * H + g0, H == 0 && g0 == 0>(u, at);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int s = 0; s < 6; ++s) {
        const int k = g0 + t + s;
        fma_lag<float>(sums[s], k < 6 ? A[k] : B[k - 6], u[t]);
      }
  });
}

// The sweep launched with step n serves steps t0 = n+1 .. n+D (depth D = S T).
// Blocks of phase t0 mod D read their history up to step n-1 once, U^{t0-i}
// for i = 2 .. min(cap-1, t0), and form for each of those steps t0+u its sum
// over that history:
//   pending[(t0+u) mod (D+1)] = sum_{i>=2} w_{i+u} (x) U^{t0-i}   (lags i+u inside the window).
// It reads neither U^n nor the pending sum of step n, so it runs in the same
// launch as the push and traction of step n (D+1 pending slots keep step n's
// sum apart from the D being written).
// Each history entry thus serves D steps.  A lane holds the sums of S of
// them (registers bound S); T lanes per mode and lag chunk take the D steps
// in groups u = g S + s, g < T.  They load the same history entries in the
// same instructions, so each entry is fetched from memory once for all D
// steps.  The kernel rows i+gS .. i+gS+2S-2 that a span of S entries needs are
// held in two register arrays used in turn, so each row is loaded once per
// lane and never moved.
//
// Lag chunks are whole spans long, so chunks never overlap and no lane needs a
// mask: chunks reach past the last entry by less than LG spans, and a lag
// i > min(cap-1, t0) either meets zero kernel rows (i + s >= cap >= W) or a
// ring slot not written since the last reset, which holds zero (the slot that
// the concurrent push writes is lag 1 or cap+1, whose rows are unused or zero).
//
// Work item (one wavefront) = (block of the phase, plane, group of Q of the
// block's 64 modes).  Its 64 lanes are Q modes x T step groups x LG lag
// chunks (Q = 64 / (T LG)): lane l takes mode l mod Q of the group, step
// group (l / Q) mod T and chunk l / (Q T) of the lags, so each history load
// fetches LG segments of Q x 8 bytes (float32), one per chunk.  The chunks
// are then summed by a butterfly over lanes l ^ QT, l ^ 2QT, ... (fixed
// order, so the result is bitwise reproducible).
// SPLIT: the item is shared by a work-group of kSplit wavefronts: each takes LG of
// kSplit LG chunks, and the wavefronts' sums meet in LDS, one step at a time, in order.
// STAGED: the history comes through LDS (fetch_stage; cap >= kStageLags).
// ALONE: the work-group is one wavefront.
template <typename R, int S, int T, bool COMP, bool SPLIT, bool STAGED, bool ALONE>
__device__ __forceinline__ void sweep_item(const SweepArgs &a, long long kb, int r) {
  constexpr int NW = SPLIT ? kSplit : 1;
  using W = typename W4<R>::T;
  const cplx<R> *__restrict__ ring = static_cast<const cplx<R> *>(a.ring);
  const W *__restrict__ table = static_cast<const W *>(a.table);
  void *const pending = a.pending;
  const long long M = a.M, step = a.step;
  const int np = a.np;
  constexpr int LG = sweep_lag_groups<R, S, T, COMP>();
  constexpr int Q = kLanes / (LG * T);  // modes per item
  constexpr int NQ = kLanes / Q;        // items per block and plane
  constexpr int D = S * T;
  const int p = r / NQ;
  const long long t0 = step + 1;
  const long long b = t0 % D + D * kb;
  // (a wavefront alone: not masked.  Known to be under 64, the compiler keeps
  // the slot arithmetic of a single chunk in scalar registers, between the loads: float64
  // 512^2, two materials, 40 lags: the sweeps alone 23.2 and 21.0 us.)
  const int lane = ALONE ? threadIdx.x : threadIdx.x & (kLanes - 1);
  const int wave = SPLIT ? static_cast<int>(threadIdx.x) / kLanes : 0;
  const int lg = lane / (Q * T);
  const int u0 = (lane / Q) % T * S;        // first of the lane's S steps (t0 + u0 ..)
  const int col = (r % NQ) * Q + lane % Q;  // lane of the mode in its block
  const long long sm = b * kLanes + col;
  const bool valid = sm < M;
  const int cap = a.blk_cap[b];
  if (cap <= kDirectLags) return;  // every lag is summed by the mode items
  // history entries (lags 2 .. min(cap-1, t0) of step t0) that the window can reach
  const int nent = static_cast<int>(max(0LL, min(static_cast<long long>(cap) - 1, t0) - 1));
  const int wl = valid ? a.win[sm] : 0;
  const long long row0 = valid ? a.row0[sm] : 0;
  const int per = (nent + NW * LG * S - 1) / (NW * LG * S) * S;  // lags per chunk
  const int i0 = 2 + (wave * LG + lg) * per;

  constexpr int G = sweep_group<R, S, COMP>();
  // plain form: the running sums; compensated form: the products since the
  // last fold into the compensated accumulators (up to 6S lags, three span pairs)
  R sums[S][kSums];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int k = 0; k < kSums; ++k) sums[s][k] = R(0);
  Acc<R, COMP> acc[S][kSums];
  if (per > 0) {  // then cap > 2, so the block has a mode with W > 0 and class 0 exists
    const long long rec_len = static_cast<long long>(np) * 3 * kLanes;
    const long long dstep = a.blk_stride[b] * rec_len;  // elements between consecutive slots
    const long long dwrap = static_cast<long long>(cap) * dstep;
    // ring slot of lag i0 of step t0 (i0 may pass t0)
    int x = mod_step(t0, cap) - i0 % cap;
    if (x < 0) x += cap;
    const cplx<R> *hp = ring +
                        (a.blk_off[b] + static_cast<long long>(x) * a.blk_stride[b]) * rec_len +
                        static_cast<long long>(p) * 3 * kLanes + col;
    // a mode without history (W = 0) reads the zero row after class 0's rows
    const W *rowp = table + (wl > 0 ? row0 : a.cls_w0);
    W ra[S], rb[S];
    load_rows<R, S>(ra, rowp, i0 + u0, wl);
    // staged history: this lane's piece, its slot, and the stage of the LDS in use
    extern __shared__ __attribute__((aligned(16))) unsigned char stages[];
    __amdgpu_buffer_rsrc_t ring_rsrc;
    unsigned piece = 0;
    int xs = 0, half = 0;
    const unsigned slot_bytes = static_cast<unsigned>(dstep) * static_cast<unsigned>(sizeof(cplx<R>));
    if constexpr (STAGED) {
      static_assert(sizeof(R) == 4 && S == 6 && T == 2 && LG == 2 && Q == 16, "layout of a stage");
      const int chunk = lane % 16 / 8;
      xs = mod_step(t0, cap) - (2 + chunk * per) % cap;
      if (xs < 0) xs += cap;
      piece = static_cast<unsigned>((p * 3 * kLanes + (r % NQ) * Q) * 8 + lane % 8 * 16);
      ring_rsrc = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<cplx<R> *>(ring + uniform64(a.blk_off[b]) * rec_len), 0,
          __builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<unsigned>(cap - 1) * slot_bytes +
                                                          static_cast<unsigned>(rec_len) * 8u)),
          kBufferWord3);
      fetch_stage(ring_rsrc, piece, xs, cap, slot_bytes, (lds_ptr)stages);
    }
    for (int it = 0; it < per; it += 2 * S) {
      const int i = i0 + u0 + it;
      load_rows<R, S>(rb, rowp, i + S, wl);
      unsigned at = 0;
      if constexpr (STAGED) {
        __builtin_amdgcn_sched_barrier(0);  // (the rows first: waiting for them must not wait for the stage)
        // the next stage (past the last one: entries of the ring that nothing uses)
        xs -= kStageLags;
        xs += xs < 0 ? cap : 0;
        at = static_cast<unsigned>(reinterpret_cast<__SIZE_TYPE__>((lds_ptr)stages)) +
             static_cast<unsigned>(half * kStageBytes + lg * 128 + lane % Q * 8);
        half ^= 1;
        fetch_stage(ring_rsrc, piece, xs, cap, slot_bytes, (lds_ptr)(stages + half * kStageBytes));
        sweep_span_staged<0>(sums, ra, rb, at);
      } else {
        sweep_span<R, S, G>(sums, ra, rb, hp, x, cap, dstep, dwrap);
      }
      if (it + S >= per) break;
      load_rows<R, S>(ra, rowp, i + 2 * S, wl);
      if constexpr (STAGED)
        sweep_span_staged<1>(sums, rb, ra, at);
      else
        sweep_span<R, S, G>(sums, rb, ra, hp, x, cap, dstep, dwrap);
      // compensated form: fold the plain partial sums of the last 6S lags
      // (every third pass of this loop; the branch is uniform over the wavefront)
      if constexpr (COMP) {
        if ((it / (2 * S)) % 3 == 2) {
#pragma unroll
          for (int s = 0; s < S; ++s)
#pragma unroll
            for (int k = 0; k < kSums; ++k) {
              acc[s][k].fold(sums[s][k]);
              sums[s][k] = R(0);
            }
        }
      }
    }
    // the stage fetched past the last one must not land in LDS that has a new owner
    if constexpr (STAGED) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int k = 0; k < kSums; ++k) acc[s][k].fold(sums[s][k]);
  // sum the lag chunks of each mode; lanes of chunk 0 store
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const long long slot = (t0 + u0 + s) % (D + 1);
#pragma unroll
    for (int k = 0; k < kSums; ++k)
#pragma unroll
      for (int off = Q * T; off < kLanes; off <<= 1) acc[s][k].fold_lane(off);
    if constexpr (SPLIT) {
      using A = Acc<R, COMP>;
      __shared__ __attribute__((aligned(16))) unsigned char lds[sizeof(A) * kSums * NW * Q * T];
      auto part = reinterpret_cast<A(*)[NW][Q * T]>(lds);
      if (lg == 0) {
#pragma unroll
        for (int k = 0; k < kSums; ++k) part[k][wave][lane] = acc[s][k];
      }
      __syncthreads();
      if (wave == 0 && lg == 0) {
#pragma unroll
        for (int k = 0; k < kSums; ++k)
#pragma unroll
          for (int w = 1; w < NW; ++w) acc[s][k].fold(part[k][w][lane]);
      }
      __syncthreads();
    }
    if (wave == 0 && lg == 0 && valid) {
#pragma unroll
      for (int t = 0; t < 5; ++t)
        store_sum<R, false>(pending, (slot * np + p) * 5LL, t, M, sm,
                            cplx<R>{acc[s][2 * t].value(), acc[s][2 * t + 1].value()});
    }
  }
}

// One launch per step of mode-space work: the sweep items of the blocks whose
// turn it is, then one mode item per (64-mode block, plane).  The two kinds
// share no data (see sweep_item), so the latency-bound push gathers and
// traction scatters run beside the streaming sweep.
template <typename R, int S, int T, bool COMP, bool STAGED = false>
__device__ __forceinline__ void step_items(const SweepArgs &sa, const ModeArgs &ma,
                                           long long sweep_items, long long nblocks) {
  const long long item = blockIdx.x;
  if (item < sweep_items) {
    // Items of one block get ids congruent mod 8, so they run on one XCD and
    // share the block's kernel rows in its L2.
    const int per_blk = sweep_lag_groups<R, S, T, COMP>() * T * sa.np;
    const long long kb = (item / (8LL * per_blk)) * 8 + (item & 7);
    if (kb < sa.nphase) sweep_item<R, S, T, COMP, false, STAGED, true>(sa, kb, static_cast<int>((item >> 3) % per_blk));
    return;
  }
  const long long k = xcd_chunk(item - sweep_items, nblocks * ma.np);
  if (k >= nblocks * ma.np) return;
  const int p = static_cast<int>(k / nblocks);
  const long long s = (k - p * nblocks) * kLanes + threadIdx.x;
  if (s < ma.M) mode_step<R, COMP, false>(ma, p, s);
}

template <typename R, int S, int T, bool COMP>
__global__ __launch_bounds__(kLanes) void step_kernel(SweepArgs sa, ModeArgs ma,
                                                      long long sweep_items, long long nblocks) {
  step_items<R, S, T, COMP>(sa, ma, sweep_items, nblocks);
}

// The float32 sweep at 6 steps per lane and two lanes per mode, held to four
// wavefronts per SIMD (128 registers; the compiler alone takes 131, three).
template <typename R, int S, int T, bool COMP>
__global__ __launch_bounds__(kLanes) __attribute__((amdgpu_waves_per_eu(4))) void step_kernel_w4(
    SweepArgs sa, ModeArgs ma, long long sweep_items, long long nblocks) {
  step_items<R, S, T, COMP>(sa, ma, sweep_items, nblocks);
}

// The compensated sweep at up to 6 steps per lane, held to two wavefronts per
// SIMD: left to itself the compiler takes the whole register file (one
// wavefront) for a couple of registers that it then keeps in scratch instead.
template <typename R, int S, int T, bool COMP>
__global__ __launch_bounds__(kLanes) __attribute__((amdgpu_waves_per_eu(2))) void step_kernel_w2(
    SweepArgs sa, ModeArgs ma, long long sweep_items, long long nblocks) {
  step_items<R, S, T, COMP>(sa, ma, sweep_items, nblocks);
}

// The float32 sweep with staged history.  Its wavefronts are few (two a SIMD), and their
// own loads kept too little in flight to cover the memory's latency; the stage of the next
// 12 lags is in flight while the current one is summed, without registers.  Now bound by
// the multiply-adds and the last, partly filled round of wavefronts.  A rupture step, one
// plane, us: 1024^2 compensated at 2000 lags 978 -> 790, 512^2 at
// 1000 226 -> 160, 128^2 at 300 77 -> 57, 64^2 at 100 38 -> 38; float32 512^2 at 1600 341
// -> 207.  (Fetching a stage in two halves, or its offsets by subtraction: the same.)
template <bool COMP>
__global__ __launch_bounds__(kLanes) __attribute__((amdgpu_waves_per_eu(2))) void step_kernel_staged(
    SweepArgs sa, ModeArgs ma, long long sweep_items, long long nblocks) {
  step_items<float, 6, 2, COMP, true>(sa, ma, sweep_items, nblocks);
}

// The same with work-groups of kSplit wavefronts, for launches that would wait for the
// chain of lags of their long blocks (each chunk's lags come one load group after the
// other): first the `nlong` long blocks of the phase, the item of one (block, plane,
// group of modes) shared by a work-group; then the others, one item per wavefront; then
// the mode items.  (Float64, window in lags: 64^2 at 100 38.5 -> 31.4 us a step, 16^2 at
// 1600 75 -> 33; windows per mode, 256^2 x 2 90 -> 51, 1024^2 343 -> 184.)
template <typename R, int S, int T, bool COMP>
__global__ __launch_bounds__(kSplit * kLanes) __attribute__((amdgpu_waves_per_eu(2))) void
step_kernel_split(SweepArgs sa, ModeArgs ma, long long long_wgs, long long sweep_wgs, long long nlong,
                  long long nblocks) {
  const long long wg = blockIdx.x;
  const int wave = static_cast<int>(threadIdx.x) / kLanes;
  const int per_blk = sweep_lag_groups<R, S, T, COMP>() * T * sa.np;
  if (wg < long_wgs) {
    const long long kb = (wg / (8LL * per_blk)) * 8 + (wg & 7);
    if (kb < nlong) sweep_item<R, S, T, COMP, true, false, false>(sa, kb, static_cast<int>((wg >> 3) % per_blk));
    return;
  }
  if (wg < sweep_wgs) {
    const long long j = wg - long_wgs;
    const long long kb = nlong + ((j / (8LL * per_blk)) * 8 + (j & 7)) * kSplit + wave;
    if (kb < sa.nphase) sweep_item<R, S, T, COMP, false, false, false>(sa, kb, static_cast<int>((j >> 3) % per_blk));
    return;
  }
  const long long n = nblocks * ma.np;
  const long long k = xcd_chunk(wg - sweep_wgs, (n + kSplit - 1) / kSplit) * kSplit + wave;
  if (k >= n) return;
  const int p = static_cast<int>(k / nblocks);
  const long long s = (k - p * nblocks) * kLanes + threadIdx.x % kLanes;
  if (s < ma.M) mode_step<R, COMP, false>(ma, p, s);
}

// -------------------------------------------------------------- tabulate

// Piece A (0 < y < 1): y = sin(t).  Piece B (1 < y < eta): y^2 = 1 + (eta^2-1) sin^2(t).
// Both map t in [0, pi/2] and remove the square-root end points of the
// branch-cut densities D_ab (see the oracle-independent derivation in the
// library notes): the substituted integrands are analytic.
struct Node {
  double y, g11, g12, g22, g33, ph_hi, ph_lo, c_step, s_step;
};

// Lags a thread of tabulate_kernel sums, kTabThreads apart.
constexpr int kTabThreads = 256;
constexpr int kTabLags = 8;

// x - 2 pi k for the double-double x = hi + lo, reduced in two parts
// (Cody-Waite): accurate to ~1e-16 absolute however many periods x spans.
__device__ __forceinline__ double reduce_two_pi(double hi, double lo) {
  const double two_pi_hi = 6.283185307179586;      // nearest double to 2 pi
  const double two_pi_lo = 2.4492935982947064e-16;  // 2 pi - two_pi_hi
  const double inv_two_pi = 0.15915494309189535;
  const double k = rint(hi * inv_two_pi);
  const double r = fma(-k, two_pi_hi, hi);  // exact
  return fma(-k, two_pi_lo, r) + lo;
}

__device__ Node make_node(int i, int npan, double eta, double dT, const double *gl_x,
                          const double *gl_w) {
  const int per_piece = npan * kGaussN;
  const int piece = i / per_piece;
  const int r = i - piece * per_piece;
  const int pan = r / kGaussN;
  const int g = r - pan * kGaussN;
  const double half_pi = 1.5707963267948966;
  const double h = half_pi / npan;
  const double t = (pan + 0.5 * (gl_x[g] + 1.0)) * h;
  const double wt = 0.5 * gl_w[g] * h;
  const double e2 = eta * eta;
  const double st = sin(t), ct = cos(t);
  Node n;
  double d11, d12, d22, d33, jac, y;
  if (piece == 0) {
    y = st;
    const double as = ct;
    const double ap = sqrt(1.0 - y * y / e2);
    const double d = e2 + 1.0 - y * y;
    jac = ct * wt;
    d11 = 2.0 * (as * (e2 - y * y) + e2 * ap) / d;
    d22 = 2.0 * e2 * ((1.0 - y * y) * ap + as) / d;
    d12 = 0.0;
    d33 = 2.0 * as;
  } else {
    y = sqrt(1.0 + (e2 - 1.0) * st * st);
    const double bs = sqrt(e2 - 1.0) * st;
    const double ap = sqrt(e2 - 1.0) * ct / eta;
    const double d = e2 + 1.0 - y * y;
    jac = (e2 - 1.0) * st * ct / y * wt;
    d11 = 2.0 * e2 * ap / d;
    d22 = 2.0 * e2 * (1.0 - y * y) * ap / d;
    d12 = -2.0 * e2 * bs * ap / d;
    d33 = 0.0;
  }
  // (2/pi) * sin(y dT / 2) / y * density * jacobian
  const double f = 0.63661977236758134 * sin(0.5 * y * dT) / y * jac;
  n.y = y;
  n.g11 = f * d11;
  n.g12 = f * d12;
  n.g22 = f * d22;
  n.g33 = f * d33;
  n.ph_hi = y * dT;                    // y dT = ph_hi + ph_lo exactly
  n.ph_lo = fma(y, dT, -n.ph_hi);
  // the phase step between the lags of one thread, kTabThreads y dT (exact scaling)
  sincos(reduce_two_pi(kTabThreads * n.ph_hi, kTabThreads * n.ph_lo), &n.s_step, &n.c_step);
  return n;
}

// w_ab,j = sum_nodes g_ab cos or sin((j + 1/2) y dT).  A thread takes lags
// j, j + kTabThreads, ..., j + (kTabLags-1) kTabThreads.  For the first the
// phase is formed as a double-double and reduced by 2 pi (reduce_two_pi) and
// its sine and cosine evaluated; each next one is that pair rotated by the
// node's phase step (at most kTabLags-1 rotations, a few ulps).
template <typename R>
__global__ __launch_bounds__(kTabThreads) void tabulate_kernel(
    typename W4<R>::T *__restrict__ table, const long long *__restrict__ cls_off,
    const double *__restrict__ cls_q, const int *__restrict__ cls_w, double cs, double dt,
    double eta, double rate, const double *__restrict__ gl_x, const double *__restrict__ gl_w) {
  __shared__ Node nodes[kTabThreads];
  const int c = blockIdx.x;
  const int W = cls_w[c];
  const double q = cls_q[c];
  const double dT = q * cs * dt;
  const double tmax = dT * W * rate;
  const int npan = max(1, static_cast<int>(ceil(tmax / 40.0)));
  const int nnodes = 2 * npan * kGaussN;
  constexpr int span = kTabThreads * kTabLags;
  for (int jb = 0; jb <= W; jb += span) {  // j = W: the zero row
    const int j0 = jb + threadIdx.x;
    // lags of this thread inside the window
    const int nl = j0 < W ? min(kTabLags, (W - 1 - j0) / kTabThreads + 1) : 0;
    const double m = j0 + 0.5;
    double w[kTabLags][4];
#pragma unroll
    for (int t = 0; t < kTabLags; ++t) w[t][0] = w[t][1] = w[t][2] = w[t][3] = 0.0;
    for (int nb = 0; nb < nnodes; nb += kTabThreads) {
      __syncthreads();
      if (nb + threadIdx.x < nnodes)
        nodes[threadIdx.x] = make_node(nb + threadIdx.x, npan, eta, dT, gl_x, gl_w);
      __syncthreads();
      const int cnt = min(kTabThreads, nnodes - nb);
      if (nl > 0) {
        for (int i = 0; i < cnt; ++i) {
          const Node &nd = nodes[i];
          const double p_hi = m * nd.ph_hi;
          const double p_lo = fma(m, nd.ph_lo, fma(m, nd.ph_hi, -p_hi));
          double sn, cn;
          sincos(reduce_two_pi(p_hi, p_lo), &sn, &cn);
#pragma unroll
          for (int t = 0; t < kTabLags; ++t) {
            if (t >= nl) break;
            w[t][0] = fma(nd.g11, cn, w[t][0]);
            w[t][1] = fma(nd.g12, sn, w[t][1]);
            w[t][2] = fma(nd.g22, cn, w[t][2]);
            w[t][3] = fma(nd.g33, cn, w[t][3]);
            const double c2 = fma(cn, nd.c_step, -sn * nd.s_step);
            sn = fma(sn, nd.c_step, cn * nd.s_step);
            cn = c2;
          }
        }
      }
    }
#pragma unroll
    for (int t = 0; t < kTabLags; ++t) {
      const int j = j0 + t * kTabThreads;
      if (t < nl) {
        typename W4<R>::T o;
        o.x = static_cast<R>(w[t][0]);
        o.y = static_cast<R>(w[t][1]);
        o.z = static_cast<R>(w[t][2]);
        o.w = static_cast<R>(w[t][3]);
        table[cls_off[c] + j] = o;
      }
      if (j == W) table[cls_off[c] + W] = typename W4<R>::T{R(0), R(0), R(0), R(0)};
    }
  }
}

template <typename R, int S, int T, bool COMP>
hipError_t step_launch_s(const sbim_handle *h, const Group &g, const SweepArgs &sa0,
                         const ModeArgs &ma, long long mode_blocks, hipEvent_t ev0, hipEvent_t ev1) {
  constexpr int D = S * T;
  SweepArgs sa = sa0;
  const int phase = static_cast<int>((sa.step + 1) % D);
  sa.nphase = g.nblocks > phase ? (g.nblocks - phase + D - 1) / D : 0;
  const long long sweep_items =
      (sa.nphase + 7) / 8 * 8 * (sweep_lag_groups<R, S, T, COMP>() * T) * g.np;
  const long long items = sweep_items + xcd_chunk_ids(mode_blocks * g.np);
  if (items == 0) return hipSuccess;
  if (ev0) {
    const hipError_t e = hipEventRecord(ev0, h->stream);
    if (e != hipSuccess) return e;
  }
  // Long blocks are split over wavefronts where the launch would wait for one of them: a
  // lag of a chain takes about 0.33 us, a mode and plane of the whole launch 0.13 ns on a
  // full chip.  So, with windows per mode, from 32 lags (float64: 36; the split costs 2 to 11
  // per cent at 26 and saves 3 to 8 at 42: 256^2, float32 34.0 and 35.9 us at 26, 38.2 and
  // 34.5 at 42) and above one lag of the longest window per 2500 modes and planes (compensated, unsplit against split: 2048^2 x 2 at 400 lags 763 and
  // 830 us a step, 2048^2 x 2 at 2000 913 and 829, 1024^2 at 300 184 and 125); with one
  // window, while the sweep has at most a wavefront per CU (float64: 256^2 at 60 lags 49
  // and 37 us, 512^2 at 40 61 and 65) and lags enough so far (256 x 64: float32 at 20 lags
  // 26.5 and 25.7, compensated at 28 29.2 and 30.7, at 34 31.5 and 31.0).
  // A handle that sums in order keeps its chains whole.
  if constexpr (S == 6 || (S * T == 8 && sizeof(R) == 4 && !COMP)) {
    const int per_blk = sweep_lag_groups<R, S, T, COMP>() * T * g.np;
    const long long lags = std::min<long long>(g.wmax, sa.step + 1);  // of the longest chain so far
    long long nlong = 0;
    if (h->cfg.window_mode == SBIM_W_PER_MODE) {
      if (lags >= (sizeof(R) == 8 ? 36 : 32) && lags * 2500 > g.M * g.np) {  // (blocks stand in order of falling window)
        const long long all = std::partition_point(g.h_blk_cap.begin(), g.h_blk_cap.end(),
                                                   [](int cap) { return cap > kLongWindow; }) -
                              g.h_blk_cap.begin();
        nlong = all > phase ? (all - phase + D - 1) / D : 0;
      }
    } else if (lags >= (COMP ? 32 : 20) && sa.nphase * per_blk <= 256) {
      nlong = sa.nphase;
    }
    if (nlong > 0 && !h->in_order) {
      const long long long_wgs = (nlong + 7) / 8 * 8 * per_blk;
      const long long rest = (sa.nphase - nlong + kSplit - 1) / kSplit;
      const long long sweep_wgs = long_wgs + (rest + 7) / 8 * 8 * per_blk;
      const long long wgs = sweep_wgs + xcd_chunk_ids((mode_blocks * g.np + kSplit - 1) / kSplit);
      hipLaunchKernelGGL((step_kernel_split<R, S, T, COMP>), dim3(static_cast<unsigned>(wgs)),
                         dim3(kSplit * kLanes), 0, h->stream, sa, ma, long_wgs, sweep_wgs, nlong,
                         mode_blocks);
      const hipError_t e = hipGetLastError();
      return e == hipSuccess && ev1 ? hipEventRecord(ev1, h->stream) : e;
    }
  }
  if constexpr (sizeof(R) == 4 && S == 6 && T == 2) {
    // Staged history: windows of a few stages or more (one window: every block's is the
    // same), a block's ring within 32-bit byte offsets (its slots are at most a phase's
    // blocks apart).  Never slower (step_kernel_staged).
    const double block_span = static_cast<double>(g.wmax) * ((g.nblocks + D - 1) / D) * g.np * 3 * kLanes * 8;
    if (h->cfg.window_mode == SBIM_W_FIXED && g.wmax >= 64 && block_span < 4.29e9) {
      hipLaunchKernelGGL((step_kernel_staged<COMP>), dim3(static_cast<unsigned>(items)), dim3(kLanes),
                         2 * kStageBytes, h->stream, sa, ma, sweep_items, mode_blocks);
      const hipError_t e = hipGetLastError();
      return e == hipSuccess && ev1 ? hipEventRecord(ev1, h->stream) : e;
    }
  }
  if constexpr (!COMP && sizeof(R) == 4 && S == 6 && T == 2)
    hipLaunchKernelGGL((step_kernel_w4<R, S, T, COMP>), dim3(static_cast<unsigned>(items)),
                       dim3(kLanes), 0, h->stream, sa, ma, sweep_items, mode_blocks);
  else if constexpr (COMP && S <= 6)
    hipLaunchKernelGGL((step_kernel_w2<R, S, T, COMP>), dim3(static_cast<unsigned>(items)),
                       dim3(kLanes), 0, h->stream, sa, ma, sweep_items, mode_blocks);
  else
    hipLaunchKernelGGL((step_kernel<R, S, T, COMP>), dim3(static_cast<unsigned>(items)),
                       dim3(kLanes), 0, h->stream, sa, ma, sweep_items, mode_blocks);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && ev1) e = hipEventRecord(ev1, h->stream);
  return e;
}

template <typename R, bool COMP>
hipError_t step_launch_r(const sbim_handle *h, const Group &g, const SweepArgs &sa,
                         const ModeArgs &ma, long long mode_blocks, hipEvent_t ev0, hipEvent_t ev1) {
  switch (h->depth) {
    case 1: return step_launch_s<R, 1, 1, COMP>(h, g, sa, ma, mode_blocks, ev0, ev1);
    case 2: return step_launch_s<R, 2, 1, COMP>(h, g, sa, ma, mode_blocks, ev0, ev1);
    case 4: return step_launch_s<R, 4, 1, COMP>(h, g, sa, ma, mode_blocks, ev0, ev1);
    case 6: return step_launch_s<R, 6, 1, COMP>(h, g, sa, ma, mode_blocks, ev0, ev1);
    case 8: return step_launch_s<R, 8, 1, COMP>(h, g, sa, ma, mode_blocks, ev0, ev1);
    case 12: return step_launch_s<R, 6, 2, COMP>(h, g, sa, ma, mode_blocks, ev0, ev1);
    case 16: return step_launch_s<R, 8, 2, COMP>(h, g, sa, ma, mode_blocks, ev0, ev1);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// The recent ring of the matrix-core form follows the blocks' rings.
void *recent_ring(const sbim_handle *h, const Group &g, void *ring) {
  return static_cast<char *>(ring) +
         g.ring_records * g.np * 3LL * kLanes * 2 * static_cast<long long>(h->rsize);
}

// The middle level's sums follow the depth + 1 slots of the pending sums.
void *mid_sums(const sbim_handle *h, const Group &g, void *pending) {
  return static_cast<char *>(pending) +
         (h->depth + 1LL) * g.np * kSums * g.M * static_cast<long long>(h->rsize);
}

hipError_t launch_step(const sbim_handle *h, const Group &g, const StepLaunch &w,
                       hipEvent_t ev0, hipEvent_t ev1) {
  ModeArgs ma;
  ma.spec = w.spec;
  ma.spec_v = w.spec_v;
  ma.ring = w.ring;
  ma.recent = h->tiled ? recent_ring(h, g, w.ring) : nullptr;
  ma.nblocks = g.nblocks;
  ma.state = reinterpret_cast<double2 *>(w.state);
  ma.pending = w.pending;
  ma.table = g.table;
  ma.mid = h->tiled ? mid_sums(h, g, w.pending) : nullptr;
  ma.row0 = g.row0;
  ma.win = g.win;
  ma.nat = g.nat;
  ma.geom = g.geom;
  ma.blk_off = g.blk_off;
  ma.blk_cap = g.blk_cap;
  ma.blk_stride = g.blk_stride;
  ma.lam = reinterpret_cast<double2 *>(w.lam);
  ma.out_a = w.out_a;
  ma.out_b = w.out_b;
  ma.M = g.M;
  ma.nh = w.nh;
  ma.step = w.step;
  ma.np = g.np;
  ma.depth = h->depth;
  ma.inv_dt = 1.0 / w.dt;
  ma.vel_rule = w.vel_rule;
  ma.state_rule = w.state_rule;
  ma.p0 = g.pl[0];
  ma.p1 = g.np > 1 ? g.pl[1] : g.pl[0];
  SweepArgs sa;
  sa.ring = w.ring;
  sa.table = g.table;
  sa.pending = w.pending;
  sa.mid = const_cast<void *>(ma.mid);
  sa.row0 = g.row0;
  sa.win = g.win;
  sa.blk_off = g.blk_off;
  sa.blk_cap = g.blk_cap;
  sa.blk_stride = g.blk_stride;
  sa.cls_w0 = g.wmax;
  sa.M = g.M;
  sa.step = w.step;
  sa.np = g.np;
  sa.nphase = 0;
  const long long mode_blocks = w.sums_only ? 0 : g.nblocks;
  if (h->tiled) return launch_step_quads(h, g, sa, ma, mode_blocks, ev0, ev1);
  if (h->mfma) return launch_step_pairs(h, g, sa, ma, mode_blocks, ev0, ev1);
  if (h->fp64) return step_launch_r<double, false>(h, g, sa, ma, mode_blocks, ev0, ev1);
  if (h->comp) return step_launch_r<float, true>(h, g, sa, ma, mode_blocks, ev0, ev1);
  return step_launch_r<float, false>(h, g, sa, ma, mode_blocks, ev0, ev1);
}

hipError_t launch_tabulate(bool fp64, const Group &g, double dt, const double *gl_x,
                           const double *gl_w, hipStream_t st) {
  if (g.nclasses == 0) return hipSuccess;
  const double rate = fmax(1.0, (g.eta * g.eta - 1.0) / 2.0);
  if (fp64) {
    hipLaunchKernelGGL(tabulate_kernel<double>, dim3(static_cast<unsigned>(g.nclasses)), dim3(kTabThreads),
                       0, st, static_cast<double4 *>(g.table), g.cls_off, g.cls_q, g.cls_w, g.cs, dt,
                       g.eta, rate, gl_x, gl_w);
  } else {
    hipLaunchKernelGGL(tabulate_kernel<float>, dim3(static_cast<unsigned>(g.nclasses)), dim3(kTabThreads),
                       0, st, static_cast<float4 *>(g.table), g.cls_off, g.cls_q, g.cls_w, g.cs, dt,
                       g.eta, rate, gl_x, gl_w);
  }
  return hipGetLastError();
}

}  // namespace sbim

