// Device code shared by the step launches (kernels.hip, quads.hip, pairs.hip): lag
// sums and the mode item of a step.
#pragma once

#include <type_traits>

#include "internal.h"

namespace sbim {
namespace {

template <typename R> struct C2;
template <> struct C2<float> { using T = float2; };
template <> struct C2<double> { using T = double2; };
template <typename R> using cplx = typename C2<R>::T;

template <typename R> struct W4;
template <> struct W4<float> { using T = float4; };
template <> struct W4<double> { using T = double4; };

// step mod n: in 32 bits while the step number fits (the 64-bit remainder is a
// long software sequence).
__device__ __forceinline__ int mod_step(long long step, int n) {
  if (step < (1LL << 31)) return static_cast<int>(static_cast<unsigned>(step) % static_cast<unsigned>(n));
  return static_cast<int>(step % n);
}

// ------------------------------------------------------------------ conv

// Neumaier's compensated addition: s + x with the rounding error kept in c.
__device__ __forceinline__ void neumaier(float &s, float &c, float x) {
  const float t = s + x;
  if (fabsf(s) >= fabsf(x))
    c += (s - t) + x;
  else
    c += (x - t) + s;
  s = t;
}

// Accumulator of one real history sum: plain (T = R) or compensated (float pair).
template <typename R, bool COMP> struct Acc;
template <typename R> struct Acc<R, false> {
  R s = R(0);
  __device__ __forceinline__ void fold(R x) { s += x; }
  __device__ __forceinline__ R value() const { return s; }
  __device__ __forceinline__ void fold(const Acc &a) { s += a.s; }
  // add the accumulator of the lane `off` lanes away (butterfly reduction)
  __device__ __forceinline__ void fold_lane(int off) { s += __shfl_xor(s, off); }
};
template <> struct Acc<float, true> {
  float s = 0.f, c = 0.f;
  // Kahan's compensated addition (c holds the part of the sum lost by s)
  __device__ __forceinline__ void fold(float x) {
    const float y = x + c;
    const float t = s + y;
    c = y - (t - s);
    s = t;
  }
  __device__ __forceinline__ float value() const { return s + c; }
  __device__ __forceinline__ void fold(const Acc &a) {
    neumaier(s, c, a.s);
    c += a.c;
  }
  __device__ __forceinline__ void fold_lane(int off) {
    const float s2 = __shfl_xor(s, off);
    const float c2 = __shfl_xor(c, off);
    neumaier(s, c, s2);
    c += c2;
  }
};

// Five complex history sums per plane: C11[U_L], C12[U_N], C22[U_N], C12[U_L], C33[U_T].
constexpr int kSums = 10;  // real accumulators per plane

// part[.] += w * u for the five history sums of one plane.
template <typename R>
__device__ __forceinline__ void fma_lag(R (&part)[kSums], const typename W4<R>::T &w,
                                        const cplx<R> (&u)[3]) {
  part[0] = fma(w.x, u[0].x, part[0]);
  part[1] = fma(w.x, u[0].y, part[1]);
  part[2] = fma(w.y, u[1].x, part[2]);
  part[3] = fma(w.y, u[1].y, part[3]);
  part[4] = fma(w.z, u[1].x, part[4]);
  part[5] = fma(w.z, u[1].y, part[5]);
  part[6] = fma(w.y, u[0].x, part[6]);
  part[7] = fma(w.y, u[0].y, part[7]);
  part[8] = fma(w.w, u[2].x, part[8]);
  part[9] = fma(w.w, u[2].y, part[9]);
}

// A value equal on every lane, moved to a scalar register.
__device__ __forceinline__ long long uniform64(long long v) {
  const unsigned lo = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(v));
  const unsigned hi = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(static_cast<unsigned long long>(v) >> 32));
  return static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo);
}

// Word 3 of a raw buffer resource on gfx9-family chips (data format 32 bits,
// no swizzle): what untyped dword loads through __builtin_amdgcn_make_buffer_rsrc need.
constexpr int kBufferWord3 = 0x00020000;
// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), in order.
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>());
  }
}

// The time-tiled ring of the matrix-core form, per block b:
//   [tile][plane][component L,N,T][64 lanes][re, im][TS steps].
// Step n takes slot (n + ring_shift(b)) mod cap (cap a multiple of TS), tile
// slot / TS, element slot mod TS; the shift lets tiles end at the steps t0-2 of the
// block's sweeps and middle levels (t0 = b mod TS) and staggers the blocks.  A tile is
// written once, whole, by the mode item of its last step; the newest steps wait in
// the "recent" ring, [step mod kRecent][block][plane][component][64 lanes] complex,
// which the mode items read.  (Writing each step into its tile instead touched every
// cache line of the tile on each of its steps: 1024^2 x 2 planes, float32: 46 us of a
// step.)
template <typename R> struct RingTile {
  static constexpr int TS = kRingTileBytes / static_cast<int>(sizeof(R));
  typedef R V __attribute__((ext_vector_type(TS)));
};
template <typename R, typename I>
__device__ __forceinline__ int ring_shift(I b) {
  constexpr int TS = RingTile<R>::TS;
  return static_cast<int>((TS + 1 - b % TS) % TS);
}

// A lane's part of the time-tiled ring: its (plane, lane) of the block's tile 0.
template <typename R>
__device__ __forceinline__ const typename RingTile<R>::V *ring_tile(const void *ring, long long blk_off,
                                                                    int np, int p, int lane) {
  return static_cast<const typename RingTile<R>::V *>(ring) +
         (blk_off / RingTile<R>::TS * np + p) * 3 * kLanes * 2 + lane * 2;
}
// The TS steps of tile x for the three components, real and imaginary parts.
template <typename R>
__device__ __forceinline__ void load_tile(typename RingTile<R>::V (&h)[3][2],
                                          const typename RingTile<R>::V *__restrict__ rp, int x, int np) {
  const typename RingTile<R>::V *q = rp + static_cast<long long>(x) * np * 3 * kLanes * 2;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    h[c][0] = q[c * kLanes * 2];
    h[c][1] = q[c * kLanes * 2 + 1];
  }
}

// Pending sum t of position s: one complex array per sum, [slot][plane][5][M], or beside the
// float64 vector sweep two real ones, [slot][plane][10][M] (1024 x 512 x 2, 128 lags: a launch
// 173.3 us with complex sums, 168.1 so; float32 1024 x 512 x 2, 5 lags, 51.3 and 52.3).
// `row`: 5 (slot planes + plane).
template <typename R, bool TILED> constexpr bool kRealSums = sizeof(R) == 8 && !TILED;
template <typename R, bool TILED>
__device__ __forceinline__ void store_sum(void *pending, long long row, int t, long long M, long long s, cplx<R> v) {
  if constexpr (kRealSums<R, TILED>) {
    R *q = static_cast<R *>(pending) + (row + t) * 2 * M + s;
    q[0] = v.x;
    q[M] = v.y;
  } else {
    static_cast<cplx<R> *>(pending)[(row + t) * M + s] = v;
  }
}
template <typename R, bool TILED>
__device__ __forceinline__ cplx<R> load_sum(const void *pending, long long row, int t, long long M, long long s) {
  if constexpr (kRealSums<R, TILED>) {
    const R *q = static_cast<const R *>(pending) + (row + t) * 2 * M + s;
    return cplx<R>{q[0], q[M]};
  } else {
    return static_cast<const cplx<R> *>(pending)[(row + t) * M + s];
  }
}

// Mode item of step n for one (mode, plane): the push, then the traction of
// the same step from the same registers.
//   push:    rotate the new spectrum into the wavevector frame, update the
//            float64 running state, store the ring slot of step n;
//   traction: the pending history sum of step n plus the lags from the
//            block's last sweep on (compensated for the compensated form),
//            damping and instantaneous terms, rotation back to (x1, x2, x3),
//            scatter into the natural half-spectrum layout.
// The lag-0 history value and the velocity of the damping term are the ones
// just computed (rounded to the working precision as the ring stores them).
template <typename R, bool COMP, bool TILED>
__device__ __forceinline__ void mode_step(const ModeArgs &a, int p, long long s) {
  using W = typename W4<R>::T;
  constexpr bool EARLY = TILED || COMP;  // (below)
  const double2 *__restrict__ spec = static_cast<const double2 *>(a.spec);
  const double2 *__restrict__ spec_v = static_cast<const double2 *>(a.spec_v);
  cplx<R> *__restrict__ ring = static_cast<cplx<R> *>(a.ring);
  double2 *__restrict__ state = a.state;
  const long long M = a.M, nh = a.nh, step = a.step;
  const int np = a.np;
  // What a step reads beside the spectrum and the state (window, kernel rows, sums) is
  // asked for at once in the matrix-core and compensated forms (2048^2 x 2, windows per
  // mode, compensated, us a step: 769 so, 782 after the push); beside the plain vector
  // sweeps, after the push: their chains of dependent loads are the launch's length, and
  // the fewer loads the mode items have in flight the shorter they are (a launch at once /
  // after: float64 512^2, two materials, 40 lags, 30.0 / 29.2; float32 512^2 x 2, 5 lags,
  // 25.7 / 24.3).
  const int natural = a.nat[s];
  if (!EARLY && natural < 0) return;  // a padding position of the matrix-core layout: no mode
  int wl = 0;
  long long row0 = 0;
  if constexpr (EARLY) {
    wl = a.win[s];
    row0 = a.row0[s];
  }
  const double4 geom = *reinterpret_cast<const double4 *>(a.geom + 4 * s);
  const int b = EARLY ? __builtin_amdgcn_readfirstlane(static_cast<int>(s >> 6)) : static_cast<int>(s >> 6);
  const int lane = static_cast<int>(s & 63);
  const int cap = a.blk_cap[b];
  const long long base = a.blk_off[b];
  const long long stride = a.blk_stride[b];
  const long long rec_len = static_cast<long long>(np) * 3 * kLanes;
  // slot of step n: in the block's ring, or in the recent ring of the matrix-core form
  const int x0 = TILED ? mod_step(step, kRecent) : (cap > 0 ? mod_step(step, cap) : 0);
  const PlaneParams &pp = p == 0 ? a.p0 : a.p1;
  const int pg = pp.index;

  // ---- where the history sums of step n come from
  // The sweep launched with step m-1 covers steps m .. m+D-1 (m = b mod D, m >= 1)
  // over the history up to step m-2, and with a middle level the launch of step m-1,
  // m = b mod kMidPeriod, adds the entries since that sweep.  Lags not in those sums:
  // from step m-1 on, or all of them before the block's first launch of either kind.
  int fresh = 0;
  cplx<R> pend[5], midv[5];
  const auto load_sums = [&]() {
    const int S = a.depth;
    const int since = mod_step(step + S - b % S, S);  // steps since m
    const bool swept = step - since >= 1 && cap > kDirectLags;
    fresh = swept ? since + 2 : static_cast<int>(min(step + 1, 1LL << 30));
    bool mids = false;
    if (TILED && cap > kDirectLags) {
      const int e = since % kMidPeriod;
      mids = step - e >= 1 && since >= kMidPeriod;
      if (step - e >= 1) fresh = e + 2;
    }
    fresh = min(wl, fresh);
#pragma unroll
    for (int t = 0; t < 5; ++t) pend[t] = midv[t] = cplx<R>{R(0), R(0)};
    if (swept && (wl > 0 || !TILED)) {
      const long long row = (mod_step(step, S + 1) * np + p) * 5LL;
#pragma unroll
      for (int t = 0; t < 5; ++t) pend[t] = load_sum<R, TILED>(a.pending, row, t, M, s);
    }
    if (mids && wl > 0) {
      const cplx<R> *__restrict__ q = static_cast<const cplx<R> *>(a.mid) +
                                      (mod_step(step, kMidPeriod + 1) * np + p) * 5LL * M + s;
#pragma unroll
      for (int t = 0; t < 5; ++t) midv[t] = q[t * M];
    }
  };
  if constexpr (EARLY) load_sums();
  if (EARLY && natural < 0) return;
  const double q = geom.x, kh1 = geom.y, kh3 = geom.z;

  // record of one step: of the block's ring, or of the recent ring
  cplx<R> *const first = ring + base * rec_len + static_cast<long long>(p) * 3 * kLanes + lane;
  const auto slot = [&](int x) {
    if constexpr (TILED)
      return static_cast<cplx<R> *>(a.recent) + (static_cast<long long>(x) * a.nblocks + b) * rec_len +
             static_cast<long long>(p) * 3 * kLanes + lane;
    else
      return first + static_cast<long long>(x) * stride * rec_len;
  };

  // ---- push
  cplx<R> u0[3], v0[3];
  {
    double2 x[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) x[c] = spec[(pg * 3 + c) * nh + natural];
    // (1, 2, 3) -> (L, N, T)
    const double2 xr[3] = {{kh1 * x[0].x + kh3 * x[2].x, kh1 * x[0].y + kh3 * x[2].y},
                           x[1],
                           {-kh3 * x[0].x + kh1 * x[2].x, -kh3 * x[0].y + kh1 * x[2].y}};
    double2 vr[3];
    if (a.vel_rule == VEL_INPUT) {
      double2 y[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) y[c] = spec_v[(pg * 3 + c) * nh + natural];
      vr[0] = double2{kh1 * y[0].x + kh3 * y[2].x, kh1 * y[0].y + kh3 * y[2].y};
      vr[1] = y[1];
      vr[2] = double2{-kh3 * y[0].x + kh1 * y[2].x, -kh3 * y[0].y + kh1 * y[2].y};
    }
    cplx<R> *rp = slot(x0);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const long long si = (static_cast<long long>(p) * 3 + c) * M + s;
      const double2 prev = state[si];
      double2 now;
      if (a.state_rule == STATE_ACCUM)
        now = double2{prev.x + xr[c].x, prev.y + xr[c].y};
      else
        now = xr[c];
      state[si] = now;
      double2 v;
      if (a.vel_rule == VEL_DIFF)
        v = double2{(now.x - prev.x) * a.inv_dt, (now.y - prev.y) * a.inv_dt};
      else if (a.vel_rule == VEL_SCALE)
        v = double2{xr[c].x * a.inv_dt, xr[c].y * a.inv_dt};
      else if (a.vel_rule == VEL_INPUT)
        v = vr[c];
      else if (a.vel_rule == VEL_ZERO)
        v = double2{0.0, 0.0};
      else
        v = xr[c];
      v0[c] = cplx<R>{static_cast<R>(v.x), static_cast<R>(v.y)};
      u0[c] = cplx<R>{static_cast<R>(now.x), static_cast<R>(now.y)};
      if (cap > 0) rp[c * kLanes] = u0[c];
    }
  }

  // ---- history sums of step n
  if constexpr (!EARLY) {
    wl = a.win[s];
    load_sums();
  }
  R cs[kSums];
  {
    Acc<R, COMP> acc[kSums];
#pragma unroll
    for (int t = 0; t < 5; ++t) {
      acc[2 * t].s = pend[t].x;
      acc[2 * t + 1].s = pend[t].y;
      if constexpr (TILED) {
        acc[2 * t].fold(midv[t].x);
        acc[2 * t + 1].fold(midv[t].y);
      }
    }
    if (fresh > 0) {
      // the newest lags: plain products (the compensated form folds their sum,
      // at most depth + 1 or kMidPeriod + 1 lags, into the pending sum once)
      const W *__restrict__ rowp = static_cast<const W *>(a.table) + (EARLY ? row0 : a.row0[s]);
      R part[kSums];
#pragma unroll
      for (int k = 0; k < kSums; ++k) part[k] = COMP ? R(0) : acc[k].s;
      fma_lag<R>(part, rowp[0], u0);
      // The older lags in batches of FB, every load of a batch in flight before
      // its products: the lag index is clamped (fresh <= W <= cap, so the ring
      // slot stays in the block's ring), the loads need no branch, and lags
      // past `fresh` take zero weights, which leave the sums unchanged.
      constexpr int FB = 4;  // measured on gfx950: as fast as 8 with fewer registers
      const int wrap = TILED ? kRecent : cap;
      // the step that completes a tile needs the TS - 1 steps before it as well
      constexpr int TS = RingTile<R>::TS;
      int tile_slot = 0;
      bool tile = false;
      if constexpr (TILED) {
        tile_slot = mod_step(step + ring_shift<R>(b), cap);
        tile = tile_slot % TS == TS - 1;
      }
      const int last = tile ? max(fresh, TS) - 1 : fresh - 1;
      for (int j0 = 1; j0 <= last; j0 += FB) {
        cplx<R> u[FB][3];
        W w[FB];
#pragma unroll
        for (int i = 0; i < FB; ++i) {
          const int j = min(j0 + i, last);
          int x = x0 - j;
          if (x < 0) x += wrap;
          const cplx<R> *qp = slot(x);
          u[i][0] = qp[0];
          u[i][1] = qp[kLanes];
          u[i][2] = qp[2 * kLanes];
          w[i] = rowp[TILED ? min(j, wl) : j];
        }
#pragma unroll
        for (int i = 0; i < FB; ++i) {
          const bool on = j0 + i < fresh;
          const W wi = {on ? w[i].x : R(0), on ? w[i].y : R(0), on ? w[i].z : R(0),
                        on ? w[i].w : R(0)};
          fma_lag<R>(part, wi, u[i]);
        }
        if constexpr (TILED) {
          static_assert(TS - 1 <= FB, "the first batch holds the rest of the tile");
          if (tile && j0 == 1) {
            typename RingTile<R>::V *tp = const_cast<typename RingTile<R>::V *>(
                ring_tile<R>(a.ring, base, np, p, lane)) +
                static_cast<long long>(tile_slot / TS) * np * 3 * kLanes * 2;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              typename RingTile<R>::V re, im;
              re[TS - 1] = u0[c].x;
              im[TS - 1] = u0[c].y;
#pragma unroll
              for (int e = 1; e < TS; ++e) {
                re[TS - 1 - e] = u[e - 1][c].x;
                im[TS - 1 - e] = u[e - 1][c].y;
              }
              tp[c * kLanes * 2] = re;
              tp[c * kLanes * 2 + 1] = im;
            }
          }
        }
      }
#pragma unroll
      for (int k = 0; k < kSums; ++k) {
        if constexpr (COMP)
          acc[k].fold(part[k]);
        else
          acc[k].s = part[k];
      }
    }
#pragma unroll
    for (int k = 0; k < kSums; ++k) cs[k] = acc[k].value();
  }

  // ---- traction of step n
  const R sg = static_cast<R>(pp.side);
  const R muq = static_cast<R>(pp.mu * q);
  const R damp = static_cast<R>(pp.mu / pp.cs);
  const R inst = static_cast<R>((2.0 - pp.eta) * pp.mu * q);
  const R eta = static_cast<R>(pp.eta);
  const R r1 = static_cast<R>(kh1), r3 = static_cast<R>(kh3);
  cplx<R> u[3] = {{R(0), R(0)}, {R(0), R(0)}, {R(0), R(0)}};
  if (cap > 0 && wl > 0) {
#pragma unroll
    for (int c = 0; c < 3; ++c) u[c] = u0[c];
  }
  // conv + instantaneous (rotated frame):
  //   A_L = -sg mu q C11 + i (2-eta) mu q U_N - i mu q C12[U_N]
  //   A_N = -sg mu q C22 - i (2-eta) mu q U_L + i mu q C12[U_L]
  //   A_T = -sg mu q C33
  cplx<R> t[3];
  t[0] = cplx<R>{-sg * muq * cs[0] - inst * u[1].y + muq * cs[3],
                 -sg * muq * cs[1] + inst * u[1].x - muq * cs[2]};
  t[1] = cplx<R>{-sg * muq * cs[4] + inst * u[0].y - muq * cs[7],
                 -sg * muq * cs[5] - inst * u[0].x + muq * cs[6]};
  t[2] = cplx<R>{-sg * muq * cs[8], -sg * muq * cs[9]};
  // damping: -sg (mu/c_s) diag(1, eta, 1) V
  const cplx<R> d[3] = {{-sg * damp * v0[0].x, -sg * damp * v0[0].y},
                        {-sg * damp * eta * v0[1].x, -sg * damp * eta * v0[1].y},
                        {-sg * damp * v0[2].x, -sg * damp * v0[2].y}};
  if (a.lam) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const long long si = (static_cast<long long>(p) * 3 + c) * M + s;
      double2 l = a.lam[si];
      l.x += static_cast<double>(t[c].x);
      l.y += static_cast<double>(t[c].y);
      a.lam[si] = l;
      t[c] = cplx<R>{static_cast<R>(l.x), static_cast<R>(l.y)};
    }
  }
  cplx<R> *__restrict__ out_a = static_cast<cplx<R> *>(a.out_a);
  cplx<R> *__restrict__ out_b = static_cast<cplx<R> *>(a.out_b);
  if (!out_b) {
#pragma unroll
    for (int c = 0; c < 3; ++c) t[c] = cplx<R>{t[c].x + d[c].x, t[c].y + d[c].y};
  }
  // (L, N, T) -> (1, 2, 3)
  out_a[(pg * 3 + 0) * nh + natural] = cplx<R>{r1 * t[0].x - r3 * t[2].x, r1 * t[0].y - r3 * t[2].y};
  out_a[(pg * 3 + 1) * nh + natural] = t[1];
  out_a[(pg * 3 + 2) * nh + natural] = cplx<R>{r3 * t[0].x + r1 * t[2].x, r3 * t[0].y + r1 * t[2].y};
  if (out_b) {
    out_b[(pg * 3 + 0) * nh + natural] =
        cplx<R>{r1 * d[0].x - r3 * d[2].x, r1 * d[0].y - r3 * d[2].y};
    out_b[(pg * 3 + 1) * nh + natural] = d[1];
    out_b[(pg * 3 + 2) * nh + natural] =
        cplx<R>{r3 * d[0].x + r1 * d[2].x, r3 * d[0].y + r1 * d[2].y};
  }
}

// Mode items in XCD-contiguous order.  Work-group ids go round-robin over the 8
// XCDs, so id m of a launch's mode part (which starts at a multiple of 8) runs on
// XCD m mod 8; it takes item (m mod 8) * per + m / 8 of the n items, so each XCD
// works through a contiguous eighth of the sorted blocks (nearby q), whose
// natural-order spectrum gathers and traction scatters then share cache lines
// in that XCD's L2.  The mode part has 8 * per ids; the ones past n return.
__device__ __forceinline__ long long xcd_chunk(long long m, long long n) {
  return (m & 7) * ((n + 7) / 8) + (m >> 3);
}
inline long long xcd_chunk_ids(long long n) { return (n + 7) / 8 * 8; }

}  // namespace
}  // namespace sbim
