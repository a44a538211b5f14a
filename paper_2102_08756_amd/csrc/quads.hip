// The step launch with the history sweep on the matrix cores, for fixed windows:
// one launch per step of sweep work-groups (quad_sweep), middle-level items
// (mid_item) and mode items (step_items.h).
#include "step_items.h"

namespace sbim {
namespace {

// ------------------------------------------------------- matrix-core sweep

// Byte offset past every resource built here: a load there returns 0.
constexpr unsigned kBufferNone = 0xfffffff0u;

// The 16x16x4 product of each precision.  Operands: A[s][k] in lane s + 16 k,
// B[k][col] in lane col + 16 k; result row(l, v), column l mod 16 in lane l,
// element v (layouts measured on gfx950 with in-bounds probes; the two differ).
// Each result element rounds like the chain of four fused multiply-adds.
template <typename R> struct Mfma;
template <> struct Mfma<float> {
  typedef float V __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ V mul(float a, float b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
  static __device__ __forceinline__ V load16(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, static_cast<int>(off), 0, 0));
  }
  template <typename T>
  static __device__ __forceinline__ T loadv(__amdgpu_buffer_rsrc_t r, unsigned off) {
    if constexpr (sizeof(T) == 8)
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, static_cast<int>(off), 0, 0));
    else
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(r, static_cast<int>(off), 0, 0));
  }
};
template <> struct Mfma<double> {
  typedef double V __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ V mul(double a, double b, V c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) + 4 * v; }
  typedef double V2 __attribute__((ext_vector_type(2)));
  static __device__ __forceinline__ V2 load16(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(V2, __builtin_amdgcn_raw_buffer_load_b128(r, static_cast<int>(off), 0, 0));
  }
  template <typename T>
  static __device__ __forceinline__ T loadv(__amdgpu_buffer_rsrc_t r, unsigned off) {
    if constexpr (sizeof(T) == 16) {
      return load16(r, off);
    } else {
      const V2 a = load16(r, off), b = load16(r, off + 16u);
      return T{a[0], a[1], b[0], b[1]};
    }
  }
};

// Orders the LDS accesses of one wavefront as written (the hardware executes them
// in order; this keeps the compiler to it across lanes).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The sweep on the matrix cores, for fixed windows (one window for every mode).
// Its sums are the same as sweep_item's: the launch of step n serves steps
// t0 = n+1 .. n+D from the history up to step n-1,
//   pending[(t0+u) mod (D+1)] = sum_{i>=2} w_{i+u} (x) U^{t0-i},
// but per class of modes the product over lags is a Toeplitz matrix times a
// matrix of history columns, done as 16x16x4 products (one per 4 lags and 16
// steps).
//
// Classes are padded to multiples of CM sorted positions (CM = 4, or 2 on grids
// where only +-m1 share q), so the CM lanes CM j .. CM j + CM-1 of a block (its
// "quad" j) share one kernel row.  The 16 columns are (time group tg, plane p of
// the group's NP, mode mq of the quad, real/imaginary part), tg < TG = 8 / (CM NP).
// A shift of 16 lags turns the sum of one 16-step group into that of the next,
//   out[16 h + s] = sum_{i'} w[i' + s] U^{t0 - (i' - 16 h)},
// so every step group takes the same Toeplitz operand and only its history is
// delayed by 16 h lags: within the columns for tg (each lane loads its own lag),
// for the G accumulator groups of a wavefront by keeping the history operands of
// the last 4 TG (G-1) blocks in registers, and for the TW wavefronts that share a
// quad by their own lags.  D = 16 TG G TW steps in all.  Per 4 "row lags"
// i' = i0 .. i0+3 the operands are
//   A[s][k] = w_type[i0 + k + s]          (rows past the class's window are 0),
//   B[k][col] = U^{t0-(i0+k-16h)}[col]    (one real of the ring; 0 where the lag is under 2),
// and the five products per group are (w11, U_L), (w12, U_N), (w22, U_N),
// (w12, U_L), (w33, U_T) -> complex sums 0..4, as fma_lag orders them.
//
// The ring of this form is tiled in time (RingTile): 16 bytes hold TS consecutive
// steps of one real, so a lane's 16-byte load feeds TS products.  A "superblock" is
// 4 tiles (SB = 4 TS lags): lane (col, k) loads tile k of it, and product e takes
// element e of every lane, i.e. the lags TS + 1 + TS k - e, k = 0..3 (a block's tiles
// end at its sweeps: step t0-2 is the last element of its tile).  The row operands
// of neighbouring lanes and products overlap, so a wavefront stages its rows in LDS,
// 32 rows at a time, each read from memory once.  (With one real per load the sweep
// was bound by the issue of its loads: 1024^2 x 2 planes, W = 2000, float32: 759 us
// per step.)
//
// Work-group = QW (quad, step part) pairs of a block of this launch's phase, LG
// wavefronts each: consecutive ranges of the superblocks, summed in LDS in a fixed order
// (the compensated sums in float64), so results are bitwise reproducible.
// Work-group ids of one block are congruent mod 8, so they run on one XCD.
// Lags past min(W-1, t0) meet zero rows or never-written (zero) ring slots.
template <typename R, bool COMP, int NP, int CM, int G, int TW> struct QuadShape {
  static constexpr int TG = 8 / (CM * NP);
  static constexpr int D = 16 * TG * G * TW;
  static constexpr int NV = G * 5 * 4;  // real sums per lane
  using Sum = std::conditional_t<COMP, double, R>;
  // Superblocks loaded ahead, measured on gfx950: 2 (1 beside a delayed group); twice
  // as many with rounds of 64 rows are within 2% (512^2 and 1024^2, every form), and
  // 10% slower for the compensated form, whose registers then hold three wavefronts
  // per SIMD.
  static constexpr int kAhead = G > 1 ? 1 : 2;
  static constexpr int kRows = 32;      // kernel rows, and lags, per round
  // LDS of a wavefront: two chunks of kernel rows, then (the rows are no
  // longer needed) its partial sums
  static constexpr int kWaveLds = NV * kLanes * static_cast<int>(sizeof(Sum));
  static_assert(kWaveLds >= 2 * kRows * 4 * static_cast<int>(sizeof(R)), "rows fit the partial sums' space");
};

template <typename R, bool COMP, int NP, int CM, int G, int TW>
__device__ __forceinline__ void quad_sweep(const SweepArgs &a, long long wg, int LG, int QW,
                                           unsigned char *lds_raw) {
  using Shape = QuadShape<R, COMP, NP, CM, G, TW>;
  using M4 = Mfma<R>;
  using V = typename M4::V;
  using Sum = typename Shape::Sum;
  constexpr int TG = Shape::TG, D = Shape::D;
  constexpr int TS = RingTile<R>::TS;
  constexpr int SB = 4 * TS;                 // lags per superblock
  constexpr int NR = Shape::kRows / SB;      // superblocks per round
  constexpr int SH = 16 / TS;                // tiles of a 16-lag shift
  constexpr int HOLD = TG * 16 / SB * (G - 1);  // superblocks of history held back for the groups
  constexpr int AH = Shape::kAhead;          // superblocks loaded ahead
  constexpr int NB = HOLD + AH;              // history operand sets held
  static_assert(NR % NB == 0, "operand sets rotate within a round");
  // Wavefront w of the work-group: its qi-th (quad, step part), lag range chunk
  // (uniform: kept in scalar registers, so the loop control below is scalar).
  const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int chunk = w % LG, qi = w / LG;
  const int per_block = kLanes / CM * TW / QW;  // work-groups per block
  const int kb = static_cast<int>(wg / (8 * per_block)) * 8 + static_cast<int>(wg & 7);
  if (kb >= a.nphase) return;     // uniform over the work-group
  const int jt = static_cast<int>((wg >> 3) % per_block) * QW + qi;
  const int j = jt / TW, tw = jt % TW;  // quad of the block, step part
  const long long M = a.M;
  const long long t0 = a.step + 1;
  const long long b = t0 % D + static_cast<long long>(D) * kb;
  const int lane = threadIdx.x & 63;
  const int s_ = lane & 15;                 // A row (step in group) / B column
  const int k_ = lane >> 4;                 // lag within a 4-lag block
  const int reim = s_ & 1, mq = (s_ >> 1) & (CM - 1);
  const int p = (s_ / (2 * CM)) & (NP - 1), tg = s_ / (2 * CM * NP);
  const int h0 = tg + TG * G * tw;          // the lane's first 16-step group
  const long long sq = b * kLanes + CM * j;  // first sorted position of the quad
  // Past the last mode (M is a multiple of CM) a quad has no work; it still takes
  // part in the work-group's barrier below (uniform over the wavefront).
  const bool active = sq < M;
  const int cap = __builtin_amdgcn_readfirstlane(a.blk_cap[b]);
  // the class's window (its first position is a mode)
  const int wl = active ? __builtin_amdgcn_readfirstlane(a.win[sq]) : 0;
  // row lags up to min(W-1, t0 + D-16): the oldest history any step group needs
  const int ilast = wl > 0 ? static_cast<int>(min(static_cast<long long>(wl) - 1, t0 + D - 16)) : 0;
  const int nsb = ilast > 1 ? (ilast - 2) / SB + 1 : 0;
  // Ranges are whole rounds: past nsb a round meets zero rows or never-written
  // slots, so no superblock needs a guard.
  const int per = (nsb + LG * NR - 1) / (LG * NR) * NR;
  const int sb0 = min(nsb, chunk * per);
  const int sb1 = min(nsb, sb0 + per);
  unsigned char *wave_lds = lds_raw + w * Shape::kWaveLds;

  V C[G][5];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int t = 0; t < 5; ++t) C[g][t] = V{R(0), R(0), R(0), R(0)};
  Sum acc[G][5][4];
  if constexpr (COMP) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int t = 0; t < 5; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[g][t][v] = 0;
  }
  if (sb1 > sb0) {
    // The quad's operands come through buffer loads: a resource per wavefront
    // (the block's ring, the class's kernel rows) and a 32-bit byte offset per
    // lane; a load past the resource's range returns 0, which gives the zero
    // rows past the window and the masked lags.  (Buffer loads also keep the
    // compiler from moving a prefetch down to its use, which it does with plain
    // loads.  Every value a resource is built from is read as uniform, so that
    // the resources live in scalar registers.)
    constexpr unsigned row_bytes = 4 * sizeof(R);
    const R *rows = static_cast<const R *>(a.table) + 4 * uniform64(a.row0[sq]);
    const __amdgpu_buffer_rsrc_t rows_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<R *>(rows), 0, static_cast<int>(static_cast<unsigned>(wl) * row_bytes), kBufferWord3);
    // History: tile x of the block at x * tile_bytes (the host keeps the block's
    // ring below kBufferNone bytes).
    constexpr unsigned comp_bytes = kLanes * 2 * 16;
    constexpr unsigned tile_bytes = NP * 3 * comp_bytes;
    const int ntile = cap / TS;  // >= 4
    const char *ring = static_cast<const char *>(a.ring) +
                       uniform64(a.blk_off[b]) * (NP * 3LL * kLanes * 2 * static_cast<long long>(sizeof(R)));
    const __amdgpu_buffer_rsrc_t ring_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(ring), 0, static_cast<int>(static_cast<unsigned>(ntile) * tile_bytes),
        kBufferWord3);
    // Kernel rows: chunk c holds rows 2 + SB sb0 + kRows c .. in half c mod 2 of the
    // wavefront's LDS ring (a row past the class's window reads 0); a lane moves
    // kRows / 16 reals of it.  A round reads chunks c and c+1; chunk c+2 is in
    // flight meanwhile and replaces chunk c when the next round begins.  (LDS
    // instructions of a wavefront execute in order: no barrier is needed.)
    constexpr int ROWS = Shape::kRows;
    typedef R VP __attribute__((ext_vector_type(ROWS / 16)));
    const V *rows_lds = reinterpret_cast<const V *>(wave_lds);
    VP *rows_put = reinterpret_cast<VP *>(wave_lds);
    unsigned roff = static_cast<unsigned>(2 + SB * sb0) * row_bytes + lane * (ROWS / 16) * sizeof(R);
    auto fetch_chunk = [&]() {
      const VP v = M4::template loadv<VP>(rows_rsrc, roff);
      roff += ROWS * row_bytes;
      return v;
    };
    {
      const VP c0 = fetch_chunk(), c1 = fetch_chunk();
      rows_put[lane] = c0;
      rows_put[64 + lane] = c1;
    }
    VP chunk_next = fetch_chunk();
    int put = lane;  // where it goes
    // This lane's next history load: ti = tiles back from the one of step t0-2, x its tile in the
    // ring, off its offset.  Every load is issued unconditionally, also past the
    // range (those values are never used), so that the loop below has no branch
    // around a load and each product waits only for its own loads, not for the
    // ones in flight behind them.
    int ti = 4 * (sb0 - HOLD) + k_ - SH * h0;
    int x = (mod_step(t0 - 2 + cap + ring_shift<R>(b), cap) / TS - ti) % ntile;
    if (x < 0) x += ntile;
    unsigned off = static_cast<unsigned>(x) * tile_bytes +
                   static_cast<unsigned>(p * 3 * kLanes * 2 + (CM * j + mq) * 2 + reim) * 16u;
    const unsigned wrap = static_cast<unsigned>(ntile - 4) * tile_bytes;
    typedef R VT __attribute__((ext_vector_type(RingTile<R>::TS)));
    VT bq[NB][3];
    auto load_history = [&](VT(&dst)[3]) {
      const unsigned o = ti < 0 ? kBufferNone - 2 * comp_bytes : off;
#pragma unroll
      for (int c = 0; c < 3; ++c) dst[c] = M4::load16(ring_rsrc, o + c * comp_bytes);
      ti += 4;  // the next superblock's tile is 4 tiles older
      x -= 4;
      off = x < 0 ? off + wrap : off - 4u * tile_bytes;
      x = x < 0 ? x + ntile : x;
    };
    static_for<HOLD + AH>([&](auto q) { load_history(bq[decltype(q)::value]); });
    int lrow = TS * k_ + s_ + (TS - 1);  // row of product 0 of the round's first superblock
    wave_lds_order();
    V aq[2];
    aq[0] = rows_lds[lrow & (2 * ROWS - 1)];
    // One superblock; qc = its number within the round (a compile-time index):
    // group g takes the history of the superblock TG 16 / SB g before.
    auto superblock = [&](auto qc) {
      constexpr int q = decltype(qc)::value;
      static_for<TS>([&](auto ec) {
        constexpr int e = decltype(ec)::value;
        constexpr int i = q * TS + e;
        const V rw = aq[i % 2];
        // the next product's rows
        constexpr int next = e + 1 < TS ? SB * q - (e + 1) : SB * (q + 1);
        aq[(i + 1) % 2] = rows_lds[(lrow + next) & (2 * ROWS - 1)];
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const VT(&u)[3] = bq[(q + HOLD - TG * 16 / SB * g + 4 * NB) % NB];
          C[g][0] = M4::mul(rw[0], u[0][e], C[g][0]);
          C[g][1] = M4::mul(rw[1], u[1][e], C[g][1]);
          C[g][2] = M4::mul(rw[2], u[1][e], C[g][2]);
          C[g][3] = M4::mul(rw[1], u[0][e], C[g][3]);
          C[g][4] = M4::mul(rw[3], u[2][e], C[g][4]);
        }
      });
      // the set past the ones held takes the superblock AH ahead
      load_history(bq[(q + HOLD + AH) % NB]);
      // keep the scheduler from sinking these loads towards their use
      __builtin_amdgcn_sched_barrier(0);
    };
    for (int sb = sb0; sb < sb1; sb += NR) {
      static_for<NR>(superblock);
      // the next round's second chunk of rows; the one after it is in flight
      wave_lds_order();
      rows_put[put] = chunk_next;
      wave_lds_order();
      put ^= 64;
      chunk_next = fetch_chunk();
      lrow += ROWS;
      if constexpr (COMP) {
        // fold the plain float32 sums of the round's lags
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int t = 0; t < 5; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              acc[g][t][v] += static_cast<Sum>(C[g][t][v]);
              C[g][t][v] = R(0);
            }
      }
    }
  }
  if constexpr (!COMP) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int t = 0; t < 5; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[g][t][v] = C[g][t][v];
  }
  // lag ranges of the other wavefronts, added in chunk order by wavefront 0
  if (LG > 1) {
    if (chunk > 0) {
      Sum *dst = reinterpret_cast<Sum *>(wave_lds) + lane;
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int t = 0; t < 5; ++t)
#pragma unroll
          for (int v = 0; v < 4; ++v) dst[((g * 5 + t) * 4 + v) * kLanes] = acc[g][t][v];
    }
    __syncthreads();
    if (chunk == 0) {
      for (int c = 1; c < LG; ++c) {
        const Sum *src = reinterpret_cast<const Sum *>(wave_lds + c * Shape::kWaveLds) + lane;
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int t = 0; t < 5; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[g][t][v] += src[((g * 5 + t) * 4 + v) * kLanes];
      }
    }
  }
  if (chunk != 0 || !active) return;
  R *__restrict__ pending = static_cast<R *>(a.pending);
  const long long col_off = 2 * (static_cast<long long>(p) * 5 * M + sq + mq) + reim;
  const int slot0 = static_cast<int>(t0 % (D + 1));
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      int slot = slot0 + 16 * (h0 + TG * g) + M4::row(lane, v);
      if (slot > D) slot -= D + 1;
      R *dst = pending + slot * (NP * 10LL * M) + col_off;
#pragma unroll
      for (int t = 0; t < 5; ++t) dst[2 * t * M] = static_cast<R>(acc[g][t][v]);
    }
}

// ------------------------------------------------------------- middle level

// Between two sweeps of a block (D steps apart on the matrix cores) the newest
// lags grow to D + 1, which every mode would read again each step.  A middle
// level bounds them by kMidPeriod + 1: the launch of step n also takes the blocks
// with t0 = n+1 = b mod kMidPeriod whose sweep is d = (t0 - b) mod D > 0 steps
// back, and forms for the next kMidPeriod steps the sum over the d entries since
// that sweep (lags 2 .. d+1 of t0),
//   mid[(t0+u) mod (kMidPeriod+1)] = sum_{i=2}^{d+1} w_{i+u} (x) U^{t0-i}.
// Like the sweep it reads neither U^n nor the sums of step n.
//
// Work item (one wavefront) = (block, plane, MQ of its modes); the lanes are MQ
// modes x MT groups of MS steps x ML ranges of the entries, so a lane holds 10 MS
// sums (bounded by the registers the launch's sweep leaves) and the chain of
// dependent loads is short; the ranges are summed by a lane butterfly.
template <typename R> struct MidShape {
  static constexpr int MS = sizeof(R) == 8 ? 2 : 4;
  static constexpr int MT = kMidPeriod / MS;
  static constexpr int ML = sizeof(R) == 8 ? 2 : 4;
  static constexpr int MQ = kLanes / (MT * ML);
  static constexpr int kParts = kLanes / MQ;  // items per block and plane
};

template <typename R, int D>
__device__ __forceinline__ void mid_item(const SweepArgs &a, int item) {
  using W = typename W4<R>::T;
  using Shape = MidShape<R>;
  using VT = typename RingTile<R>::V;
  constexpr int TS = RingTile<R>::TS;
  constexpr int MS = Shape::MS, ML = Shape::ML, MQ = Shape::MQ;
  const int np = a.np;
  const int bi = item / (np * Shape::kParts), r = item - bi * (np * Shape::kParts);
  const int p = r / Shape::kParts, part = r - p * Shape::kParts;
  const long long t0 = a.step + 1, M = a.M;
  const int b = static_cast<int>(t0 % kMidPeriod) + kMidPeriod * bi;
  const int d = static_cast<int>((t0 - b % D + D) % D);
  if (d == 0) return;  // this launch sweeps the block
  const int lane = threadIdx.x & 63;
  const int col = part * MQ + lane % MQ;
  const int lg = lane / MQ % ML;
  const int u0 = lane / (MQ * ML) * MS;
  const long long s = static_cast<long long>(b) * kLanes + col;
  const int wl = s < M ? a.win[s] : 0;
  const int cap = a.blk_cap[b];
  // entries: lags 2 .. d+1 of t0, whole tiles from the one of step t0-2 back, as far
  // as the window goes (earlier than the first step they are zero)
  static_assert(kMidPeriod % TS == 0, "the entries are whole tiles");
  const int ntiles = wl > 2 ? min(d / TS, (wl - 2 + TS - 1) / TS) : 0;
  const int per = (ntiles + ML - 1) / ML;       // tiles per range
  const int q0 = lg * per, q1 = min(ntiles, q0 + per);
  R sums[MS][kSums];
#pragma unroll
  for (int u = 0; u < MS; ++u)
#pragma unroll
    for (int k = 0; k < kSums; ++k) sums[u][k] = R(0);
  if (wl > 0) {
    const W *__restrict__ rowp = static_cast<const W *>(a.table) + a.row0[s];
    const int ring_tiles = cap / TS;
    const VT *__restrict__ rp = ring_tile<R>(a.ring, a.blk_off[b], np, p, col);
    int x = mod_step(t0 - 2 + cap + ring_shift<R>(b), cap) / TS - q0 % ring_tiles;
    if (x < 0) x += ring_tiles;
    for (int q = q0; q < q1; ++q) {
      VT h[3][2];
      load_tile<R>(h, rp, x, np);
      // element e is lag TS (q + 1) + 1 - e
      W w[TS + MS - 1];
#pragma unroll
      for (int k = 0; k < TS + MS - 1; ++k) w[k] = rowp[min(TS * q + 2 + u0 + k, wl)];
#pragma unroll
      for (int e = 0; e < TS; ++e) {
        cplx<R> u[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) u[c] = cplx<R>{h[c][0][e], h[c][1][e]};
#pragma unroll
        for (int v = 0; v < MS; ++v) fma_lag<R>(sums[v], w[TS - 1 - e + v], u);
      }
      x = x == 0 ? ring_tiles - 1 : x - 1;
    }
  }
#pragma unroll
  for (int off = MQ; off < MQ * ML; off <<= 1)
#pragma unroll
    for (int u = 0; u < MS; ++u)
#pragma unroll
      for (int k = 0; k < kSums; ++k) sums[u][k] += __shfl_xor(sums[u][k], off);
  if (wl == 0) return;
  // each of the ML lanes of a mode stores its share of the MS steps
  cplx<R> *__restrict__ mid = static_cast<cplx<R> *>(a.mid);
#pragma unroll
  for (int u = 0; u < MS; ++u) {
    if (u % ML != lg) continue;
    const int slot = static_cast<int>((t0 + u0 + u) % (kMidPeriod + 1));
    cplx<R> *dst = mid + (slot * np + p) * 5LL * M + s;
#pragma unroll
    for (int t = 0; t < 5; ++t) dst[t * M] = cplx<R>{sums[u][2 * t], sums[u][2 * t + 1]};
  }
}

// The launch of the matrix-core form: work-groups of LG QW wavefronts, first the
// quad sweeps of this launch's phase, then the items of the middle level and the
// mode items (one per wavefront).  LDS (dynamic) holds the partial sums of
// wavefronts 1 .. LG-1 of a quad.
template <typename R, bool COMP, int NP, int CM, int G, int TW, int WAVES>
__global__ __launch_bounds__(4 * kLanes) __attribute__((amdgpu_waves_per_eu(WAVES))) void
step_kernel_mfma(SweepArgs sa, ModeArgs ma, long long sweep_wgs, long long mid_wgs, int mid_items,
                 long long nblocks, int LG, int QW, unsigned spread) {
  extern __shared__ __align__(16) unsigned char quad_lds[];
  // Groups of 8 ids (one per XCD): the sweep's are spread over the first `spread`
  // groups (see the launch).
  const unsigned g8 = blockIdx.x >> 3, ns = static_cast<unsigned>(sweep_wgs >> 3);
  long long wg;
  {
    const unsigned before = g8 < spread ? static_cast<unsigned>(static_cast<unsigned long long>(g8) * ns / spread) : ns;
    const unsigned after = g8 < spread ? static_cast<unsigned>(static_cast<unsigned long long>(g8 + 1) * ns / spread) : ns;
    if (after > before) {
      quad_sweep<R, COMP, NP, CM, G, TW>(sa, before * 8LL + (blockIdx.x & 7), LG, QW, quad_lds);
      return;
    }
    wg = (g8 - before) * 8LL + (blockIdx.x & 7);
  }
  const int waves = LG * QW;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  if (wg < mid_wgs) {
    const long long wgs = (mid_items + waves - 1) / waves;
    const long long mw = xcd_chunk(wg, wgs);
    const long long k = mw * waves + wave;
    if (mw < wgs && k < mid_items)
      mid_item<R, QuadShape<R, COMP, NP, CM, G, TW>::D>(sa, static_cast<int>(k));
    return;
  }
  wg -= mid_wgs;
  const long long mode_wgs = (nblocks * NP + waves - 1) / waves;
  const long long mw = xcd_chunk(wg, mode_wgs);
  if (mw >= mode_wgs) return;
  const long long k = mw * waves + wave;
  if (k >= nblocks * NP) return;
  const int p = static_cast<int>(k / nblocks);
  const long long s = (k - p * nblocks) * kLanes + (threadIdx.x & 63);
  if (s < ma.M) mode_step<R, COMP, true>(ma, p, s);
}

template <typename R, bool COMP, int NP, int CM, int G, int TW>
hipError_t step_launch_q(const sbim_handle *h, const Group &g, const SweepArgs &sa0,
                         const ModeArgs &ma, long long mode_blocks, hipEvent_t ev0, hipEvent_t ev1) {
  using Shape = QuadShape<R, COMP, NP, CM, G, TW>;
  constexpr int D = Shape::D;
  if (h->depth != D) return hipErrorInvalidValue;
  SweepArgs sa = sa0;
  const long long t0 = sa.step + 1;
  const int phase = static_cast<int>(t0 % D);
  sa.nphase = g.nblocks > phase ? (g.nblocks - phase + D - 1) / D : 0;
  const int LG = h->lag_chunks, QW = h->sweep_quads;
  const long long sweep_wgs = (sa.nphase + 7) / 8 * 8 * (kLanes / CM * TW / QW);
  int mid_items = 0;
  if (sa.mid) {
    const int ph = static_cast<int>(t0 % kMidPeriod);
    if (g.nblocks > ph)
      mid_items = static_cast<int>((g.nblocks - ph + kMidPeriod - 1) / kMidPeriod * NP * MidShape<R>::kParts);
  }
  const int waves = LG * QW;
  const long long mid_wgs = xcd_chunk_ids((mid_items + waves - 1) / waves);
  const long long mode_wgs = (mode_blocks * NP + waves - 1) / waves;
  const size_t lds = static_cast<size_t>(waves) * Shape::kWaveLds;
  if (sweep_wgs + mid_wgs + mode_wgs == 0) return hipSuccess;
  if (ev0) {
    const hipError_t e = hipEventRecord(ev0, h->stream);
    if (e != hipSuccess) return e;
  }
  // Wavefronts per SIMD: four (128 registers), three for float64 (its mode items
  // alone take 150).
  constexpr int WAVES = sizeof(R) == 8 ? 3 : 4;
  // The sweep's work-groups lie among the first half of the others': its matrix-core
  // work then overlaps their memory traffic (measured with four lag ranges, us per
  // step with the sweep first / spread over half / over all of them: 1024^2, W = 2000,
  // float32 633 / 582 / 600; 512^2, W = 1000, float64 214 / 211 / 221, compensated
  // 133 / 133 / 136).
  const unsigned spread =
      static_cast<unsigned>(sweep_wgs / 8 + (mid_wgs + xcd_chunk_ids(mode_wgs)) / 16);
  hipLaunchKernelGGL((step_kernel_mfma<R, COMP, NP, CM, G, TW, WAVES>),
                     dim3(static_cast<unsigned>(sweep_wgs + mid_wgs + xcd_chunk_ids(mode_wgs))),
                     dim3(waves * kLanes), lds, h->stream, sa, ma, sweep_wgs, mid_wgs, mid_items,
                     mode_blocks, LG, QW, spread);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && ev1) e = hipEventRecord(ev1, h->stream);
  return e;
}

// The matrix-core launch for this handle's planes per group, modes per quad and depth.
template <typename R, bool COMP>
hipError_t step_launch_quads(const sbim_handle *h, const Group &g, const SweepArgs &sa,
                             const ModeArgs &ma, long long mode_blocks, hipEvent_t ev0, hipEvent_t ev1) {
  if (h->lag_chunks < 1 || h->sweep_quads < 1 || h->lag_chunks * h->sweep_quads > 4)
    return hipErrorInvalidValue;
  if (g.np == 2 && h->quad_modes == 4) {
    if (h->depth == 16) return step_launch_q<R, COMP, 2, 4, 1, 1>(h, g, sa, ma, mode_blocks, ev0, ev1);
    // 32 steps: two accumulator groups per wavefront share each operand load; the
    // float64 and compensated sums (two registers each) take a wavefront per group
    // instead (measured, us per step of 512^2, W = 1000: compensated 132 against 171;
    // float64 211 against 214; float32 1024^2, W = 2000: 647 against 572)
    constexpr bool wide = COMP || sizeof(R) == 8;
    return step_launch_q<R, COMP, 2, 4, wide ? 1 : 2, wide ? 2 : 1>(h, g, sa, ma, mode_blocks, ev0, ev1);
  }
  if (g.np == 2) return step_launch_q<R, COMP, 2, 2, 1, 1>(h, g, sa, ma, mode_blocks, ev0, ev1);
  if (h->quad_modes == 4) return step_launch_q<R, COMP, 1, 4, 1, 1>(h, g, sa, ma, mode_blocks, ev0, ev1);
  return step_launch_q<R, COMP, 1, 2, 1, 1>(h, g, sa, ma, mode_blocks, ev0, ev1);
}

}  // namespace

hipError_t launch_step_quads(const sbim_handle *h, const Group &g, const SweepArgs &sa,
                             const ModeArgs &ma, long long mode_blocks, hipEvent_t ev0, hipEvent_t ev1) {
  if (h->fp64) return step_launch_quads<double, false>(h, g, sa, ma, mode_blocks, ev0, ev1);
  if (h->comp) return step_launch_quads<float, true>(h, g, sa, ma, mode_blocks, ev0, ev1);
  return step_launch_quads<float, false>(h, g, sa, ma, mode_blocks, ev0, ev1);
}

}  // namespace sbim
