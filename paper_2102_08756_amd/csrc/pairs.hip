// The step launch of float32 handles that drive a fault or a strip, two planes of one
// material, fixed windows: the history sweep on the matrix cores with the lags summed
// in order (each product of 4 consecutive lags), over the sorted classes and rings of
// the vector form.  The fault's stick/slip state follows the rounding of these sums
// step by step, so their order is kept; quads.hip's form, faster and equally
// accurate, rounds differently.
#include "step_items.h"

namespace sbim {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

// Kernel-row blocks a compensated quad sweep sums in plain float32 (the
// matrix-core accumulators) before folding them into its compensated sums:
// 8 blocks of 4 lags.
constexpr int kQuadFold = 8;
// Blocks of 4 lags whose history and kernel rows the quad sweep has in flight
// ahead of its products (measured on gfx950: 2 to 8 within 3%; 2 fits the
// compensated form's register budget best).
constexpr int kQuadAhead = 2;

// The sweep on the matrix cores, for float32 history of two planes that share
// their kernel rows (one material group, one window for every mode).  Its
// sums are the same as sweep_item's: the launch of step n serves steps
// t0 = n+1 .. n+D (D = 16 G) from the history up to step n-1,
//   pending[(t0+u) mod (D+1)] = sum_{i>=2} w_{i+u} (x) U^{t0-i},
// but per class of modes the product over lags is a Toeplitz matrix times a
// matrix of history columns:
//   out[u][col] = sum_i w[i + u] U^{t0-i}[col],
// done as 16x16x4 float32 products (one per 4 lags and 16 steps), each the
// sequence of four fused multiply-adds of a lane's FMA chain in lag order.
//
// Classes are padded to multiples of 4 sorted positions, so the four lanes
// 4j .. 4j+3 of a block ("quad" j) share one kernel row.  The 16 columns are
// (plane p, mode mq of the quad, real/imaginary part): col = 8 p + 2 mq + reim.
// Per 4 lags i0 .. i0+3 and 16-step group g the operands are
//   A[s][k] = w_type[i0 + k + s + 16 g]   (lane s + 16 k; rows past the class's
//                                          window clamp to its zero row),
//   B[k][col] = U^{t0-i0-k}[col]          (lane col + 16 k, one float of the ring),
// and the five products per group are (w11, U_L), (w12, U_N), (w22, U_N),
// (w12, U_L), (w33, U_T) -> sums 2 tau + reim, tau = 0..4, as fma_lag orders
// them.  Output lane l, register v of group g: step u = 16 g + 4 (l/16) + v,
// column l mod 16.
//
// Work-group = one quad of a block of this launch's phase; its LG wavefronts
// take consecutive ranges of the 4-lag blocks and are summed in LDS in a fixed
// order (the compensated sums with Neumaier's rule), so results are bitwise
// reproducible.  Work-group ids of one block are congruent mod 8, so the 16
// quads of a block, which share the history's cache lines, run on one XCD.
// Lags past min(cap-1, t0) meet zero rows or never-written (zero) ring slots,
// as in sweep_item.
// One component of the next block's Toeplitz operand of a 16-step group: lane
// (s, k) = s + 16 k takes lane s + 4 of `cur` for s < 12 and lane s - 12 of
// `above` (the group 16 steps later) for s >= 12 (DPP row shifts within rows of
// 16 lanes).
__device__ __forceinline__ float shift_row4(float cur, float above) {
  const int t = __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, 0.f),
                                            __builtin_bit_cast(int, above), 0x11C /* row_shr:12 */,
                                            0xF, 0xF, false);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(t, __builtin_bit_cast(int, cur),
                                                               0x104 /* row_shl:4 */, 0xF, 0xF,
                                                               false));
}
__device__ __forceinline__ float4 shift_rows4(float4 cur, float4 above) {
  return float4{shift_row4(cur.x, above.x), shift_row4(cur.y, above.y),
                shift_row4(cur.z, above.z), shift_row4(cur.w, above.w)};
}

template <bool COMP, int G>
__device__ __forceinline__ void pair_sweep(const SweepArgs &a, long long wg, int LG, int QW,
                                           float *__restrict__ lds) {
  constexpr int D = 16 * G;
  // Wavefront w of the work-group: quad qi = w / LG of the work-group's QW
  // quads, lag range chunk = w mod LG (uniform: kept in scalar registers, so
  // the loop control below is scalar).
  const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int chunk = w % LG, qi = w / LG;
  const int per_block = 16 / QW;  // work-groups per block
  const long long kb = (wg / (8 * per_block)) * 8 + (wg & 7);
  if (kb >= a.nphase) return;     // uniform over the work-group
  const int j = static_cast<int>((wg >> 3) % per_block) * QW + qi;  // quad of the block
  const long long M = a.M, step = a.step;
  const long long t0 = step + 1;
  const long long b = t0 % D + D * kb;
  const int lane = threadIdx.x & 63;
  const int s_ = lane & 15;                 // A row (step in group) / B column
  const int k_ = lane >> 4;                 // lag within a 4-lag block
  const int p = s_ >> 3, mq = (s_ >> 1) & 3, reim = s_ & 1;
  const long long sq = b * kLanes + 4 * j;  // first sorted position of the quad
  // Past the last mode (M is a multiple of 4) a quad has no work; it still takes
  // part in the work-group's barrier below (uniform over the wavefront).
  const bool active = sq < M;
  const int cap = __builtin_amdgcn_readfirstlane(a.blk_cap[b]);
  // the class's window (its first position is a mode)
  const int wl = active ? __builtin_amdgcn_readfirstlane(a.win[sq]) : 0;
  const int nent = wl > 0 ? static_cast<int>(max(0LL, min(static_cast<long long>(cap) - 1, t0) - 1)) : 0;
  const int nblk = (nent + 3) / 4;
  const int per = (nblk + LG - 1) / LG;
  const int beta0 = min(nblk, chunk * per);
  const int beta1 = min(nblk, beta0 + per);

  v4f C[G][5];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int t = 0; t < 5; ++t) C[g][t] = v4f{0.f, 0.f, 0.f, 0.f};
  Acc<float, COMP> acc[G][5][4];
  if (beta1 > beta0) {
    // The quad's operands come through buffer loads: a resource per work-group
    // (the block's slot 0 of the ring, the class's first kernel row) and a
    // 32-bit byte offset per lane; a load past the resource's range returns 0.
    // (Buffer loads also keep the compiler from moving a prefetch down to its
    // use, which it does with plain loads.)
    // (every value a resource is built from is read as uniform, so that the
    // resources live in scalar registers)
    const float4 *rowp = static_cast<const float4 *>(a.table) + uniform64(a.row0[sq]);
    const __amdgpu_buffer_rsrc_t rows_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float4 *>(rowp), 0, (wl + 1) * 16, kBufferWord3);
    // History: slot x of the block at x * dstep floats (the host keeps the
    // block's capacity times dstep below 2^30 floats, so byte offsets fit 32 bits).
    const float *run =
        static_cast<const float *>(a.ring) + uniform64(a.blk_off[b]) * (2LL * 3 * kLanes * 2);
    const int dstep = __builtin_amdgcn_readfirstlane(a.blk_stride[b]) * (2 * 3 * kLanes * 2);
    // (byte counts and offsets in unsigned 32-bit arithmetic: they reach 2^32 - 1)
    const unsigned udstep = static_cast<unsigned>(dstep);
    const __amdgpu_buffer_rsrc_t ring_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(run), 0,
        static_cast<int>((static_cast<unsigned>(cap - 1) * udstep + 2u * 3u * kLanes * 2u) * 4u),
        kBufferWord3);
    const int col = ((p * 3) * kLanes + 4 * j + mq) * 2 + reim;
    // (the builtins return the loaded bits as integers)
    auto hist = [&](int x, int c) {
      return __builtin_bit_cast(
          float, __builtin_amdgcn_raw_buffer_load_b32(
                     ring_rsrc,
                     static_cast<int>((static_cast<unsigned>(x) * udstep +
                                       static_cast<unsigned>(col + c * kLanes * 2)) * 4u),
                     0, 0));
    };
    auto row = [&](int r) {
      const v4f v = __builtin_bit_cast(
          v4f, __builtin_amdgcn_raw_buffer_load_b128(rows_rsrc, min(r, wl) * 16, 0, 0));
      return float4{v[0], v[1], v[2], v[3]};
    };
    // The history loads run kQuadAhead blocks ahead of the products (they come
    // from memory); xl is the ring slot of this lane's lag in the next block to load.
    // Every load is issued unconditionally, also for blocks past the range (their
    // values are never used), so that the loop below has no branch around a load
    // and each product waits only for the loads of its own block, not for the
    // ones in flight behind them.  Those loads stay in range: the slot index is
    // clamped at 0 (it only goes negative when cap < 4, and then the range has a
    // single block) and the rows clamp to the class's zero row.
    int xl = static_cast<int>((((t0 - (2 + 4 * beta0) - k_) % cap) + cap) % cap);
    float bq[kQuadAhead][3];
#pragma unroll
    for (int q = 0; q < kQuadAhead; ++q) {
#pragma unroll
      for (int c = 0; c < 3; ++c) bq[q][c] = hist(max(xl, 0), c);
      // the next block's slot is 4 lags older
      xl -= 4;
      if (xl < 0) xl += cap;
    }
    // Kernel-row operands: the top 16-step group's rows are loaded (as far ahead
    // as the history, since the rows' leading edge comes from memory); the
    // lower group's operand follows by a row shift of 4 lanes: lane (s, k) of
    // the next block takes lane (s + 4, k) of its own group, or lane (s - 12, k)
    // of the group above for s >= 12.
    const int r0 = k_ + s_;
    float4 fq[kQuadAhead];
#pragma unroll
    for (int q = 0; q < kQuadAhead; ++q) fq[q] = row(2 + 4 * (beta0 + q) + r0 + 16 * (G - 1));
    float4 a0 = G == 2 ? row(2 + 4 * beta0 + r0) : float4{0.f, 0.f, 0.f, 0.f};
    int fold = 0;
    // One 4-lag block from register set Q (a compile-time index).
    auto block = [&](auto qc, int beta) {
      constexpr int q = decltype(qc)::value;
      const float4 top = fq[q];
      float4 rw[G];
      if constexpr (G == 2) {
        rw[0] = a0;
        rw[1] = top;
      } else {
        rw[0] = top;
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        C[g][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(rw[g].x, bq[q][0], C[g][0], 0, 0, 0);
        C[g][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(rw[g].y, bq[q][1], C[g][1], 0, 0, 0);
        C[g][2] = __builtin_amdgcn_mfma_f32_16x16x4f32(rw[g].z, bq[q][1], C[g][2], 0, 0, 0);
        C[g][3] = __builtin_amdgcn_mfma_f32_16x16x4f32(rw[g].y, bq[q][0], C[g][3], 0, 0, 0);
        C[g][4] = __builtin_amdgcn_mfma_f32_16x16x4f32(rw[g].w, bq[q][2], C[g][4], 0, 0, 0);
      }
      if constexpr (G == 2) a0 = shift_rows4(a0, top);
      // this register set now takes block beta + kQuadAhead (loaded also past the
      // range, see above)
#pragma unroll
      for (int c = 0; c < 3; ++c) bq[q][c] = hist(max(xl, 0), c);
      fq[q] = row(2 + 4 * (beta + kQuadAhead) + r0 + 16 * (G - 1));
      // keep the scheduler from sinking these loads towards their use
      __builtin_amdgcn_sched_barrier(0);
      xl -= 4;
      if (xl < 0) xl += cap;
      if constexpr (COMP) {
        // fold the plain partial sums of the last kQuadFold blocks (uniform branch)
        if (++fold == kQuadFold) {
          fold = 0;
#pragma unroll
          for (int g = 0; g < G; ++g)
#pragma unroll
            for (int t = 0; t < 5; ++t)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                acc[g][t][v].fold(C[g][t][v]);
                C[g][t][v] = 0.f;
              }
        }
      }
    };
    // Whole rounds of kQuadAhead blocks with no branch between the loads of one
    // block and the products of the next (so the compiler's waits are exact:
    // the products of a block wait for its own loads only), then the rest.
    int base = beta0;
    for (; base + kQuadAhead <= beta1; base += kQuadAhead)
      static_for<kQuadAhead>([&](auto qc) { block(qc, base + decltype(qc)::value); });
    static_for<kQuadAhead - 1>([&](auto qc) {
      if (base + decltype(qc)::value < beta1) block(qc, base + decltype(qc)::value);
    });
  }
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int t = 0; t < 5; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[g][t][v].fold(C[g][t][v]);
  // lag ranges of the other wavefronts, added in chunk order by wavefront 0
  if (LG > 1) {
    constexpr int NV = G * 5 * 4;
    constexpr int PER = COMP ? 2 : 1;
    lds += static_cast<long long>(qi) * (LG - 1) * NV * PER * kLanes;  // this quad's partial sums
    if (chunk > 0) {
      float *dst = lds + static_cast<long long>(chunk - 1) * NV * PER * kLanes + lane;
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int t = 0; t < 5; ++t)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int idx = (g * 5 + t) * 4 + v;
            dst[(idx * PER) * kLanes] = acc[g][t][v].s;
            if constexpr (COMP) dst[(idx * PER + 1) * kLanes] = acc[g][t][v].c;
          }
    }
    __syncthreads();
    if (chunk == 0) {
      for (int w = 1; w < LG; ++w) {
        const float *src = lds + static_cast<long long>(w - 1) * NV * PER * kLanes + lane;
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int t = 0; t < 5; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int idx = (g * 5 + t) * 4 + v;
              if constexpr (COMP) {
                neumaier(acc[g][t][v].s, acc[g][t][v].c, src[(idx * PER) * kLanes]);
                acc[g][t][v].c += src[(idx * PER + 1) * kLanes];
              } else {
                acc[g][t][v].s += src[(idx * PER) * kLanes];
              }
            }
      }
    }
  }
  if (chunk != 0 || !active) return;
  float *__restrict__ pending = static_cast<float *>(a.pending);
  const long long col_off = 2 * (static_cast<long long>(p) * 5 * M + sq + mq) + reim;
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const long long slot = (t0 + 16 * g + 4 * k_ + v) % (D + 1);
      float *dst = pending + slot * 2 * kSums * M + col_off;
#pragma unroll
      for (int t = 0; t < 5; ++t) dst[2 * t * M] = acc[g][t][v].value();
    }
}

// The launch of the matrix-core form: work-groups of LG wavefronts, first the
// quad sweeps of this launch's phase, then the mode items (LG (block, plane)
// items per work-group, one per wavefront).  LDS (dynamic) holds the partial
// sums of wavefronts 1 .. LG-1 of a quad.
template <bool COMP, int G, int WAVES>
__global__ __launch_bounds__(4 * kLanes) __attribute__((amdgpu_waves_per_eu(WAVES))) void
step_kernel_pairs(SweepArgs sa, ModeArgs ma, long long sweep_wgs, long long nblocks, int LG, int QW) {
  extern __shared__ float quad_lds[];
  const long long wg = blockIdx.x;
  if (wg < sweep_wgs) {
    pair_sweep<COMP, G>(sa, wg, LG, QW, quad_lds);
    return;
  }
  const long long mode_wgs = (nblocks * ma.np + LG * QW - 1) / (LG * QW);
  const long long mw = xcd_chunk(wg - sweep_wgs, mode_wgs);
  if (mw >= mode_wgs) return;
  const long long k = mw * (LG * QW) + (threadIdx.x >> 6);
  if (k >= nblocks * ma.np) return;
  const int p = static_cast<int>(k / nblocks);
  const long long s = (k - p * nblocks) * kLanes + (threadIdx.x & 63);
  if (s < ma.M) mode_step<float, COMP, false>(ma, p, s);
}

template <bool COMP, int G>
hipError_t step_launch_p(const sbim_handle *h, const Group &g, const SweepArgs &sa0,
                         const ModeArgs &ma, long long mode_blocks, hipEvent_t ev0, hipEvent_t ev1) {
  constexpr int D = 16 * G;
  SweepArgs sa = sa0;
  const int phase = static_cast<int>((sa.step + 1) % D);
  sa.nphase = g.nblocks > phase ? (g.nblocks - phase + D - 1) / D : 0;
  const int LG = h->lag_chunks, QW = h->sweep_quads;
  const long long sweep_wgs = (sa.nphase + 7) / 8 * 8 * (16 / QW);
  const long long mode_wgs = (mode_blocks * g.np + LG * QW - 1) / (LG * QW);
  if (sweep_wgs + mode_wgs == 0) return hipSuccess;
  const size_t lds = static_cast<size_t>(QW) * (LG - 1) * G * 5 * 4 * (COMP ? 2 : 1) * kLanes *
                     sizeof(float);
  if (ev0) {
    const hipError_t e = hipEventRecord(ev0, h->stream);
    if (e != hipSuccess) return e;
  }
  // Register budget: three wavefronts per SIMD (168 registers; the compensated
  // two-group form takes 165).  At two wavefronts per SIMD the 2080 sweep
  // wavefronts of a 512^2 phase (1040 quads, two lag ranges each) do not all
  // fit at once, and the rest take a second round (measured on gfx950 with one
  // quad per work-group: 4-8% slower).
  constexpr int WAVES = 3;
  hipLaunchKernelGGL((step_kernel_pairs<COMP, G, WAVES>),
                     dim3(static_cast<unsigned>(sweep_wgs + xcd_chunk_ids(mode_wgs))),
                     dim3(LG * QW * kLanes), lds, h->stream, sa, ma, sweep_wgs, mode_blocks, LG, QW);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && ev1) e = hipEventRecord(ev1, h->stream);
  return e;
}

}  // namespace

hipError_t launch_step_pairs(const sbim_handle *h, const Group &g, const SweepArgs &sa,
                             const ModeArgs &ma, long long mode_blocks, hipEvent_t ev0, hipEvent_t ev1) {
  if (g.np != 2 || h->fp64 || (h->depth != 16 && h->depth != 32) || h->lag_chunks < 1 ||
      h->lag_chunks * h->sweep_quads > 4)
    return hipErrorInvalidValue;
  if (h->comp)
    return h->depth == 32 ? step_launch_p<true, 2>(h, g, sa, ma, mode_blocks, ev0, ev1)
                          : step_launch_p<true, 1>(h, g, sa, ma, mode_blocks, ev0, ev1);
  return h->depth == 32 ? step_launch_p<false, 2>(h, g, sa, ma, mode_blocks, ev0, ev1)
                        : step_launch_p<false, 1>(h, g, sa, ma, mode_blocks, ev0, ev1);
}

}  // namespace sbim
