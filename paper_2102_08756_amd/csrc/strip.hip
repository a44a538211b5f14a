// Finite-element strip of the hybrid scheme: 8-node hexahedra on a regular grid
// between the fault (node layer 0) and the boundary S+ (node layer N2), periodic
// in x1 and x3 with the boundary-integral grid; explicit central differences in
// the predictor-corrector form of Sec. 2.2 (Eqs. fepred, feintdisp, tintf,
// fecorr); the traction of the half-space above S+ from the boundary relation
// (Eq. SBI, Sec. 2.4 items 2-4); the fault either as a symmetry plane or, in
// the two-sided strip, as split nodes between two element blocks, with the
// stick traction of the forward Lagrange multiplier (Eqs. freeslip,
// sticktraction) limited by the slip-weakening strength (Eqs. stickslip,
// slipweak).
//
// Fields are float64 [component][node layer][x1][x3] (x3 fastest); one thread
// per node in the predictor, per column of a few node layers in the corrector, per
// fault cell for the split nodes.  The stiffness is applied node by node as a
// 27-point stencil of 3x3 blocks, one stencil per node layer (the element layers
// above and below it may differ), precomputed on the host from the element stiffness.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.h"

// Plain float64 rounding of each product and sum, as in the interface solve of
// the fault kernel: the stick/slip choice compares two such results.  The
// stencil sums alone are contracted into fused multiply-adds.
#pragma clang fp contract(off)

namespace sbim {
namespace {

// Pointers of known kind: device memory, and tables read through the scalar cache.
using global_f64 = const __attribute__((address_space(1))) double *;
using table_f64 = const __attribute__((address_space(4))) double *;
using table_i32 = const __attribute__((address_space(4))) int *;

constexpr int kStripThreads = 128;  // (1024^2, us a pass: 128 771, 256 781, 512 828)

// The predictor of the next step from a node's new acceleration and velocity
// (Eq. fepred and the displacement update), with the push inputs of S+ (plane
// 0) or S- (plane 1) when the node lies on one of them.
template <typename R>
__device__ __forceinline__ void strip_predict(const StripArgs &a, long long base, int push_plane,
                                              unsigned cell, int c, double u, double vn, double acc) {
  const double dt = a.dt;
  const double vh = vn + 0.5 * dt * acc;        // v_{t+3/2}
  const double un = u + dt * vh;                // u_{t+2}
  (a.v + base)[cell] = vn;
  (a.vh + base)[cell] = vh;
  (a.u_next + base)[cell] = un;
  if (push_plane >= 0) {
    R *__restrict__ pu = static_cast<R *>(a.push_u);
    R *__restrict__ pv = static_cast<R *>(a.push_v);
    const long long t = (push_plane * 3 + c) * a.cells;
    (pu + t)[cell] = static_cast<R>(a.increment ? dt * vh : un);
    (pv + t)[cell] = static_cast<R>(vn + dt * acc);  // predicted velocity of Eq. fepred
  }
}

// Everything after the stiffness forces for one node (cell: its place in the layer; u: its u_{t+1}, vh: its
// v_{t+1/2}): the S+ (S-) traction,
// the fault solve on layer 0 of the one-sided strip, the corrector and the
// fault outputs, then the predictor of the next step.
template <typename R>
__device__ __forceinline__ void strip_finish(const StripArgs &a, int layer, unsigned cell,
                                             double r[3], const double u[3],
                                             const double vh[3]) {
  const long long nodes = a.nodes, cells = a.cells;
  const double A = a.area;
  const R *__restrict__ ts = static_cast<const R *>(a.tau_sbi);
  if (layer == a.n2) {                           // S+: traction of the half-space above
#pragma unroll
    for (int p = 0; p < 3; ++p) r[p] += A * static_cast<double>((ts + p * cells)[cell]);
  }
  const bool two = a.fault_lo >= 0;
  if (two && layer == 0) {                       // S-: outward normal -e2
#pragma unroll
    for (int p = 0; p < 3; ++p) r[p] -= A * static_cast<double>((ts + (3 + p) * cells)[cell]);
  }
  if (two && (layer == a.fault_lo || layer == a.fault_lo + 1)) {
    // split fault nodes: the two copies are solved together by strip_fault2
    const int side = layer == a.fault_lo ? 1 : 0;
#pragma unroll
    for (int p = 0; p < 3; ++p) (a.r_fault + (side * 3 + p) * cells)[cell] = r[p];
    return;
  }
  const double M = a.mass[layer];
  const double dt = a.dt;
  if (!two && layer == 0) {                      // fault node: stick traction and strength
    const double t00 = a.tau0[cell], t01 = (a.tau0 + cells)[cell], t02 = (a.tau0 + 2 * cells)[cell];
    const double vs0 = vh[0] + dt * r[0] / M;
    const double vs2 = vh[2] + dt * r[2] / M;
    const double st0 = t00 + M * vs0 / (dt * A);
    const double st2 = t02 + M * vs2 / (dt * A);
    const double mag = sqrt(st0 * st0 + st2 * st2);
    const double s0 = 2.0 * u[0], s2 = 2.0 * u[2];
    const double delta = sqrt(s0 * s0 + s2 * s2);
    const double mus = a.mu_s[cell], muk = a.mu_k[cell], dc = a.d_c[cell];
    const double mu = delta < dc ? mus - (mus - muk) * delta / dc : muk;
    const double strength = fmax(-t01, 0.0) * mu;
    double tau0 = st0, tau2 = st2;
    const bool sliding = mag > strength;
    if (sliding) {
      const double sc = strength / mag;
      tau0 = st0 * sc;
      tau2 = st2 * sc;
    }
    r[0] -= A * (tau0 - t00);
    r[2] -= A * (tau2 - t02);
    a.tau[cell] = tau0;
    (a.tau + cells)[cell] = t01;
    (a.tau + 2 * cells)[cell] = tau2;
    a.slip[cell] = s0;
    (a.slip + cells)[cell] = s2;
    a.sliding[cell] = sliding ? 1.0 : 0.0;
    if (a.tau_out) {
      a.tau_out[cell] = tau0;
      (a.tau_out + cells)[cell] = t01;
      (a.tau_out + 2 * cells)[cell] = tau2;
    }
  }
  const int push_plane = layer == a.n2 ? 0 : (two && layer == 0 ? 1 : -1);
  double vn[3];
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const double acc = r[p] / M;
    vn[p] = vh[p] + 0.5 * dt * acc;              // v_{t+1} (Eqs. tintf, fecorr)
    strip_predict<R>(a, p * nodes + layer * cells, push_plane, cell, p, u[p], vn[p], acc);
  }
  if (!two && layer == 0) {
    a.rate[cell] = 2.0 * vn[0];
    (a.rate + cells)[cell] = 2.0 * vn[2];
    if (a.rate_out) {
      a.rate_out[cell] = 2.0 * vn[0];
      (a.rate_out + cells)[cell] = 2.0 * vn[2];
    }
  }
}

// The value of the lane before / after in the wavefront (`edge` at its ends).
__device__ __forceinline__ double lane_shift(double v, double edge, bool left) {
  const unsigned long long a = __builtin_bit_cast(unsigned long long, v);
  const unsigned long long e = __builtin_bit_cast(unsigned long long, edge);
  unsigned lo, hi;
  if (left) {  // wave_shr:1
    lo = __builtin_amdgcn_update_dpp(static_cast<int>(e), static_cast<int>(a), 0x138, 0xF, 0xF, false);
    hi = __builtin_amdgcn_update_dpp(static_cast<int>(e >> 32), static_cast<int>(a >> 32), 0x138, 0xF, 0xF, false);
  } else {     // wave_shl:1
    lo = __builtin_amdgcn_update_dpp(static_cast<int>(e), static_cast<int>(a), 0x130, 0xF, 0xF, false);
    hi = __builtin_amdgcn_update_dpp(static_cast<int>(e >> 32), static_cast<int>(a >> 32), 0x130, 0xF, 0xF, false);
  }
  return __builtin_bit_cast(double, static_cast<unsigned long long>(hi) << 32 | lo);
}

// One thread per (x1, x3) column of `depth` consecutive node layers.  It walks through
// the node layers l0-1 .. l0+depth: a layer's displacement on the rows x1-1, x1, x1+1
// comes from memory, its x3 neighbours from the lanes beside (lanes at the ends of a
// wavefront or of the periodic grid load that neighbour's column themselves), and it is
// added to the forces on the target layers l-1, l, l+1; the force on a layer is complete
// one layer later, when its corrector and predictor follow.  Each force sums its terms
// in the order offset in x2, x1, x3, component, whatever the depth.
// UNIFORM: every wavefront lies in one run of layers, so the stencil comes through the
// scalar cache (table_f64: after the loop's stores the compiler would read it through
// vector memory otherwise).  A stencil is 1.9 KB of that cache's 16, which two CUs share and
// wavefronts of different layers fill together: with one for every layer it no longer held
// them from ten layers up, so layers of equal stencils share one (512^2, two sides of 4 / 6
// element layers, a pass of three steps: 706 / 865 us with a stencil per layer, 681 / 786
// with three a side; float32 with 57 lags 758 / 903 and 723 / 835).  Three wavefronts a SIMD hide the rows' latency; a prefetch
// of the next layer costs the occupancy and more than it hides.
// Bound by the small grid's latency and by memory on large ones: 48 B read and 72 B
// written per node.  256^2 cells, two sides of 3 element layers: 49 us with one thread per
// 4 x 3 nodes (x1, layers) and no lane exchange, 20.5 here; 1024^2, 2 element layers: 161
// and 142 us (0.6 GB with the fault's and S+'s fields).
template <typename R, bool UNIFORM>
__global__ __launch_bounds__(kStripThreads) __attribute__((amdgpu_waves_per_eu(3))) void
strip_correct_kernel(StripArgs a, int depth) {
  const long long nodes = a.nodes, cells = a.cells;
  const int n1 = a.n1, n3 = a.n3, n2 = a.n2;
  // Work-groups go round-robin over the 8 XCDs; each XCD takes a contiguous eighth of
  // them, so that a row's neighbours meet in its L2.
  const long long wgs = (gridDim.x + 7LL) / 8;
  const long long tid = ((blockIdx.x & 7) * wgs + (blockIdx.x >> 3)) * kStripThreads + threadIdx.x;
  const int nruns = (n2 + depth) / depth;
  if (tid >= cells * nruns) return;  // (a whole number of rows: a lane's neighbours in its row are active)
  const int run = UNIFORM ? __builtin_amdgcn_readfirstlane(static_cast<int>(tid / cells))
                          : static_cast<int>(tid / cells);
  const int l0 = run * depth, l1 = min(l0 + depth, n2 + 1);  // target layers [l0, l1)
  const unsigned cell = static_cast<unsigned>(tid - run * cells);
  const int i1 = static_cast<int>(cell / n3), i3 = static_cast<int>(cell - static_cast<unsigned>(i1) * n3);
  const int lane = threadIdx.x & 63;
  const bool left_edge = lane == 0 || i3 == 0, right_edge = lane == 63 || i3 == n3 - 1;
  // (never both: n3 >= 4 divides or is a multiple of 64)
  const unsigned ecol = static_cast<unsigned>(left_edge ? (i3 == 0 ? n3 - 1 : i3 - 1)
                                                        : (i3 == n3 - 1 ? 0 : i3 + 1));
  const unsigned row[3] = {static_cast<unsigned>(i1 == 0 ? n1 - 1 : i1 - 1) * n3,
                           static_cast<unsigned>(i1) * n3,
                           static_cast<unsigned>(i1 == n1 - 1 ? 0 : i1 + 1) * n3};
  double C[3][3], E[3][3];  // this column and the edge lanes' neighbour: [component][row]
  auto load = [&](int l) {
    const bool edge = left_edge || right_edge;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      global_f64 ul = (global_f64)(a.u + c * nodes + static_cast<long long>(l) * cells);
      // (opaque: one base per component and 32-bit offsets, not a pointer per load
      // kept through the loop)
      if constexpr (UNIFORM)
        asm volatile("" : "+s"(ul));
      else
        asm volatile("" : "+v"(ul));
#pragma unroll
      for (int q = 0; q < 3; ++q) C[c][q] = ul[row[q] + static_cast<unsigned>(i3)];
      if (edge) {
#pragma unroll
        for (int q = 0; q < 3; ++q) E[c][q] = ul[row[q] + ecol];
      }
    }
  };
#pragma unroll
  for (int c = 0; c < 3; ++c) E[c][0] = E[c][1] = E[c][2] = 0.0;
  // forces on the layers before, at and after the source layer
  double f[3][3] = {};
  double um[3] = {};   // u of the layer before
  const int first = max(l0 - 1, 0);
#pragma unroll 1
  for (int l = first; l <= l1; ++l) {            // source layer (none above n2)
    if (l <= n2) load(l);
    double vh[3], uc[3];
    // (opaque, so that the node's addresses are formed here from scalar bases and one
    // offset, not kept as a pointer per array through the loop)
    unsigned at = cell;
    asm volatile("" : "+v"(at));
    if (l > l0) {
#pragma unroll
      for (int p = 0; p < 3; ++p) vh[p] = (a.vh + p * nodes + (l - 1LL) * cells)[at];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) uc[c] = C[c][1];
    if (l <= n2) {
#pragma clang fp contract(fast)
#pragma unroll
      for (int q = 0; q < 3; ++q) {               // row at offset q - 1 in x1
        double v[3][3];                           // [offset in x3][component]
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const double lo = lane_shift(C[c][q], E[c][q], true);
          const double hi = lane_shift(C[c][q], E[c][q], false);
          v[0][c] = left_edge ? E[c][q] : lo;
          v[1][c] = C[c][q];
          v[2][c] = right_edge ? E[c][q] : hi;
        }
#pragma unroll
        for (int t = 0; t < 3; ++t) {             // target layer l - 1 + t, which sees l at offset 1 - t
          const int lt = l - 1 + t;
          if (lt < l0 || lt >= l1) continue;
          table_f64 B = (table_f64)a.stencil + (((table_i32)a.stencil_of)[lt] * 9 + (2 - t) * 3 + q) * 27;
#pragma unroll
          for (int o3 = 0; o3 < 3; ++o3)
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
              for (int c = 0; c < 3; ++c) f[t][p] -= B[9 * o3 + 3 * p + c] * v[o3][c];
        }
        // (row by row: coefficients of all rows in flight would not fit the scalar registers)
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // layer l - 1 has all its forces
    if (l > l0) strip_finish<R>(a, l - 1, at, f[0], um, vh);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      um[c] = uc[c];
      f[0][c] = f[1][c];
      f[1][c] = f[2][c];
      f[2][c] = 0.0;
    }
  }
}

// Split fault nodes (two-sided strip), one thread per cell: the traction change
// that closes the jump of the next half-step velocities of the two copies
// (Eqs. freeslip, sticktraction), applied in full to the normal component (no
// opening) and limited on the shear pair by the slip-weakening strength at the
// current normal traction (Eqs. stickslip, slipweak); then both copies' corrector
// and the predictor of the next step.
__global__ __launch_bounds__(kStripThreads) void strip_fault2_kernel(StripArgs a) {
  const long long cell = static_cast<long long>(blockIdx.x) * kStripThreads + threadIdx.x;
  const long long cells = a.cells, nodes = a.nodes;
  if (cell >= cells) return;
  const long long im = static_cast<long long>(a.fault_lo) * cells + cell;   // lower copy
  const long long ip = im + cells;                                          // upper copy
  const double Mm = a.mass[a.fault_lo], Mp = a.mass[a.fault_lo + 1];
  const double dt = a.dt, A = a.area;
  double rp[3], rm[3], t0[3], stick[3];
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    rp[p] = a.r_fault[p * cells + cell];
    rm[p] = a.r_fault[(3 + p) * cells + cell];
    t0[p] = a.tau0[p * cells + cell];
  }
  const double zinv = dt * A * (1.0 / Mp + 1.0 / Mm);
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const double vsp = a.vh[p * nodes + ip] + dt * rp[p] / Mp;
    const double vsm = a.vh[p * nodes + im] + dt * rm[p] / Mm;
    stick[p] = t0[p] + (vsp - vsm) / zinv;
  }
  double tau[3] = {stick[0], stick[1], stick[2]};
  const double mag = sqrt(stick[0] * stick[0] + stick[2] * stick[2]);
  const double s0 = a.u[ip] - a.u[im], s2 = a.u[2 * nodes + ip] - a.u[2 * nodes + im];
  const double delta = sqrt(s0 * s0 + s2 * s2);
  const double mus = a.mu_s[cell], muk = a.mu_k[cell], dc = a.d_c[cell];
  const double mu = delta < dc ? mus - (mus - muk) * delta / dc : muk;
  const double strength = fmax(-tau[1], 0.0) * mu;
  const bool sliding = mag > strength;
  if (sliding) {
    const double sc = strength / mag;
    tau[0] = stick[0] * sc;
    tau[2] = stick[2] * sc;
  }
  double vp[3], vm[3];
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const double dtau = A * (tau[p] - t0[p]);
    const double ap = (rp[p] - dtau) / Mp;
    const double am = (rm[p] + dtau) / Mm;
    vp[p] = a.vh[p * nodes + ip] + 0.5 * dt * ap;
    vm[p] = a.vh[p * nodes + im] + 0.5 * dt * am;
    // the split copies lie on neither S+ nor S-
    strip_predict<double>(a, p * nodes + ip - cell, -1, static_cast<unsigned>(cell), p, a.u[p * nodes + ip], vp[p], ap);
    strip_predict<double>(a, p * nodes + im - cell, -1, static_cast<unsigned>(cell), p, a.u[p * nodes + im], vm[p], am);
    a.tau[p * cells + cell] = tau[p];
    if (a.tau_out) a.tau_out[p * cells + cell] = tau[p];
  }
  a.slip[cell] = s0;
  a.slip[cells + cell] = s2;
  a.sliding[cell] = sliding ? 1.0 : 0.0;
  a.rate[cell] = vp[0] - vm[0];
  a.rate[cells + cell] = vp[2] - vm[2];
  if (a.rate_out) {
    a.rate_out[cell] = vp[0] - vm[0];
    a.rate_out[cells + cell] = vp[2] - vm[2];
  }
}

// A new step size before a step (the quasi-dynamic boundary relation allows
// one): the predictor that the last step ran with its own size dt_old is redone
// with the new size dt, one thread per node, from u_{t+1}, v_{t+1} and the
// stored half-step velocity v_{t+1} + dt_old/2 a_{t+1}; the push inputs of S+
// (and S-) follow.
template <typename R>
__global__ __launch_bounds__(kStripThreads) void strip_repredict_kernel(
    double *u_pred, const double *u_prev, double *vh, const double *v, R *push_u, R *push_v,
    long long nodes, long long cells, int two_sided, int increment, double dt, double dt_old) {
  const long long id = static_cast<long long>(blockIdx.x) * kStripThreads + threadIdx.x;
  if (id >= nodes) return;
  const long long top0 = nodes - cells;
  const int plane = id >= top0 ? 0 : (two_sided && id < cells ? 1 : -1);
  const long long cell = plane == 0 ? id - top0 : id;
  const double ratio = dt / dt_old;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const long long k = c * nodes + id;
    const double vn = v[k];
    const double half = vh[k] - vn;             // dt_old/2 a_{t+1}
    const double h2 = vn + ratio * half;        // v_{t+3/2} with the new size
    const double un = u_prev[k] + dt * h2;
    vh[k] = h2;
    u_pred[k] = un;
    if (plane >= 0) {
      const long long t = (plane * 3 + c) * cells + cell;
      push_u[t] = static_cast<R>(increment ? dt * h2 : un);
      push_v[t] = static_cast<R>(vn + 2.0 * ratio * half);
    }
  }
}

}  // namespace

hipError_t launch_strip_repredict(bool fp64, double *u_pred, const double *u_prev, double *vh,
                                  const double *v, void *push_u, void *push_v, long long nodes,
                                  long long cells, bool two_sided, bool increment, double dt,
                                  double dt_old, hipStream_t st) {
  const unsigned blocks = static_cast<unsigned>((nodes + kStripThreads - 1) / kStripThreads);
  if (fp64)
    strip_repredict_kernel<double><<<blocks, kStripThreads, 0, st>>>(
        u_pred, u_prev, vh, v, static_cast<double *>(push_u), static_cast<double *>(push_v),
        nodes, cells, two_sided, increment, dt, dt_old);
  else
    strip_repredict_kernel<float><<<blocks, kStripThreads, 0, st>>>(
        u_pred, u_prev, vh, v, static_cast<float *>(push_u), static_cast<float *>(push_v),
        nodes, cells, two_sided, increment, dt, dt_old);
  return hipGetLastError();
}

hipError_t launch_strip_fault2(const StripArgs &a, hipStream_t st) {
  const unsigned blocks = static_cast<unsigned>((a.cells + kStripThreads - 1) / kStripThreads);
  strip_fault2_kernel<<<blocks, kStripThreads, 0, st>>>(a);
  return hipGetLastError();
}

template <typename R>
static hipError_t strip_correct(const StripArgs &a, int depth, hipStream_t st) {
  const long long threads = a.cells * ((a.n2 + depth) / depth);
  const unsigned blocks =
      static_cast<unsigned>((threads + 8 * kStripThreads - 1) / (8 * kStripThreads) * 8);
  if (a.cells % 64 == 0)
    strip_correct_kernel<R, true><<<blocks, kStripThreads, 0, st>>>(a, depth);
  else
    strip_correct_kernel<R, false><<<blocks, kStripThreads, 0, st>>>(a, depth);
  return hipGetLastError();
}

// Layers per thread: equal runs of layers, as few as leave four wavefronts to a SIMD (4096 in
// all) and no run longer than eight: more layers a thread read fewer rows twice, but a small
// grid waits for the chain of layers, and a last, short run still reads its two outer layers
// (us a pass of three steps at 1 / 2 / 3 / 4 / 5 / 8 layers a thread, a stencil per layer: 512^2 with 10 node layers
// 769 / 713 / 754 / 748 / 706 / 832, with 5 370 / 363 / 355 / 382 / 336 / 335; 256^2 with 10
// 255 / 264 / 250 / 265 / 273 / 324).
hipError_t launch_strip_correct(bool fp64, const StripArgs &a, hipStream_t st) {
  const int layers = a.n2 + 1;
  const long long runs = std::max((4096LL * 64 + a.cells - 1) / a.cells, (layers + 7LL) / 8);
  const int depth = static_cast<int>((layers + runs - 1) / runs);
  return fp64 ? strip_correct<double>(a, depth, st) : strip_correct<float>(a, depth, st);
}

}  // namespace sbim
