// C ABI of the boundary-integral library: configuration checks, the mode
// ordering and kernel-row classes, device memory, and the per-call launch
// sequences.  No arithmetic of the method runs here; it all runs in the HIP
// kernels of fft.hip and kernels.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <numeric>
#include <string>
#include <vector>

#include "api_internal.h"
#include "checks.h"

using sbim::Group;

namespace sbim_api {

thread_local std::string g_init_error;

int fail(sbim_handle *h, int code, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (h)
    h->err = buf;
  else
    g_init_error = buf;
  return code;
}

int hip_fail(sbim_handle *h, hipError_t e, const char *what) {
  return fail(h, SBIM_E_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

bool pow2_in(int n, int lo, int hi) { return n >= lo && n <= hi && (n & (n - 1)) == 0; }

bool finite_pos(double x) { return std::isfinite(x) && x > 0; }

// Gauss-Legendre nodes/weights on [-1, 1] by Newton iteration on P_n in long double.
void gauss_legendre(int n, std::vector<double> &x, std::vector<double> &w) {
  x.resize(n);
  w.resize(n);
  const long double pi = 3.141592653589793238462643383279502884L;
  for (int i = 0; i < n; ++i) {
    long double z = cosl(pi * (i + 0.75L) / (n + 0.5L));
    long double dp = 0;
    for (int it = 0; it < 100; ++it) {
      long double p0 = 1, p1 = z;
      for (int k = 2; k <= n; ++k) {
        const long double p2 = ((2 * k - 1) * z * p1 - (k - 1) * p0) / k;
        p0 = p1;
        p1 = p2;
      }
      dp = n * (z * p1 - p0) / (z * z - 1);
      const long double dz = p1 / dp;
      z -= dz;
      if (fabsl(dz) < 1e-19L) break;
    }
    long double p0 = 1, p1 = z;
    for (int k = 2; k <= n; ++k) {
      const long double p2 = ((2 * k - 1) * z * p1 - (k - 1) * p0) / k;
      p0 = p1;
      p1 = p2;
    }
    dp = n * (z * p1 - p0) / (z * z - 1);
    x[i] = static_cast<double>(z);
    w[i] = static_cast<double>(2 / ((1 - z * z) * dp * dp));
  }
}

// The matrix-core sweep needs windows of at least 4 lags (its ring steps), and
// outside the two-plane float32 form enough work: more than this many modes x lags
// per plane.
constexpr int kQuadMinWindow = 4;
constexpr double kQuadMinLags = 262144.0;

struct ModeKey {
  int w;
  double q;
  int nat;
};

hipError_t dev_alloc_bytes(void **p, size_t bytes) {
  *p = nullptr;
  if (bytes == 0) return hipSuccess;
  return hipMalloc(p, bytes);
}

void free_group(Group &g) {
  void *ptrs[] = {g.nat,   g.row0,  g.win,   g.geom,      g.blk_off,   g.blk_cap, g.blk_stride, g.cls_off,
                  g.cls_q, g.cls_w, g.table, g.ring,      g.state,     g.pending,
                  g.ring_adj, g.state_adj, g.lam_adj, g.pending_adj};
  for (void *p : ptrs)
    if (p) (void)hipFree(p);
  g = Group();
}

void free_handle(sbim_handle *h) {
  if (!h) return;
  (void)hipStreamSynchronize(h->stream);
  for (int i = 0; i < h->ngroups; ++i) free_group(h->g[i]);
  if (h->twiddle64 && h->twiddle64 != h->twiddle) (void)hipFree(h->twiddle64);
  void *ptrs[] = {h->twiddle, h->spec, h->spec_v, h->out_spec, h->out_adj};
  for (void *p : ptrs)
    if (p) (void)hipFree(p);
  for (auto e : h->ev_start) (void)hipEventDestroy(e);
  for (auto e : h->ev_stop) (void)hipEventDestroy(e);
  delete h;
}

// Free device memory; the environment variable SBIM_MEMORY_LIMIT (bytes) stands in for less.
hipError_t free_memory(size_t *free_b) {
  size_t total = 0;
  const hipError_t e = hipMemGetInfo(free_b, &total);
  if (const char *env = std::getenv("SBIM_MEMORY_LIMIT"))
    *free_b = std::min(*free_b, static_cast<size_t>(std::strtoull(env, nullptr, 10)));
  return e;
}

sbim::Form form_of(const sbim_handle *h) {
  return {h->depth, h->mfma ? h->quad_modes : 0, h->tiled, false};
}
long long ring_bytes(const sbim::Form &f, const Group &g, size_t real) {
  return (g.ring_records + (f.tiled ? sbim::kRecent * g.nblocks : 0)) * g.np * 3LL * sbim::kLanes * 2 *
         static_cast<long long>(real);
}
long long ring_bytes(const sbim_handle *h, const Group &g) { return ring_bytes(form_of(h), g, h->rsize); }
long long table_bytes(const sbim_handle *h, const Group &g) {
  return g.table_rows * 4LL * static_cast<long long>(h->rsize);
}
long long state_bytes_g(const Group &g) { return g.np * 3LL * g.M * 16; }
long long pending_bytes(const sbim::Form &f, const Group &g, size_t real) {
  return (f.depth + 1LL + (f.tiled ? sbim::kMidPeriod + 1 : 0)) * g.np * 10LL * g.M *
         static_cast<long long>(real);
}
long long pending_bytes(const sbim_handle *h, const Group &g) {
  return pending_bytes(form_of(h), g, h->rsize);
}
long long out_spec_bytes(const sbim_handle *h) {
  return static_cast<long long>(h->cfg.nplanes) * 3 * h->nh * 2 * static_cast<long long>(h->rsize);
}

int validate(const sbim_config *c) {
  if (!c) return fail(nullptr, SBIM_E_INVALID, "config is NULL");
  if (!pow2_in(c->n1, 4, 4096) || !pow2_in(c->n3, 4, 4096))
    return fail(nullptr, SBIM_E_INVALID, "n1=%d, n3=%d: each must be a power of two in [4, 4096]",
                c->n1, c->n3);
  if (!finite_pos(c->dx1) || !finite_pos(c->dx3) || !finite_pos(c->dt))
    return fail(nullptr, SBIM_E_INVALID, "dx1, dx3 and dt must be finite and > 0");
  if (c->nplanes < 1 || c->nplanes > SBIM_MAX_PLANES)
    return fail(nullptr, SBIM_E_INVALID, "nplanes=%d: must be 1 or 2", c->nplanes);
  for (int p = 0; p < c->nplanes; ++p) {
    const sbim_plane &pl = c->plane[p];
    if (pl.side != 1 && pl.side != -1)
      return fail(nullptr, SBIM_E_INVALID, "plane %d: side must be +1 or -1", p);
    if (!finite_pos(pl.mu) || !finite_pos(pl.cs) || !std::isfinite(pl.cp))
      return fail(nullptr, SBIM_E_INVALID, "plane %d: mu, cs must be finite and > 0", p);
    if (!(pl.cp > pl.cs * std::sqrt(4.0 / 3.0)))
      return fail(nullptr, SBIM_E_INVALID,
                  "plane %d: cp=%g must exceed cs*sqrt(4/3)=%g (positive bulk modulus)", p, pl.cp,
                  pl.cs * std::sqrt(4.0 / 3.0));
  }
  if (c->window_cap < 1 || c->window_cap > (1 << 20))
    return fail(nullptr, SBIM_E_INVALID, "window_cap=%d: must be in [1, 2^20]", c->window_cap);
  if (c->window_mode != SBIM_W_FIXED && c->window_mode != SBIM_W_PER_MODE &&
      c->window_mode != SBIM_W_STATIC)
    return fail(nullptr, SBIM_E_INVALID, "window_mode=%d unknown", c->window_mode);
  if (c->window_mode == SBIM_W_PER_MODE && !finite_pos(c->eta_w))
    return fail(nullptr, SBIM_E_INVALID, "eta_w must be finite and > 0");
  if (c->precision != SBIM_FP64 && c->precision != SBIM_FP32 && c->precision != SBIM_FP32_COMP)
    return fail(nullptr, SBIM_E_INVALID, "precision=%d unknown", c->precision);
  if (c->input_kind != SBIM_ABSOLUTE && c->input_kind != SBIM_INCREMENT)
    return fail(nullptr, SBIM_E_INVALID, "input_kind=%d unknown", c->input_kind);
  return SBIM_OK;
}

// Mean history window over the half-spectrum's modes of a plane with shear
// wave speed cs (the per-mode window rule of plan_group).
double mean_window(const sbim_config &c, double cs) {
  if (c.window_mode == SBIM_W_STATIC) return 1.0;
  if (c.window_mode == SBIM_W_FIXED) return c.window_cap;
  const int n1 = c.n1, h3 = c.n3 / 2 + 1;
  const double two_pi = 2.0 * M_PI;
  double sum = 0;
  for (int i1 = 0; i1 < n1; ++i1) {
    const int m1 = i1 < n1 / 2 ? i1 : i1 - n1;
    const double k1 = (two_pi * m1) / (n1 * c.dx1);
    for (int i3 = 0; i3 < h3; ++i3) {
      const double k3 = (two_pi * i3) / (c.n3 * c.dx3);
      const double q = std::sqrt(k1 * k1 + k3 * k3);
      if (q > 0)
        sum += std::min(static_cast<double>(c.window_cap),
                        std::ceil((two_pi * c.eta_w) / (q * cs * c.dt)));
    }
  }
  return sum / (static_cast<double>(n1) * h3);
}

// (q is bitwise the same for +-m1, so half of the bins are sorted.)
WaveOrder wave_order(const sbim_config &c) {
  const int n1 = c.n1, h3 = c.n3 / 2 + 1, half = n1 / 2 + 1;
  const double two_pi = 2.0 * M_PI;
  std::vector<std::pair<double, int>> v(static_cast<size_t>(half) * h3);
  for (int i3 = 0; i3 < h3; ++i3) {
    const double k3 = (two_pi * i3) / (c.n3 * c.dx3);
    for (int m1 = 0; m1 < half; ++m1) {
      const double k1 = (two_pi * m1) / (n1 * c.dx1);
      v[static_cast<size_t>(i3) * half + m1] = {std::sqrt(k1 * k1 + k3 * k3), i3 * half + m1};
    }
  }
  std::sort(v.begin(), v.end());
  WaveOrder o;
  std::vector<int> at(v.size());
  for (const auto &[q, bin] : v) {
    if (o.q.empty() || q != o.q.back()) o.q.push_back(q);
    at[bin] = static_cast<int>(o.q.size()) - 1;
  }
  o.rank.resize(static_cast<size_t>(n1) * h3);
  for (int i3 = 0; i3 < h3; ++i3)
    for (int i1 = 0; i1 < n1; ++i1)
      o.rank[static_cast<size_t>(i3) * n1 + i1] = at[static_cast<size_t>(i3) * half + std::min(i1, n1 - i1)];
  return o;
}

// How the modes share kernel rows (one for every distinct q): `quad`, the sorted positions
// per kernel row of the matrix-core sweep, 4 where the classes pad to multiples of 4 with
// little waste, as on square grids ((+-m1, m3) and (+-m3, m1)), 2 where mostly only +-m1
// share q; and the modes per distinct q.
struct RowSharing {
  int quad;
  double modes;
};
std::vector<int> modes_per_q(const WaveOrder &o) {
  std::vector<int> count(o.q.size(), 0);
  for (int r : o.rank) ++count[r];
  return count;
}
RowSharing row_sharing(const WaveOrder &o) {
  long long by4 = 0, by2 = 0;  // padded positions
  for (int n : modes_per_q(o)) {
    by4 += (n + 3) / 4 * 4;
    by2 += (n + 1) / 2 * 2;
  }
  return {4 * by4 <= 5 * by2 ? 4 : 2, static_cast<double>(o.rank.size()) / o.q.size()};
}

// The window from which the time-tiled form is faster than the vector sweep (outside the
// two-plane float32 form, where it is from 64 on).  Its fixed work (the middle level, 42 to
// 74 slots of sums, two rings written) shows on grids that fill the chip, the more where its
// quads share fewer modes than the vector sweep's rows do.  us a step, vector / tiled, one
// plane if not said: 256^2 float64 W = 64 35.7 / 32.7; 512 x 256 float64 64 46 / 49, 128
// 56 / 52; 512^2 float64 90 67 / 68, 128 74 / 71, float32 64 48.7 / 50.2, 90 52.2 / 51.2,
// compensated 64 51.0 / 49.7; with two modes a quad: 512^2 float64 128 two planes 129 / 133,
// 200 one plane 91 / 83, float32 90 55 / 57, 128 61 / 58; 1024 x 512, 3.7 modes a row,
// float64 200 142 / 156, 320 185 / 167, two planes 320 304 / 314, 450 370 / 350.
int tiled_window(const sbim_config &c, int np, const RowSharing &rows) {
  const long long nh = static_cast<long long>(c.n1) * (c.n3 / 2 + 1);
  const bool fp64 = c.precision == SBIM_FP64;
  if (nh < (1 << 16)) return 64;
  if (nh < (1 << 17)) return fp64 ? 96 : 64;
  if (rows.quad == 4) return fp64 ? 112 : c.precision == SBIM_FP32 ? 80 : 64;
  if (!fp64) return 132;
  return rows.modes < 3 ? 160 : np == 2 ? 384 : 256;
}

// Order of the time-tiled form's positions.  `keys` come sorted by (W desc, q asc,
// bin); each run of equal (W, q) is cut into quads of `quad` modes (padding: nat = -1),
// and the quads, whose order is free where every window is the same, are put so that
// a block's spectrum gathers and traction scatters are runs of neighbouring bins:
// with quads of 4, (+-m1, m3) and (+-m3, m1), along a Z curve over 4 x 4 tiles of
// (max, min) of the two indices (a block of 64 positions is one tile and touches
// four 4 x 4 patches of the spectrum); with quads of 2, +-m1, in spectrum order.
// (Sorted by q they were single bins: 1024^2 x 2 planes, float32: the traction
// scatter alone took 45 us of a step.)
void quad_order(const sbim_config &c, int quad, std::vector<ModeKey> &keys) {
  const int n1 = c.n1;
  auto m1 = [n1](int nat) { const int i = nat % n1; return i < n1 - i ? i : n1 - i; };  // |m1|
  auto m3 = [n1](int nat) { return nat / n1; };
  struct Quad { int w; unsigned long long key; size_t first; int count; };
  std::vector<Quad> quads;
  quads.reserve(keys.size() / quad + keys.size() / 8 + 1);
  auto spread = [](unsigned v) {  // bits of v to the even places
    unsigned long long r = 0;
    for (int i = 0; i < 16; ++i) r |= static_cast<unsigned long long>((v >> i) & 1u) << (2 * i);
    return r;
  };
  for (size_t s0 = 0; s0 < keys.size();) {
    size_t s1 = s0;
    while (s1 < keys.size() && keys[s1].w == keys[s0].w && keys[s1].q == keys[s0].q) ++s1;
    // modes of one orbit (equal max and min of the indices) next to each other
    auto lo = [&](int nat) { return std::min(m1(nat), m3(nat)); };
    auto hi = [&](int nat) { return std::max(m1(nat), m3(nat)); };
    if (quad == 4)
      std::sort(keys.begin() + s0, keys.begin() + s1, [&](const ModeKey &x, const ModeKey &y) {
        if (hi(x.nat) != hi(y.nat)) return hi(x.nat) < hi(y.nat);
        return x.nat < y.nat;
      });
    for (size_t s = s0; s < s1; s += quad) {
      const int nat = keys[s].nat;
      const unsigned a = quad == 4 ? hi(nat) : m1(nat), b = quad == 4 ? lo(nat) : m3(nat);
      const unsigned long long key = quad == 4
          ? ((spread(a >> 2) | spread(b >> 2) << 1) << 4 | (b & 3) << 2 | (a & 3))
          : static_cast<unsigned long long>(b) << 32 | a;
      quads.push_back(Quad{keys[s].w, key, s, static_cast<int>(std::min<size_t>(quad, s1 - s))});
    }
    s0 = s1;
  }
  std::sort(quads.begin(), quads.end(), [](const Quad &x, const Quad &y) {
    if (x.w != y.w) return x.w > y.w;
    if (x.key != y.key) return x.key < y.key;
    return x.first < y.first;
  });
  std::vector<ModeKey> out;
  out.reserve(quads.size() * quad);
  for (const Quad &z : quads)
    for (int i = 0; i < quad; ++i)
      out.push_back(i < z.count ? keys[z.first + i] : ModeKey{z.w, keys[z.first].q, -1});
  keys.swap(out);
}

// Mode geometry, windows, ordering and classes of one material group (host).
// With `quad` > 0 (the matrix-core sweeps: 2 or 4) every class is padded to a
// multiple of `quad` sorted positions with positions that hold no mode (bin -1,
// window 0, the class's row set), so each aligned group of `quad` lanes shares one
// kernel row; `tiled` also orders those groups (quad_order) and lays the rings out
// in time tiles.
void plan_group(const sbim_config &c, const WaveOrder &order, const sbim::Form &form, Group &g,
                std::vector<double> &geom, std::vector<long long> &blk_off, std::vector<int> &blk_cap,
                std::vector<int> &blk_stride, std::vector<double> &cls_q) {
  const int depth = form.depth, quad = form.quad;
  const bool tiled = form.tiled;
  const int n1 = c.n1, h3 = c.n3 / 2 + 1;
  const long long M = static_cast<long long>(n1) * h3;
  const double two_pi = 2.0 * M_PI;
  std::vector<ModeKey> keys(M);
  std::vector<double> qv(M), k1v(M), k3v(M);
  for (int i1 = 0; i1 < n1; ++i1) {
    const int m1 = i1 < n1 / 2 ? i1 : i1 - n1;
    const double k1 = (two_pi * m1) / (n1 * c.dx1);
    for (int i3 = 0; i3 < h3; ++i3) {
      const double k3 = (two_pi * i3) / (c.n3 * c.dx3);
      const long long f = static_cast<long long>(i3) * n1 + i1;  // spectrum bin
      const double q = order.q[order.rank[f]];
      int w = 0;
      if (q > 0) {
        if (c.window_mode == SBIM_W_STATIC) {
          w = 1;
        } else if (c.window_mode == SBIM_W_FIXED) {
          w = c.window_cap;
        } else {
          const double x = (two_pi * c.eta_w) / (q * g.cs * c.dt);
          w = static_cast<int>(std::min(static_cast<double>(c.window_cap), std::ceil(x)));
        }
      }
      keys[f] = ModeKey{w, q, static_cast<int>(f)};
      qv[f] = q;
      k1v[f] = k1;
      k3v[f] = k3;
    }
  }
  // Blocks hold modes of equal window.  With one window for all modes, modes
  // of equal q sit together so that a block's lanes share kernel rows.  With
  // per-mode windows (short histories, where the push and traction gathers
  // dominate) and in the quasi-dynamic limit (one lag, no sweep) modes of equal
  // window stay in spectrum order, so the gathers of the spectrum and the scatters of
  // the traction spectrum are contiguous runs (quasi-dynamic, 1024^2 float64: the step
  // launch 40 us against 82 in order of q).
  const bool by_q = c.window_mode == SBIM_W_FIXED || form.by_q;
  // (the keys come by bin: a stable counting sort, by q, where the one mode without a
  // window, q = 0, goes last, or by falling window)
  {
    int wtop = 0;
    for (const ModeKey &k : keys) wtop = std::max(wtop, k.w);
    const int nq = static_cast<int>(order.q.size());
    const auto place = [&](const ModeKey &k) {
      if (!by_q) return wtop - k.w;
      return k.w > 0 ? order.rank[k.nat] : nq;
    };
    std::vector<long long> first(static_cast<size_t>(by_q ? nq : wtop) + 2, 0);
    for (const ModeKey &k : keys) ++first[place(k) + 1];
    std::partial_sum(first.begin(), first.end(), first.begin());
    std::vector<ModeKey> sorted(keys.size());
    for (const ModeKey &k : keys) sorted[first[place(k)]++] = k;
    keys.swap(sorted);
  }
  cls_q.clear();
  g.h_cls_w.clear();
  if (quad && !tiled) {
    // pad each run of equal (W, q) (a class, sorted together) to a multiple of `quad`;
    // a padding position carries nat = -1
    std::vector<ModeKey> padded;
    padded.reserve(M + M / 2);
    for (long long s0 = 0; s0 < M;) {
      long long s1 = s0;
      while (s1 < M && keys[s1].w == keys[s0].w && keys[s1].q == keys[s0].q) ++s1;
      for (long long s = s0; s < s1; ++s) padded.push_back(keys[s]);
      for (long long r = (s1 - s0) % quad; r != 0 && r < quad; ++r)
        padded.push_back(ModeKey{keys[s0].w, keys[s0].q, -1});
      s0 = s1;
    }
    keys.swap(padded);
  }
  if (tiled) {
    for (const ModeKey &k : keys)
      if (k.w > 0 && (cls_q.empty() || cls_q.back() != k.q)) {
        cls_q.push_back(k.q);
        g.h_cls_w.push_back(k.w);
      }
    quad_order(c, quad, keys);
  }
  const long long Ms = static_cast<long long>(keys.size());  // sorted positions
  g.M = Ms;
  g.nblocks = (Ms + sbim::kLanes - 1) / sbim::kLanes;
  g.h_nat.resize(Ms);
  g.h_cls.resize(Ms);
  g.h_win.resize(Ms);
  geom.assign(4 * Ms, 0.0);
  // a class per distinct q (which fixes W): kernel rows are shared whatever the order;
  // spectrum order numbers them as they come up
  std::vector<int> class_of(!by_q && !tiled ? order.q.size() : 0, -1);
  for (long long s = 0; s < Ms; ++s) {
    const ModeKey &k = keys[s];
    if (k.nat < 0) {  // padding: the class of the position before it, no window, no bin
      g.h_nat[s] = -1;
      g.h_cls[s] = g.h_cls[s - 1];
      g.h_win[s] = 0;
      continue;
    }
    int cls = 0;
    if (k.w > 0 && tiled) {          // numbered in order of q, without q = 0
      cls = order.rank[k.nat] - 1;
    } else if (k.w > 0) {
      bool known = false;
      int *at = nullptr;
      if (by_q) {                    // sorted by (W, q): equal keys are neighbours
        known = s > 0 && k.w == keys[s - 1].w && k.q == keys[s - 1].q;
        if (known) cls = g.h_cls[s - 1];
      } else {
        at = &class_of[order.rank[k.nat]];
        known = *at >= 0;
        if (known) cls = *at;
      }
      if (!known) {
        cls = static_cast<int>(cls_q.size());
        if (at) *at = cls;
        cls_q.push_back(k.q);
        g.h_cls_w.push_back(k.w);
      }
    }
    g.h_nat[s] = k.nat;
    g.h_cls[s] = cls;
    g.h_win[s] = k.w;
    const double q = qv[k.nat];
    geom[4 * s + 0] = q;
    geom[4 * s + 1] = q > 0 ? k1v[k.nat] / q : 1.0;
    geom[4 * s + 2] = q > 0 ? k3v[k.nat] / q : 0.0;
  }
  g.nclasses = static_cast<long long>(cls_q.size());
  g.wmax = Ms > 0 ? keys[0].w : 0;
  blk_off.resize(g.nblocks);
  blk_cap.resize(g.nblocks);
  blk_stride.resize(g.nblocks);
  for (long long b = 0; b < g.nblocks; ++b) {  // the largest window of the block's modes
    int cap = 0;
    for (long long s = b * sbim::kLanes; s < std::min(Ms, (b + 1) * sbim::kLanes); ++s)
      cap = std::max(cap, g.h_win[s]);
    blk_cap[b] = cap;
  }
  if (tiled) {  // whole tiles of the time-tiled ring, at least four
    const int ts = sbim::kRingTileBytes / (c.precision == SBIM_FP64 ? 8 : 4);
    for (int &cap : blk_cap)
      if (cap > 0) cap = std::max((cap + ts - 1) / ts * ts, 4 * ts);
  }
  g.h_blk_cap = blk_cap;
  // Blocks of one sweep phase (b mod depth) are stored together; within a
  // phase, runs of consecutive blocks with equal capacity are stored slot-major.
  // The time-tiled form addresses a block's tiles with 32-bit offsets, so there
  // every block's ring is contiguous (a run of one; measured equal on gfx950).
  long long rec = 0;
  for (int ph = 0; ph < depth; ++ph) {
    for (long long b0 = ph; b0 < g.nblocks;) {
      long long b1 = b0, len = 0;
      while (b1 < g.nblocks && blk_cap[b1] == blk_cap[b0] && !(tiled && len > 0)) {
        b1 += depth;
        ++len;
      }
      for (long long b = b0, i = 0; b < b1; b += depth, ++i) {
        blk_off[b] = rec + i;
        blk_stride[b] = static_cast<int>(len);
      }
      rec += static_cast<long long>(blk_cap[b0]) * len;
      b0 = b1;
    }
  }
  g.ring_records = rec;
  // class-major table: the W_c rows of class c start at entry cls_off[c] and
  // are followed by one zero row
  g.h_cls_off.assign(g.nclasses, 0);
  long long off = 0;
  for (long long c = 0; c < g.nclasses; ++c) {
    g.h_cls_off[c] = off;
    off += g.h_cls_w[c] + 1;
  }
  g.table_rows = off;
}

hipError_t upload(void *dst, const void *src, size_t bytes, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  return hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, st);
}

int check_ptr(sbim_handle *h, const void *p, const char *name) {
  if (!p) return fail(h, SBIM_E_INVALID, "%s is NULL", name);
  return SBIM_OK;
}

int check_ready(sbim_handle *h) {
  if (h->ready) return SBIM_OK;
  return fail(h, SBIM_E_STATE, "the handle has no history buffers: planning it again failed");
}

// Forward real 2-D FFT of a [P][3][n1][n3] field into `spec`.
hipError_t fft_forward(sbim_handle *h, const void *field, void *spec) {
  return sbim::launch_fft_forward(h->fp64, field, spec, h->cfg.nplanes * 3, h->n1, h->n3,
                                  h->twiddle64, !h->in_order, h->stream);
}

// Inverse of a traction spectrum (destroyed) into a [P][3][n1][n3] field.
hipError_t fft_inverse(sbim_handle *h, const void *spec, void *scratch, void *field,
                       const void *add) {
  return sbim::launch_fft_inverse(h->fp64, spec, scratch, field, add, h->cfg.nplanes * 3, h->n1,
                                  h->n3,
                                  1.0 / (static_cast<double>(h->n1) * h->n3), h->twiddle,
                                  !h->in_order, h->stream);
}

// Adjoint buffers of every group, allocated and cleared on first use.  A group
// is complete once its state_adj is set; a failed allocation or clear frees
// that group's partial buffers again, so a later call starts from scratch.
int ensure_adjoint(sbim_handle *h) {
  size_t free_b = 0;
  if (h->tiled && h->bstep == 0 && free_memory(&free_b) == hipSuccess) {
    // no room beside the time-tiled form: the handle goes over to one that holds less
    size_t all = 0;
    for (int i = 0; i < h->ngroups; ++i)
      if (const Group &g = h->g[i]; !g.state_adj)
        all += ring_bytes(h, g) + 2 * state_bytes_g(g) + pending_bytes(h, g);
    if (all && all + (h->out_adj ? 0 : out_spec_bytes(h)) > free_b && adjoint_fits_in_order(h, free_b))
      if (const int rc = replan_in_order(h)) return rc;
  }
  for (int i = 0; i < h->ngroups; ++i) {
    Group &g = h->g[i];
    if (g.state_adj) continue;
    const size_t rb = static_cast<size_t>(ring_bytes(h, g));
    const size_t sb = static_cast<size_t>(state_bytes_g(g));
    const size_t pb = static_cast<size_t>(pending_bytes(h, g));
    const size_t need = rb + 2 * sb + pb + (h->out_adj ? 0 : static_cast<size_t>(out_spec_bytes(h)));
    if (free_memory(&free_b) == hipSuccess && need > free_b)
      return fail(h, SBIM_E_OOM, "adjoint buffers need %zu bytes, %zu free", need, free_b);
    void *ring = nullptr, *pending = nullptr;
    double *state = nullptr, *lam = nullptr;
    auto release = [&]() {
      void *ptrs[] = {ring, pending, state, lam};
      for (void *q : ptrs)
        if (q) (void)hipFree(q);
    };
    hipError_t e;
    if ((e = dev_alloc_bytes(&ring, rb)) != hipSuccess ||
        (e = dev_alloc_bytes(&pending, pb)) != hipSuccess ||
        (e = dev_alloc(&state, sb / 8)) != hipSuccess ||
        (e = dev_alloc(&lam, sb / 8)) != hipSuccess) {
      release();
      return fail(h, SBIM_E_OOM, "adjoint allocation failed: %s", hipGetErrorString(e));
    }
    if (!h->out_adj && (e = dev_alloc_bytes(&h->out_adj, out_spec_bytes(h))) != hipSuccess) {
      release();
      return fail(h, SBIM_E_OOM, "adjoint allocation failed: %s", hipGetErrorString(e));
    }
    e = rb ? hipMemsetAsync(ring, 0, rb, h->stream) : hipSuccess;
    if (e == hipSuccess) e = hipMemsetAsync(state, 0, sb, h->stream);
    if (e == hipSuccess) e = hipMemsetAsync(lam, 0, sb, h->stream);
    if (e != hipSuccess) {
      (void)hipStreamSynchronize(h->stream);
      release();
      return hip_fail(h, e, "clearing adjoint state");
    }
    g.ring_adj = ring;
    g.pending_adj = pending;
    g.lam_adj = lam;
    g.state_adj = state;
  }
  return SBIM_OK;
}

// The launch of step `w.step` for one group (push, traction spectrum and the
// sweep for the coming steps); while sbim_profile_conv is on, every n-th such
// launch is bracketed by a pair of the handle's reusable events.
int step_group(sbim_handle *h, Group &g, const sbim::StepLaunch &w, bool timed) {
  hipError_t e;
  if (timed && h->profile_every > 0 && h->profile_seen++ % h->profile_every == 0) {
    if (h->ev_used == h->ev_start.size()) {  // grow the reusable event pool
      hipEvent_t e0, e1;
      if ((e = hipEventCreate(&e0)) != hipSuccess) return hip_fail(h, e, "hipEventCreate");
      if ((e = hipEventCreate(&e1)) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return hip_fail(h, e, "hipEventCreate");
      }
      h->ev_start.push_back(e0);
      h->ev_stop.push_back(e1);
    }
    e = sbim::launch_step(h, g, w, h->ev_start[h->ev_used], h->ev_stop[h->ev_used]);
    ++h->ev_used;
  } else {
    e = sbim::launch_step(h, g, w);
  }
  if (e != hipSuccess) return hip_fail(h, e, "step kernel");
  return SBIM_OK;
}

// Groups of planes with equal (c_s, c_p), which share kernel tables and one pass.
void make_groups(sbim_handle *h) {
  const sbim_config *cfg = &h->cfg;
  h->ngroups = 0;
  for (int p = 0; p < cfg->nplanes; ++p) {
    const sbim_plane &pl = cfg->plane[p];
    int gi = -1;
    for (int i = 0; i < h->ngroups; ++i)
      if (h->g[i].cs == pl.cs && h->g[i].cp == pl.cp) gi = i;
    if (gi < 0) {
      gi = h->ngroups++;
      h->g[gi] = Group();
      h->g[gi].cs = pl.cs;
      h->g[gi].cp = pl.cp;
      h->g[gi].eta = pl.cp / pl.cs;
    }
    Group &g = h->g[gi];
    g.pl[g.np++] = sbim::PlaneParams{pl.mu, pl.cs, pl.cp / pl.cs, pl.side, p};
  }
}

// The form of a handle's material groups by its configuration; `in_order`: the float32
// history sums keep the lag order of the vector and in-order forms.
sbim::Form choose_form(const sbim_handle *h, const WaveOrder &order, bool in_order) {
  const sbim_config &c = h->cfg;
  // Sweep depth: steps served by one pass over a block's history.  Deeper
  // sweeps divide the history traffic, but the newest lags of each step (up
  // to depth + 1 of them) are summed by the mode items.  A lane holds the 10
  // sums of up to 8 steps (float32) or 6 (float64 and the compensated form,
  // whose sums take two registers each); depths 12 and 16 give each mode two
  // lanes, one per half of the steps.  Measured on gfx950 (two planes,
  // 512^2 at W = 1000, 1024^2 at W = 2000, 2048^2 with per-mode windows of
  // mean 18 lags): with long windows float64 and the compensated form run
  // fastest at 12; float32 at 8 for W = 1000 (by 5%) and at 12 for W = 2000
  // (by 7%); with mean windows under 64 lags every form runs fastest at 6.
  double wbar = 0;
  for (int p = 0; p < c.nplanes; ++p)
    wbar = std::max(wbar, mean_window(c, c.plane[p].cs));
  // Matrix-core sweep: one window for every mode (modes of a class then share
  // their kernel rows), windows of 64 lags or more so that the deep sweep pays, and
  // (outside the two-plane float32 forms) more than kQuadMinLags modes x lags per
  // plane and the windows of tiled_window: measured on gfx950 against the vector sweep, us
  // per step, 128 x 64 two-material float64 W = 150: 45 against 86; 512 x 128 two-material
  // float32 W = 250: 58 against 103; 512^2 x 2 float64 W = 1000: 207 against 352; one plane
  // 256^2 float32 W = 300, forward and adjoint: 33 against 38.
  const int np0 = h->g[0].np;  // (planes per group: the same for every group)
  const bool pair32 = !h->fp64 && np0 == 2;
  // (and a block's ring within the 32-bit byte offsets of the sweep's buffer loads)
  const bool able = c.window_mode == SBIM_W_FIXED && (in_order ? pair32 : c.window_cap >= kQuadMinWindow) &&
                    c.window_cap * (np0 * 3.0 * sbim::kLanes * 2) * static_cast<double>(h->rsize) < 4.29e9;
  const char *kind = std::getenv("SBIM_SWEEP_KIND");  // tuning override
  const bool vector = kind && std::strcmp(kind, "valu") == 0, matrix = kind && std::strcmp(kind, "mfma") == 0;
  RowSharing rows{4, 0};
  if (able && !in_order && !vector && (wbar >= 64 || matrix)) rows = row_sharing(order);
  const bool mfma = able && !vector &&
                    (matrix || (wbar >= 64 &&
                                (pair32 || (static_cast<double>(h->nh) * c.window_cap > kQuadMinLags &&
                                            c.window_cap >= tiled_window(c, np0, rows)))));
  int want_depth = 0;
  if (const char *env = std::getenv("SBIM_SWEEP_DEPTH")) want_depth = std::atoi(env);  // tuning override
  sbim::Form f;
  if (!mfma) {
    if (want_depth == 1 || want_depth == 2 || want_depth == 4 || want_depth == 6 ||
        want_depth == 8 || want_depth == 12 || want_depth == 16)
      f.depth = want_depth;
    else
      f.depth = wbar < 64 ? 6 : (h->comp || h->fp64 || wbar >= 1500 ? 12 : 8);
    return f;
  }
  const bool short_depth = np0 == 2 && want_depth == 16;
  f.tiled = !in_order;
  f.quad = f.tiled && !short_depth ? rows.quad : 4;
  f.depth = short_depth ? 16 : f.quad == 2 && np0 == 1 ? 64 : 32;
  if (!f.tiled) {
    // The in-order form addresses a block's history with 32-bit byte offsets from
    // its slot 0: every block's capacity times its slot stride (the blocks of its phase)
    // must stay below 2^30 floats, else the vector sweep plans the group instead.
    const std::vector<int> count = modes_per_q(order);
    long long padded = 0;
    for (size_t r = 1; r < count.size(); ++r) padded += (count[r] + 3) / 4 * 4;
    const long long blocks = (padded + sbim::kLanes - 1) / sbim::kLanes;
    if (c.window_cap * ((blocks + f.depth - 1) / f.depth) * 2LL * 3 * sbim::kLanes * 2 >= (1LL << 30))
      return {wbar < 64 ? 6 : (h->comp || wbar >= 1500 ? 12 : 8), 0, false, false};
  }
  return f;
}

// The plan of a handle's material groups (sweep form, mode order) and their device
// memory, tables and cleared state; `extra` more bytes are needed beside them.  With
// `in_order` the float32 history sums keep the lag order of the vector and in-order
// forms.  `tables` (or null): kernel tables of an earlier plan of the same fixed
// windows, whose classes and rows are the same; the groups take them over.  Errors are
// reported on `eh` (null: for sbim_last_error(NULL)); the caller frees the groups then.
int plan_handle(sbim_handle *h, bool in_order, size_t extra, sbim_handle *eh, void **tables) {
  const sbim_config &c = h->cfg;
  hipError_t e;
  h->ready = false;
  make_groups(h);
  const WaveOrder order = wave_order(c);
  struct HostPlan {
    std::vector<double> geom, cls_q;
    std::vector<long long> blk_off, row0;
    std::vector<int> blk_cap, blk_stride;
  };
  const sbim::Form form = choose_form(h, order, in_order);
  h->depth = form.depth;
  h->mfma = form.quad != 0;
  h->tiled = form.tiled;
  h->quad_modes = form.quad ? form.quad : 4;
  std::vector<HostPlan> plan(h->ngroups);
  for (int i = 0; i < h->ngroups; ++i)
    plan_group(c, order, form, h->g[i], plan[i].geom, plan[i].blk_off, plan[i].blk_cap,
               plan[i].blk_stride, plan[i].cls_q);
  if (h->mfma) {
    if (h->tiled) {
      // Lag ranges per quad, one wavefront each: one for fewer than 4 rounds of 32 lags,
      // two for fewer than 16, else four (measured on gfx950, us per pass at 1 / 2 / 4
      // ranges: W = 150 float64 rupture 128 x 64 238 / 222 / 232; W = 250 float32
      // 512 x 128 65 / 59 / 60; W = 1000 float64 512^2 with the sweep spread among the
      // other work - / 219 / 211, compensated - / 136 / 133; eight are slower there).
      // Plain float32 sums a range without a break: two from 3 rounds and four from 8 (two
      // planes) or 11, so that its error is that of the vector sweep's four ranges or of
      // the in-order form (against float64, 64^2 x 2 at 470 lags: 2.31e-7 with two ranges,
      // 1.84e-7 with four, 1.99e-7 in order; 128^2 one plane at 300 1.95e-7 with two,
      // 2.05e-7 in the vector sweep).
      const int rounds = (c.window_cap + 31) / 32;
      const bool plain = !h->fp64 && !h->comp;
      const int two = plain ? 3 : 4, four = !plain ? 16 : h->g[0].np == 2 ? 8 : 11;
      h->lag_chunks = rounds < two ? 1 : rounds < four ? 2 : 4;
    } else {
      // in-order form: as many as fit at least 16 blocks of 4 lags, up to two for the
      // compensated form (its registers allow three wavefronts per SIMD), four for
      // plain float32
      const int nblk = (std::max(0, h->g[0].wmax - 2) + 3) / 4;
      const int want = h->comp ? 2 : 4;
      h->lag_chunks = 1;
      while (h->lag_chunks < want && nblk >= 16 * 2 * h->lag_chunks) h->lag_chunks *= 2;
    }
    if (const char *env = std::getenv("SBIM_SWEEP_CHUNKS")) {  // tuning override
      const int v = std::atoi(env);
      if (v == 1 || v == 2 || v == 4) h->lag_chunks = v;
    }
    // Quads per work-group.  Time-tiled form: one, its history tiles are whole cache
    // lines (two quads measured within 2%, either way).  In-order form: two for the
    // compensated form, whose neighbouring quads share the cache lines of their history
    // (1024^2 at W = 2000: 5% faster), one for plain float32.
    h->sweep_quads = !h->tiled && h->comp && h->lag_chunks <= 2 ? 2 : 1;
    if (const char *env = std::getenv("SBIM_SWEEP_QUADS")) {  // tuning override
      const int v = std::atoi(env);
      if ((v == 1 || v == 2 || v == 4) && v * h->lag_chunks <= 4) h->sweep_quads = v;
    }
  }
  size_t need = extra;
  for (int i = 0; i < h->ngroups; ++i) {
    const Group &g = h->g[i];
    need += ring_bytes(h, g) + state_bytes_g(g) + pending_bytes(h, g);
    if (!(tables && tables[i])) need += table_bytes(h, g);
    need += g.M * (4 * 2 + 8 + 32) + g.nblocks * 16 + g.nclasses * 20;
  }
  size_t free_b = 0;
  e = free_memory(&free_b);
  if (e != hipSuccess) return fail(eh, SBIM_E_DEVICE, "hipMemGetInfo: %s", hipGetErrorString(e));
  // The time-tiled form holds more sums per mode: without room for it, the forms that hold
  // less.  (Its adjoint's room is looked at when an adjoint is asked for: ensure_adjoint.)
  if (h->tiled && need > free_b) return plan_handle(h, true, extra, eh, tables);
  if (need > free_b)
    return fail(eh, SBIM_E_OOM, "needs %zu bytes of device memory, %zu free", need, free_b);

  std::vector<double> glx, glw;
  gauss_legendre(sbim::kGaussN, glx, glw);
  double *d_glx = nullptr, *d_glw = nullptr;

#define TRY(expr)                                         \
  do {                                                    \
    e = (expr);                                           \
    if (e != hipSuccess) {                                \
      const int code = (e == hipErrorOutOfMemory) ? SBIM_E_OOM : SBIM_E_DEVICE; \
      (void)hipStreamSynchronize(h->stream);              \
      if (d_glx) (void)hipFree(d_glx);                    \
      if (d_glw) (void)hipFree(d_glw);                    \
      return fail(eh, code, "%s: %s", #expr, hipGetErrorString(e)); \
    }                                                     \
  } while (0)

  TRY(dev_alloc(&d_glx, glx.size()));
  TRY(dev_alloc(&d_glw, glw.size()));
  TRY(upload(d_glx, glx.data(), glx.size() * sizeof(double), h->stream));
  TRY(upload(d_glw, glw.data(), glw.size() * sizeof(double), h->stream));
  for (int i = 0; i < h->ngroups; ++i) {
    Group &g = h->g[i];
    HostPlan &hp = plan[i];
    hp.row0.resize(g.M);
    for (long long s = 0; s < g.M; ++s) hp.row0[s] = g.nclasses ? g.h_cls_off[g.h_cls[s]] : 0;
    TRY(dev_alloc(&g.nat, g.M));
    TRY(dev_alloc(&g.row0, g.M));
    TRY(dev_alloc(&g.win, g.M));
    TRY(dev_alloc(&g.geom, 4 * g.M));
    TRY(dev_alloc(&g.blk_off, g.nblocks));
    TRY(dev_alloc(&g.blk_cap, g.nblocks));
    TRY(dev_alloc(&g.blk_stride, g.nblocks));
    TRY(dev_alloc(&g.cls_off, g.nclasses));
    TRY(dev_alloc(&g.cls_q, g.nclasses));
    TRY(dev_alloc(&g.cls_w, g.nclasses));
    const bool kept = tables && tables[i];
    if (kept) {
      g.table = tables[i];
      tables[i] = nullptr;
    } else {
      TRY(dev_alloc_bytes(&g.table, table_bytes(h, g)));
    }
    TRY(dev_alloc_bytes(&g.ring, ring_bytes(h, g)));
    TRY(dev_alloc(&g.state, state_bytes_g(g) / 8));
    TRY(dev_alloc_bytes(&g.pending, pending_bytes(h, g)));
    TRY(upload(g.nat, g.h_nat.data(), g.M * sizeof(int), h->stream));
    TRY(upload(g.row0, hp.row0.data(), g.M * sizeof(long long), h->stream));
    TRY(upload(g.win, g.h_win.data(), g.M * sizeof(int), h->stream));
    TRY(upload(g.geom, hp.geom.data(), hp.geom.size() * sizeof(double), h->stream));
    TRY(upload(g.blk_off, hp.blk_off.data(), hp.blk_off.size() * sizeof(long long), h->stream));
    TRY(upload(g.blk_cap, hp.blk_cap.data(), hp.blk_cap.size() * sizeof(int), h->stream));
    TRY(upload(g.blk_stride, hp.blk_stride.data(), hp.blk_stride.size() * sizeof(int), h->stream));
    TRY(upload(g.cls_off, g.h_cls_off.data(), g.h_cls_off.size() * sizeof(long long), h->stream));
    TRY(upload(g.cls_q, hp.cls_q.data(), hp.cls_q.size() * sizeof(double), h->stream));
    TRY(upload(g.cls_w, g.h_cls_w.data(), g.h_cls_w.size() * sizeof(int), h->stream));
    if (ring_bytes(h, g)) TRY(hipMemsetAsync(g.ring, 0, ring_bytes(h, g), h->stream));
    TRY(hipMemsetAsync(g.state, 0, state_bytes_g(g), h->stream));
    TRY(hipMemsetAsync(g.pending, 0, pending_bytes(h, g), h->stream));
    if (c.window_mode == SBIM_W_STATIC) {
      // one row per class: the static integrals G_ab(infinity) of the kernels,
      // i.e. the static surface stiffness K_ab(0) less the instantaneous L-N
      // coupling, (w11, w12, w22, w33); then the zero row
      const double e2 = g.eta * g.eta;
      const double row[4] = {2.0 * e2 / (e2 + 1.0), -2.0 / (e2 + 1.0) - (g.eta - 2.0),
                             2.0 * e2 / (e2 + 1.0), 1.0};
      std::vector<double> t64(static_cast<size_t>(g.table_rows) * 4, 0.0);
      for (long long c = 0; c < g.nclasses; ++c)
        for (int k = 0; k < 4; ++k) t64[static_cast<size_t>(g.h_cls_off[c]) * 4 + k] = row[k];
      if (h->fp64) {
        TRY(upload(g.table, t64.data(), t64.size() * sizeof(double), h->stream));
        TRY(hipStreamSynchronize(h->stream));
      } else {
        std::vector<float> t32(t64.begin(), t64.end());
        TRY(upload(g.table, t32.data(), t32.size() * sizeof(float), h->stream));
        TRY(hipStreamSynchronize(h->stream));
      }
    } else if (!kept) {
      TRY(sbim::launch_tabulate(h->fp64, g, c.dt, d_glx, d_glw, h->stream));
    }
    // the host vectors must outlive the asynchronous copies
    TRY(hipStreamSynchronize(h->stream));
  }
  TRY(hipStreamSynchronize(h->stream));
#undef TRY
  (void)hipFree(d_glx);
  (void)hipFree(d_glw);
  h->ready = true;
  return SBIM_OK;
}

// The in-order form for a handle that will drive a strip, or in float32 a fault: the
// stick/slip state follows the rounding of the history sums from step to step, so the
// order of the sums is part of those results.  (A strip can amplify it: float64 strips on
// small grids, at a few tens of steps, ended 1e-7 to 1 apart with sums in another order;
// float64 faults stay within 1e-11.)  For the same reason its transforms keep the two-kernel
// form (the compiler fuses multiply-adds differently in the whole-field one).
int keep_sum_order(sbim_handle *h, bool strip) {
  if (h->fp64 && !strip) return SBIM_OK;
  const bool was = h->in_order;
  h->in_order = true;
  const int rc = h->tiled ? replan_in_order(h) : SBIM_OK;
  if (rc) h->in_order = was;
  return rc;
}

// One forward step: transform u (and v for VEL_INPUT), then the step launch of
// every material group with the given rule for the damping term's velocity.
int push_fields(sbim_handle *h, const void *u, const void *v, int vel_rule) {
  if (int rc = check_ready(h)) return rc;
  hipError_t e = fft_forward(h, u, h->spec);
  if (e != hipSuccess) return hip_fail(h, e, "forward FFT of u");
  if (vel_rule == sbim::VEL_INPUT) {
    e = fft_forward(h, v, h->spec_v);
    if (e != hipSuccess) return hip_fail(h, e, "forward FFT of v");
  }
  const bool incr = h->cfg.input_kind == SBIM_INCREMENT;
  for (int i = 0; i < h->ngroups; ++i) {
    Group &g = h->g[i];
    sbim::StepLaunch w;
    w.spec = h->spec;
    w.spec_v = vel_rule == sbim::VEL_INPUT ? h->spec_v : nullptr;
    w.ring = g.ring;
    w.state = g.state;
    w.pending = g.pending;
    w.lam = nullptr;
    w.out_a = h->out_spec;
    w.out_b = nullptr;
    w.nh = h->nh;
    w.step = h->step;
    w.dt = h->cfg.dt;
    w.state_rule = incr ? sbim::STATE_ACCUM : sbim::STATE_REPLACE;
    w.vel_rule = vel_rule;
    int rc = step_group(h, g, w, true);
    if (rc) return rc;
  }
  h->step += 1;
  return SBIM_OK;
}

}  // namespace sbim_api

using namespace sbim_api;

extern "C" {

int sbim_init(const sbim_config *cfg, sbim_handle **out) {
  if (!out) return fail(nullptr, SBIM_E_INVALID, "out is NULL");
  *out = nullptr;
  int rc = validate(cfg);
  if (rc != SBIM_OK) return rc;
  sbim_handle *h = new (std::nothrow) sbim_handle();
  if (!h) return fail(nullptr, SBIM_E_OOM, "host allocation failed");
  h->cfg = *cfg;
  h->stream = static_cast<hipStream_t>(cfg->stream);
  h->fp64 = cfg->precision == SBIM_FP64;
  h->comp = cfg->precision == SBIM_FP32_COMP;
  h->rsize = h->fp64 ? 8 : 4;
  h->n1 = cfg->n1;
  h->n3 = cfg->n3;
  h->h3 = cfg->n3 / 2 + 1;
  h->nh = static_cast<long long>(h->n1) * h->h3;
  hipError_t e = hipGetDevice(&h->device);
  if (e != hipSuccess) {
    delete h;
    return fail(nullptr, SBIM_E_DEVICE, "hipGetDevice: %s", hipGetErrorString(e));
  }
  // the device address of the allocation-free count's static scratch (once per device)
  e = sbim::count_scratch_address(h->device, &h->count_scratch);
  if (e != hipSuccess) {
    delete h;
    return fail(nullptr, SBIM_E_DEVICE, "hipGetSymbolAddress(scratch) on device %d: %s",
                h->device, hipGetErrorString(e));
  }

  const size_t spec_bytes = static_cast<size_t>(cfg->nplanes) * 3 * h->nh * 2 * sizeof(double);
  const size_t out_bytes = static_cast<size_t>(cfg->nplanes) * 3 * h->nh * 2 * h->rsize;
  // input spectra are float64 in every form; the traction spectrum is real_t
  rc = plan_handle(h, false, 2 * spec_bytes + out_bytes + sbim::kTwiddleN * 2 * (h->rsize + sizeof(double)),
                   nullptr);
  if (rc != SBIM_OK) {
    free_handle(h);
    return rc;
  }
#define TRY(expr)                                         \
  do {                                                    \
    e = (expr);                                           \
    if (e != hipSuccess) {                                \
      const int code = (e == hipErrorOutOfMemory) ? SBIM_E_OOM : SBIM_E_DEVICE; \
      free_handle(h);                                     \
      return fail(nullptr, code, "%s: %s", #expr, hipGetErrorString(e)); \
    }                                                     \
  } while (0)
  TRY(dev_alloc_bytes(&h->twiddle, sbim::kTwiddleN * 2 * h->rsize));
  if (h->fp64) {
    h->twiddle64 = h->twiddle;
  } else {
    TRY(dev_alloc_bytes(&h->twiddle64, sbim::kTwiddleN * 2 * sizeof(double)));
    TRY(sbim::upload_twiddles(true, h->twiddle64, h->stream));
  }
  TRY(dev_alloc_bytes(&h->spec, spec_bytes));
  TRY(dev_alloc_bytes(&h->spec_v, spec_bytes));
  TRY(dev_alloc_bytes(&h->out_spec, out_bytes));
  TRY(sbim::upload_twiddles(h->fp64, h->twiddle, h->stream));
  TRY(hipStreamSynchronize(h->stream));
#undef TRY
  *out = h;
  return SBIM_OK;
}

int sbim_push_displacement(sbim_handle *h, const void *u, const void *v) {
  if (!h) return fail(nullptr, SBIM_E_INVALID, "handle is NULL");
  int rc = check_ptr(h, u, "u");
  if (rc) return rc;
  const bool incr = h->cfg.input_kind == SBIM_INCREMENT;
  return push_fields(h, u, v, v ? sbim::VEL_INPUT : (incr ? sbim::VEL_SCALE : sbim::VEL_DIFF));
}

int sbim_tractions(sbim_handle *h, const void *tau_inf, void *tau) {
  if (!h) return fail(nullptr, SBIM_E_INVALID, "handle is NULL");
  int rc = check_ptr(h, tau, "tau");
  if (rc) return rc;
  if (h->step == 0) return fail(h, SBIM_E_STATE, "sbim_tractions before any push");
  // the traction spectrum of the last step was completed by its push; the
  // forward spectrum buffer serves as scratch until the next push
  hipError_t e = fft_inverse(h, h->out_spec, h->spec, tau, tau_inf);
  if (e != hipSuccess) return hip_fail(h, e, "inverse FFT");
  return SBIM_OK;
}

int sbim_backward(sbim_handle *h, const void *g_tau, void *du, void *dv) {
  if (!h) return fail(nullptr, SBIM_E_INVALID, "handle is NULL");
  int rc = check_ptr(h, g_tau, "dL_dtau");
  if (rc) return rc;
  rc = check_ptr(h, du, "dL_du");
  if (rc) return rc;
  rc = check_ready(h);
  if (rc) return rc;
  rc = ensure_adjoint(h);
  if (rc) return rc;
  hipError_t e = fft_forward(h, g_tau, h->spec);
  if (e != hipSuccess) return hip_fail(h, e, "forward FFT of dL/dtau");
  const bool incr = h->cfg.input_kind == SBIM_INCREMENT;
  for (int i = 0; i < h->ngroups; ++i) {
    Group &g = h->g[i];
    sbim::StepLaunch w;
    w.spec = h->spec;
    w.spec_v = nullptr;
    w.ring = g.ring_adj;
    w.state = g.state_adj;
    w.pending = g.pending_adj;
    w.lam = incr ? g.lam_adj : nullptr;
    w.out_a = h->out_adj;
    w.out_b = dv ? h->spec_v : nullptr;
    w.nh = h->nh;
    w.step = h->bstep;
    w.dt = h->cfg.dt;
    w.state_rule = sbim::STATE_REPLACE;
    // transpose of the velocity rule of the forward push
    w.vel_rule = dv ? sbim::VEL_COPY : (incr ? sbim::VEL_SCALE : sbim::VEL_DIFF);
    rc = step_group(h, g, w, false);
    if (rc) return rc;
  }
  e = fft_inverse(h, h->out_adj, h->spec, du, nullptr);
  if (e != hipSuccess) return hip_fail(h, e, "inverse FFT of dL/du");
  if (dv) {
    e = fft_inverse(h, h->spec_v, h->spec, dv, nullptr);
    if (e != hipSuccess) return hip_fail(h, e, "inverse FFT of dL/dv");
  }
  h->bstep += 1;
  return SBIM_OK;
}

int sbim_backward_reset(sbim_handle *h) {
  if (!h) return fail(nullptr, SBIM_E_INVALID, "handle is NULL");
  if (int rc = check_ready(h)) return rc;
  for (int i = 0; i < h->ngroups; ++i) {
    Group &g = h->g[i];
    if (!g.state_adj) continue;
    const size_t rb = static_cast<size_t>(ring_bytes(h, g));
    hipError_t e = hipSuccess;
    if (rb) e = hipMemsetAsync(g.ring_adj, 0, rb, h->stream);
    if (e == hipSuccess) e = hipMemsetAsync(g.state_adj, 0, state_bytes_g(g), h->stream);
    if (e == hipSuccess) e = hipMemsetAsync(g.lam_adj, 0, state_bytes_g(g), h->stream);
    if (e != hipSuccess) return hip_fail(h, e, "clearing adjoint state");
  }
  h->bstep = 0;
  return SBIM_OK;
}

int sbim_reset(sbim_handle *h) {
  if (!h) return fail(nullptr, SBIM_E_INVALID, "handle is NULL");
  if (int rc = check_ready(h)) return rc;
  for (int i = 0; i < h->ngroups; ++i) {
    Group &g = h->g[i];
    hipError_t e = hipSuccess;
    if (ring_bytes(h, g)) e = hipMemsetAsync(g.ring, 0, ring_bytes(h, g), h->stream);
    if (e == hipSuccess) e = hipMemsetAsync(g.state, 0, state_bytes_g(g), h->stream);
    if (e != hipSuccess) return hip_fail(h, e, "clearing state");
  }
  h->step = 0;
  return sbim_backward_reset(h);
}

int sbim_destroy(sbim_handle *h) {
  free_handle(h);
  return SBIM_OK;
}

const char *sbim_last_error(const sbim_handle *h) {
  return h ? h->err.c_str() : g_init_error.c_str();
}

int sbim_set_stream(sbim_handle *h, void *stream) {
  if (!h) return fail(nullptr, SBIM_E_INVALID, "handle is NULL");
  hipStream_t next = static_cast<hipStream_t>(stream);
  if (next != h->stream) {
    // work queued on the new stream starts after everything queued so far
    hipEvent_t ev;
    hipError_t e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e != hipSuccess) return hip_fail(h, e, "sbim_set_stream: hipEventCreate");
    e = hipEventRecord(ev, h->stream);
    if (e == hipSuccess) e = hipStreamWaitEvent(next, ev, 0);
    (void)hipEventDestroy(ev);
    if (e != hipSuccess) return hip_fail(h, e, "sbim_set_stream: ordering after the old stream");
  }
  h->stream = next;
  h->cfg.stream = stream;
  return SBIM_OK;
}

int sbim_set_dt(sbim_handle *h, double dt) {
  if (!h) return fail(nullptr, SBIM_E_INVALID, "handle is NULL");
  if (!(dt > 0) || !std::isfinite(dt)) return fail(h, SBIM_E_INVALID, "dt must be finite and > 0");
  if (h->cfg.window_mode != SBIM_W_STATIC)
    return fail(h, SBIM_E_STATE, "the time step of a dynamic handle is fixed at sbim_init");
  h->cfg.dt = dt;
  return SBIM_OK;
}

}  // extern "C"
