// C ABI, snapshots: the full forward state and the running state, and history moved from one
// sweep form into another.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <iterator>
#include <string>
#include <vector>

#include "api_internal.h"

using sbim::Form;
using sbim::Group;
using namespace sbim_api;

namespace {

// A snapshot is the device memory as it lies.  Its header says all that decides how: the
// order of the modes, the padding of their classes, the size of its reals, the sweep depth
// (which blocks lie together, how many pending sums); and its size.  Two earlier kinds
// are told by their second word: one that names the order alone, and one without a mark,
// in lag order (by q also where one lag is all); their pending sums lay in other ways.
struct SnapshotHeader {
  long long step, mark, bytes;
  int order, quad, real, depth;
};
constexpr long long kHeaderBytes = 256;
constexpr long long kFormMark = 0x5342494d464f524d;
enum Order : int { kLagOrder = 0, kTimeTiled = 1, kSpectrumOrder = 2 };
constexpr long long kOrderMark[3] = {0x5342494d4c414730, 0x5342494d54494c30, 0x5342494d53504330};

Order order_of(const sbim_handle *h) {
  if (h->tiled) return kTimeTiled;
  return h->cfg.window_mode == SBIM_W_STATIC ? kSpectrumOrder : kLagOrder;
}

hipError_t save_header(const sbim_handle *h, void *dst, long long bytes) {
  const Form f = form_of(h);
  const SnapshotHeader hd{h->step, kFormMark, bytes, order_of(h), f.quad, static_cast<int>(h->rsize), f.depth};
  const hipError_t e = hipMemcpyAsync(dst, &hd, sizeof hd, hipMemcpyHostToDevice, h->stream);
  return e != hipSuccess ? e : hipStreamSynchronize(h->stream);  // hd goes with this frame
}

int load_header(sbim_handle *h, const void *src, SnapshotHeader &hd) {
  hipError_t e = hipMemcpyAsync(&hd, src, sizeof hd, hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) return hip_fail(h, e, "snapshot header");
  if (hd.step < 0) return fail(h, SBIM_E_INVALID, "snapshot header is corrupt");
  return SBIM_OK;
}

// A material group as another form lays it out (host).
struct Layout {
  Group g;
  std::vector<double> geom, cls_q;
  std::vector<long long> off;
  std::vector<int> cap, stride;
};
std::vector<Layout> lay_out(const sbim_handle *h, const Form &f) {
  const WaveOrder order = wave_order(h->cfg);
  std::vector<Layout> l(h->ngroups);
  for (int i = 0; i < h->ngroups; ++i) {
    l[i].g.cs = h->g[i].cs;
    l[i].g.np = h->g[i].np;
    plan_group(h->cfg, order, f, l[i].g, l[i].geom, l[i].off, l[i].cap, l[i].stride, l[i].cls_q);
  }
  return l;
}

long long snapshot_bytes(const sbim_handle *h, const Form &f, const Group *g[], bool running) {
  long long b = kHeaderBytes + (running ? 0 : out_spec_bytes(h));
  for (int i = 0; i < h->ngroups; ++i) {
    b += state_bytes_g(*g[i]);
    if (!running) b += ring_bytes(f, *g[i], h->rsize) + pending_bytes(f, *g[i], h->rsize);
  }
  return b;
}
long long own_bytes(const sbim_handle *h, bool running) {
  const Group *g[SBIM_MAX_PLANES] = {};
  for (int i = 0; i < h->ngroups; ++i) g[i] = &h->g[i];
  return snapshot_bytes(h, form_of(h), g, running);
}

// The form of a snapshot for handle h.  own: it lies as the handle's own memory does.
// (The running state is float64 in every precision and does not depend on the depth.)
int snapshot_form(sbim_handle *h, const SnapshotHeader &hd, bool running, Form &f, bool &own,
                  std::vector<Layout> &from) {
  const bool fixed = h->cfg.window_mode == SBIM_W_FIXED, is_static = h->cfg.window_mode == SBIM_W_STATIC;
  const Form mine = form_of(h);
  f = mine;
  own = true;
  if (hd.mark != kFormMark) {
    const bool marked = std::find(std::begin(kOrderMark), std::end(kOrderMark), hd.mark) != std::end(kOrderMark);
    if (marked ? hd.mark != kOrderMark[order_of(h)] : h->tiled)
      return fail(h, SBIM_E_INVALID, "snapshot orders the modes in another way than this handle");
    f.by_q = is_static && !marked;
    own = running && !f.by_q;  // (its pending sums are formed again)
    if (!own) from = lay_out(h, f);
    return SBIM_OK;
  }
  f.depth = running ? mine.depth : hd.depth;
  f.quad = hd.quad;
  f.tiled = hd.order == kTimeTiled;
  f.by_q = false;
  own = f == mine && (running || hd.real == static_cast<int>(h->rsize)) && hd.bytes == own_bytes(h, running);
  if (own) return SBIM_OK;
  bool fits = f.depth >= 1 && f.depth <= 64 && (f.quad == 0 || f.quad == 2 || f.quad == 4) &&
              (hd.order == kSpectrumOrder ? is_static : !is_static) && (f.quad == 0 || fixed) &&
              (!f.tiled || f.quad != 0) && (running || hd.real == static_cast<int>(h->rsize));
  if (fits) {
    from = lay_out(h, f);
    const Group *g[SBIM_MAX_PLANES] = {};
    for (int i = 0; i < h->ngroups; ++i) g[i] = &from[i].g;
    fits = snapshot_bytes(h, f, g, running) == hd.bytes;
  }
  return fits ? SBIM_OK : fail(h, SBIM_E_INVALID, "snapshot of another configuration or precision");
}

// The pending sums of group g, as the launches of the last `depth` steps before `step`
// formed them, from the history in its ring.  (Entries that a later step has replaced
// since meet rows past the window in the sums of `step` and after.)
hipError_t form_sums(const sbim_handle *h, const Group &g, void *ring, void *pending, long long step) {
  sbim::StepLaunch w{};
  w.ring = ring;
  w.pending = pending;
  w.nh = h->nh;
  w.dt = h->cfg.dt;
  w.sums_only = true;
  hipError_t e = hipMemsetAsync(pending, 0, pending_bytes(h, g), h->stream);
  for (w.step = std::max(0LL, step - h->depth); w.step < step && e == hipSuccess; ++w.step)
    e = sbim::launch_step(h, g, w);
  return e;
}

// A group's forward or adjoint history: ring, running state, adjoint's reverse running sum.
struct History {
  void *ring;
  double *state, *lam;
};

// Moves a history of form f into group g's own layout at `to` and forms its pending sums;
// without a ring only the state, and an empty history.  Synchronises.
int move_group(sbim_handle *h, const Group &g, const Form &f, const Layout &from, const History &src,
               const History &to, void *pending, long long step) {
  const long long nb = from.g.nblocks;
  std::vector<int> at(h->nh, -1), map(g.M, -1);
  for (long long t = 0; t < from.g.M; ++t)
    if (from.g.h_nat[t] >= 0) at[from.g.h_nat[t]] = static_cast<int>(t);
  for (long long s = 0; s < g.M; ++s)
    if (g.h_nat[s] >= 0) map[s] = at[g.h_nat[s]];
  int *d_map = nullptr, *d_cap = nullptr, *d_stride = nullptr;
  long long *d_off = nullptr;
  hipError_t e = dev_alloc(&d_map, g.M);
  if (e == hipSuccess) e = dev_alloc(&d_off, nb);
  if (e == hipSuccess) e = dev_alloc(&d_cap, nb);
  if (e == hipSuccess) e = dev_alloc(&d_stride, nb);
  if (e == hipSuccess) e = upload(d_map, map.data(), g.M * sizeof(int), h->stream);
  if (e == hipSuccess) e = upload(d_off, from.off.data(), nb * sizeof(long long), h->stream);
  if (e == hipSuccess) e = upload(d_cap, from.cap.data(), nb * sizeof(int), h->stream);
  if (e == hipSuccess) e = upload(d_stride, from.stride.data(), nb * sizeof(int), h->stream);
  if (e == hipSuccess)
    e = sbim::launch_relocate_state(src.state, from.g.M, to.state, g.M, d_map, g.np * 3, h->stream);
  if (e == hipSuccess && src.lam)
    e = sbim::launch_relocate_state(src.lam, from.g.M, to.lam, g.M, d_map, g.np * 3, h->stream);
  const size_t rb = static_cast<size_t>(ring_bytes(h, g));
  if (e == hipSuccess && rb) e = hipMemsetAsync(to.ring, 0, rb, h->stream);
  if (src.ring) {
    const sbim::RingSide a{src.ring, d_off, d_cap, d_stride, from.g.M, nb, from.g.ring_records, f.tiled};
    const sbim::RingSide b{to.ring, g.blk_off, g.blk_cap, g.blk_stride, g.M, g.nblocks, g.ring_records,
                           h->tiled};
    if (e == hipSuccess)
      e = sbim::launch_relocate_ring(h->fp64, a, b, d_map, g.np, step, g.wmax, h->stream);
    if (e == hipSuccess) e = form_sums(h, g, to.ring, pending, step);
  } else if (e == hipSuccess) {
    e = hipMemsetAsync(pending, 0, pending_bytes(h, g), h->stream);
  }
  const hipError_t e2 = hipStreamSynchronize(h->stream);  // the host arrays and the maps go
  if (e == hipSuccess) e = e2;
  for (void *p : {static_cast<void *>(d_map), static_cast<void *>(d_off), static_cast<void *>(d_cap),
                  static_cast<void *>(d_stride)})
    if (p) (void)hipFree(p);
  return e == hipSuccess ? SBIM_OK : hip_fail(h, e, "moving a history into this handle's form");
}

}  // namespace

namespace sbim_api {

bool adjoint_fits_in_order(const sbim_handle *h, size_t free_b) {
  const Form f = choose_form(h, wave_order(h->cfg), true);
  const std::vector<Layout> to = lay_out(h, f);
  long long need = h->out_adj ? 0 : out_spec_bytes(h), have = static_cast<long long>(free_b);
  for (int i = 0; i < h->ngroups; ++i) {
    const Group &a = to[i].g, &b = h->g[i];
    need += 2 * (ring_bytes(f, a, h->rsize) + pending_bytes(f, a, h->rsize)) + 3 * state_bytes_g(a) + a.M * 48;
    have += ring_bytes(h, b) + pending_bytes(h, b) + state_bytes_g(b) + b.M * 48;
  }
  return need <= have;
}

// The histories wait in host memory meanwhile, which the moves read directly: both forms
// need not fit the device together.
int replan_in_order(sbim_handle *h) {
  const Form was = form_of(h);
  const int n = h->ngroups;
  const bool fwd = h->step > 0, adj = h->bstep > 0;
  std::vector<Layout> from;
  if (fwd || adj) from = lay_out(h, was);
  size_t total = 0;
  for (int i = 0; i < n; ++i) {
    const size_t rb = ring_bytes(h, h->g[i]), sb = state_bytes_g(h->g[i]);
    total += (fwd ? rb + sb : 0) + (adj ? rb + 2 * sb : 0);
  }
  char *host = nullptr;
  hipError_t e = total ? hipHostMalloc(reinterpret_cast<void **>(&host), total, hipHostMallocDefault) : hipSuccess;
  if (e != hipSuccess) return fail(h, SBIM_E_OOM, "host memory for the history of a handle planned again");
  // (forward ring, state; adjoint ring, state, reverse sum) per group, from or to `p`
  const auto each = [&](auto &&part) {
    char *p = host;
    for (int i = 0; i < n; ++i) {
      const Group &g = fwd || adj ? from[i].g : h->g[i];
      const size_t rb = ring_bytes(was, g, h->rsize), sb = state_bytes_g(g);
      for (int a = 0; a < 2; ++a) {
        if (!(a ? adj : fwd)) continue;
        part(i, a != 0, History{p, reinterpret_cast<double *>(p + rb), reinterpret_cast<double *>(p + rb + sb)}, rb, sb);
        p += rb + (a ? 2 : 1) * sb;
      }
    }
  };
  each([&](int i, bool a, const History &to, size_t rb, size_t sb) {
    const Group &g = h->g[i];
    const hipMemcpyKind kind = hipMemcpyDeviceToHost;
    if (e == hipSuccess) e = hipMemcpyAsync(to.ring, a ? g.ring_adj : g.ring, rb, kind, h->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(to.state, a ? g.state_adj : g.state, sb, kind, h->stream);
    if (e == hipSuccess && a) e = hipMemcpyAsync(to.lam, g.lam_adj, sb, kind, h->stream);
  });
  const hipError_t e2 = hipStreamSynchronize(h->stream);
  if (e == hipSuccess) e = e2;
  if (e != hipSuccess) {
    if (host) (void)hipHostFree(host);
    return hip_fail(h, e, "planning the history sums in order");
  }
  // (fixed windows: classes are the distinct q in ascending order in every form, so the
  // kernel tables stay)
  const auto plan = [&](bool in_order) {
    void *tables[SBIM_MAX_PLANES] = {};
    for (int i = 0; i < n; ++i) {
      std::swap(tables[i], h->g[i].table);
      free_group(h->g[i]);
    }
    const int code = plan_handle(h, in_order, 0, h, tables);
    for (void *t : tables)
      if (t) (void)hipFree(t);
    return code;
  };
  int rc = plan(true);
  std::string why = h->err;
  if (rc) (void)plan(false);  // back to what it was; without memory for either the handle is not ready
  int back = h->ready ? SBIM_OK : SBIM_E_STATE;
  if (!back && adj) back = ensure_adjoint(h);
  each([&](int i, bool a, const History &src, size_t, size_t) {
    Group &g = h->g[i];
    if (back) return;
    back = a ? move_group(h, g, was, from[i], src, {g.ring_adj, g.state_adj, g.lam_adj}, g.pending_adj, h->bstep)
             : move_group(h, g, was, from[i], {src.ring, src.state, nullptr}, {g.ring, g.state, nullptr},
                          g.pending, h->step);
  });
  if (host) (void)hipHostFree(host);
  if (back) h->ready = false;  // (its history is lost)
  if (!rc && back) rc = back, why = h->err;
  if (rc) h->err = why;
  return rc;
}

}  // namespace sbim_api

extern "C" {

long long sbim_state_bytes(const sbim_handle *h) { return h ? own_bytes(h, false) : -1; }

long long sbim_running_state_bytes(const sbim_handle *h) { return h ? own_bytes(h, true) : -1; }

long long sbim_snapshot_bytes(sbim_handle *h, const void *src, int running) {
  if (!h) return fail(nullptr, SBIM_E_INVALID, "handle is NULL");
  int rc = check_ptr(h, src, "src");
  if (rc) return rc;
  SnapshotHeader hd{};
  rc = load_header(h, src, hd);
  if (rc) return rc;
  return hd.mark == kFormMark && hd.bytes > 0 ? hd.bytes : own_bytes(h, running != 0);
}

int sbim_save_state(sbim_handle *h, void *dst) {
  if (!h) return fail(nullptr, SBIM_E_INVALID, "handle is NULL");
  int rc = check_ptr(h, dst, "dst");
  if (!rc) rc = check_ready(h);
  if (rc) return rc;
  char *d = static_cast<char *>(dst);
  hipError_t e = save_header(h, d, own_bytes(h, false));
  d += kHeaderBytes;
  if (e == hipSuccess)
    e = hipMemcpyAsync(d, h->out_spec, out_spec_bytes(h), hipMemcpyDeviceToDevice, h->stream);
  d += out_spec_bytes(h);
  for (int i = 0; i < h->ngroups && e == hipSuccess; ++i) {
    Group &g = h->g[i];
    const size_t rb = ring_bytes(h, g), sb = state_bytes_g(g);
    if (rb) e = hipMemcpyAsync(d, g.ring, rb, hipMemcpyDeviceToDevice, h->stream);
    d += rb;
    if (e == hipSuccess) e = hipMemcpyAsync(d, g.state, sb, hipMemcpyDeviceToDevice, h->stream);
    d += sb;
    const size_t pb = pending_bytes(h, g);
    if (e == hipSuccess) e = hipMemcpyAsync(d, g.pending, pb, hipMemcpyDeviceToDevice, h->stream);
    d += pb;
  }
  if (e != hipSuccess) return hip_fail(h, e, "sbim_save_state");
  return SBIM_OK;
}

int sbim_load_state(sbim_handle *h, const void *src) {
  if (!h) return fail(nullptr, SBIM_E_INVALID, "handle is NULL");
  int rc = check_ptr(h, src, "src");
  if (!rc) rc = check_ready(h);
  if (rc) return rc;
  const char *s = static_cast<const char *>(src);
  SnapshotHeader hd{};
  Form f;
  bool own;
  std::vector<Layout> from;
  rc = load_header(h, s, hd);
  if (!rc) rc = snapshot_form(h, hd, false, f, own, from);
  if (rc) return rc;
  s += kHeaderBytes;
  hipError_t e = hipMemcpyAsync(h->out_spec, s, out_spec_bytes(h), hipMemcpyDeviceToDevice, h->stream);
  s += out_spec_bytes(h);
  for (int i = 0; i < h->ngroups && e == hipSuccess; ++i) {
    Group &g = h->g[i];
    const Group &sg = own ? g : from[i].g;
    const long long rb = ring_bytes(f, sg, h->rsize), sb = state_bytes_g(sg), pb = pending_bytes(f, sg, h->rsize);
    if (own) {
      if (rb) e = hipMemcpyAsync(g.ring, s, rb, hipMemcpyDeviceToDevice, h->stream);
      if (e == hipSuccess) e = hipMemcpyAsync(g.state, s + rb, sb, hipMemcpyDeviceToDevice, h->stream);
      if (e == hipSuccess) e = hipMemcpyAsync(g.pending, s + rb + sb, pb, hipMemcpyDeviceToDevice, h->stream);
    } else {
      char *p = const_cast<char *>(s);
      rc = move_group(h, g, f, from[i], {p, reinterpret_cast<double *>(p + rb), nullptr},
                      {g.ring, g.state, nullptr}, g.pending, hd.step);
      if (rc) return rc;
    }
    s += rb + sb + pb;
  }
  if (e != hipSuccess) return hip_fail(h, e, "sbim_load_state");
  h->step = hd.step;
  return SBIM_OK;
}

int sbim_save_running_state(sbim_handle *h, void *dst) {
  if (!h) return fail(nullptr, SBIM_E_INVALID, "handle is NULL");
  int rc = check_ptr(h, dst, "dst");
  if (!rc) rc = check_ready(h);
  if (rc) return rc;
  char *d = static_cast<char *>(dst);
  hipError_t e = save_header(h, d, own_bytes(h, true));
  d += kHeaderBytes;
  for (int i = 0; i < h->ngroups && e == hipSuccess; ++i) {
    const Group &g = h->g[i];
    e = hipMemcpyAsync(d, g.state, state_bytes_g(g), hipMemcpyDeviceToDevice, h->stream);
    d += state_bytes_g(g);
  }
  if (e != hipSuccess) return hip_fail(h, e, "sbim_save_running_state");
  return SBIM_OK;
}

int sbim_load_running_state(sbim_handle *h, const void *src) {
  if (!h) return fail(nullptr, SBIM_E_INVALID, "handle is NULL");
  int rc = check_ptr(h, src, "src");
  if (!rc) rc = check_ready(h);
  if (rc) return rc;
  const char *s = static_cast<const char *>(src);
  SnapshotHeader hd{};
  Form f;
  bool own;
  std::vector<Layout> from;
  rc = load_header(h, s, hd);
  if (!rc) rc = snapshot_form(h, hd, true, f, own, from);
  if (rc) return rc;
  s += kHeaderBytes;
  hipError_t e = hipSuccess;
  for (int i = 0; i < h->ngroups && e == hipSuccess; ++i) {
    Group &g = h->g[i];
    // the history before the snapshot is gone: start from an empty ring and no pending sums
    if (own) {
      e = hipMemcpyAsync(g.state, s, state_bytes_g(g), hipMemcpyDeviceToDevice, h->stream);
      const size_t rb = static_cast<size_t>(ring_bytes(h, g));
      if (e == hipSuccess && rb) e = hipMemsetAsync(g.ring, 0, rb, h->stream);
      if (e == hipSuccess) e = hipMemsetAsync(g.pending, 0, pending_bytes(h, g), h->stream);
      s += state_bytes_g(g);
    } else {
      rc = move_group(h, g, f, from[i], {nullptr, reinterpret_cast<double *>(const_cast<char *>(s)), nullptr},
                      {g.ring, g.state, nullptr}, g.pending, hd.step);
      if (rc) return rc;
      s += state_bytes_g(from[i].g);
    }
  }
  if (e != hipSuccess) return hip_fail(h, e, "sbim_load_running_state");
  h->step = hd.step;
  return SBIM_OK;
}

}  // extern "C"
