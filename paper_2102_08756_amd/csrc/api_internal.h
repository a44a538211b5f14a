// Host helpers shared by the C-ABI translation units (sbim_api.cpp defines them):
// error reporting, device allocation, buffer sizes and the per-step launch
// sequences that the fault and the strip reuse.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <vector>

#include "internal.h"

namespace sbim_api {

// Record a message on the handle (or, without one, for sbim_last_error(NULL)) and return `code`.
int fail(sbim_handle *h, int code, const char *fmt, ...);
// SBIM_E_DEVICE with the HIP error string.
int hip_fail(sbim_handle *h, hipError_t e, const char *what);

template <typename T>
hipError_t dev_alloc(T **p, size_t count) {
  *p = nullptr;
  if (count == 0) return hipSuccess;
  return hipMalloc(reinterpret_cast<void **>(p), count * sizeof(T));
}
hipError_t dev_alloc_bytes(void **p, size_t bytes);
hipError_t upload(void *dst, const void *src, size_t bytes, hipStream_t st);
int check_ptr(sbim_handle *h, const void *p, const char *name);
int check_ready(sbim_handle *h);  // the groups hold their buffers (a failed plan leaves none)

// The distinct wavenumbers q of a configuration's modes, ascending, and each bin's place
// among them.
struct WaveOrder {
  std::vector<double> q;
  std::vector<int> rank;  // [n1 h3] by bin i3 * n1 + i1
};
WaveOrder wave_order(const sbim_config &c);
sbim::Form form_of(const sbim_handle *h);
sbim::Form choose_form(const sbim_handle *h, const WaveOrder &order, bool in_order);
// Mode geometry, windows, order and classes of a material group in a form (host).
void plan_group(const sbim_config &c, const WaveOrder &order, const sbim::Form &form, sbim::Group &g,
                std::vector<double> &geom, std::vector<long long> &blk_off, std::vector<int> &blk_cap,
                std::vector<int> &blk_stride, std::vector<double> &cls_q);

// Device bytes of one material group's buffers (in the handle's form, or in another) and
// of the traction spectrum.
long long ring_bytes(const sbim::Form &f, const sbim::Group &g, size_t real);
long long pending_bytes(const sbim::Form &f, const sbim::Group &g, size_t real);
long long ring_bytes(const sbim_handle *h, const sbim::Group &g);
long long table_bytes(const sbim_handle *h, const sbim::Group &g);
long long state_bytes_g(const sbim::Group &g);
long long pending_bytes(const sbim_handle *h, const sbim::Group &g);
long long out_spec_bytes(const sbim_handle *h);

// Forward transform of a [P][3][n1][n3] field into a spectrum buffer; inverse of a
// traction spectrum (intact) into a field, with `scratch` for the intermediate.
hipError_t fft_forward(sbim_handle *h, const void *field, void *spec);
hipError_t fft_inverse(sbim_handle *h, const void *spec, void *scratch, void *field,
                       const void *add);
// The plan of a handle's groups and their device memory (sbim_api.cpp); the groups' memory
// freed; the adjoint buffers, allocated and cleared on first use.
int plan_handle(sbim_handle *h, bool in_order, size_t extra, sbim_handle *eh, void **tables = nullptr);
void free_group(sbim::Group &g);
int ensure_adjoint(sbim_handle *h);
// Plans a handle in the time-tiled form again with its sums in lag order, its forward and
// adjoint histories kept (snapshot_api.cpp).
int replan_in_order(sbim_handle *h);
// Whether that plan and its adjoint fit what is free and what the present plan holds.
bool adjoint_fits_in_order(const sbim_handle *h, size_t free_b);
// Plan a handle of a strip, or a float32 handle of a fault, with its sums in lag order.
int keep_sum_order(sbim_handle *h, bool strip);
// One forward step: transform u (and v for VEL_INPUT), then the step launch of
// every material group with the given rule for the damping term's velocity.
int push_fields(sbim_handle *h, const void *u, const void *v, int vel_rule);

}  // namespace sbim_api
