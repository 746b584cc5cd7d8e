// lattice.hip -- the C ABI of include/oreg.h: lattice handles, validation,
// device buffers, stream ordering and error reporting.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>

#include "kernels.hpp"
#include "staging.hpp"
#include "oreg.h"

using namespace oreg;

struct lb_lattice {
  lb_options opt{};
  int device = 0;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  void* buf[2] = {nullptr, nullptr};  // A/B population buffers
  int cur = 0;                        // buffer holding the current state
  size_t elem = 8;                    // bytes per stored population
  Geometry geo{};
  int fused_rows[8] = {};             // output rows per strip of fused launches, by step count
  int strips = 0;                     // wavefronts per strip of the strip pipeline; 0: not used
  int cus = 256;                      // compute units of the device
  StepPlan best;                      // the multi-step launch with the least time per step
  StepPlan exact[kPlanLevels + 1];    // plans for launches of exactly L steps (us = 0: not made yet)
  Coef64 coef{};
  double theta_energy = 0.0;          // theta of p = rho theta in the energy sum
  bool initialized = false;
  int64_t t = 0;
  double* tmp = nullptr;              // 3 * plane FP64 staging (lazy)
  double* aux = nullptr;              // kDiagBlocks*6 partials + 8 results
  unsigned int* counter = nullptr;    // invalid-input count of lb_init*, then the format flags
  bool numbers = false;               // steps store five numbers per node (see fused_numbers)
  // Format flag of buffer b (null where every buffer holds populations).
  unsigned int* fmt(int b) const { return numbers ? counter + 1 + b : nullptr; }
  PinnedPieces pieces;                // for copies to the caller's arrays
  std::string err;
};

namespace {

thread_local std::string t_err;

lb_status fail(lb_lattice* h, lb_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (h) h->err = buf;
  t_err = buf;
  return st;
}

lb_status hip_fail(lb_lattice* h, hipError_t e, const char* what) {
  const lb_status st = (e == hipErrorOutOfMemory) ? LB_ENOMEM : LB_EDEVICE;
  return fail(h, st, "%s: %s (%d)", what, hipGetErrorString(e), (int)e);
}

#define HIP_TRY(h, call)                                 \
  do {                                                   \
    hipError_t e_ = (call);                              \
    if (e_ != hipSuccess) return hip_fail((h), e_, #call); \
  } while (0)

// Makes the lattice's device current for the scope of one call.
struct DeviceScope {
  int prev = -1;
  bool ok = true;
  explicit DeviceScope(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    if (prev != dev) ok = (hipSetDevice(dev) == hipSuccess);
  }
  ~DeviceScope() {
    if (prev >= 0) {
      int now = -1;
      if (hipGetDevice(&now) == hipSuccess && now != prev) (void)hipSetDevice(prev);
    }
  }
};

bool is_finite(double v) { return std::isfinite(v); }

size_t storage_bytes(lb_storage s) {
  switch (s) {
    case LB_F64: return 8;
    case LB_F32S: return 4;
    case LB_F16S:
    case LB_BF16S: return 2;
  }
  return 0;
}

lb_status validate(const lb_options* o) {
  if (!o) return fail(nullptr, LB_EINVAL, "options pointer is NULL");
  if (o->nx < 1 || o->ny < 1) return fail(nullptr, LB_EINVAL, "nx and ny must be >= 1 (got %d x %d)", o->nx, o->ny);
  if (o->equilibrium != LB_EQ_GUIDED && o->equilibrium != LB_EQ_POLY2)
    return fail(nullptr, LB_EINVAL, "unknown equilibrium %d", (int)o->equilibrium);
  if (o->storage < LB_F64 || o->storage > LB_BF16S)
    return fail(nullptr, LB_EINVAL, "unknown storage %d", (int)o->storage);
  if (o->collision != LB_COLL_OREG && o->collision != LB_COLL_BGK)
    return fail(nullptr, LB_EINVAL, "unknown collision %d", (int)o->collision);
  if (o->boundary_x != LB_BC_PERIODIC && o->boundary_x != LB_BC_BOUNCEBACK)
    return fail(nullptr, LB_EINVAL, "unknown boundary %d", (int)o->boundary_x);
  // A HIP launch covers fewer than 2^32 work-items per dimension: the
  // single-step sweep launches sweep_work_items() of them (the row rounded up
  // to the storage's workgroup tile), the per-node kernels nx * ny rounded up
  // to 256.
  const int64_t plane = (int64_t)o->nx * (int64_t)o->ny;
  const int64_t items = std::max(sweep_work_items(o->storage, o->nx, o->ny), (plane + 255) / 256 * 256);
  if (items > (int64_t)4294967040LL)
    return fail(nullptr, LB_EINVAL, "lattice %d x %d is too large for one launch", o->nx, o->ny);
  if (!is_finite(o->tau) || !(o->tau > 0.5))
    return fail(nullptr, LB_EINVAL, "tau must be finite and > 1/2 (got %g)", o->tau);
  if (!is_finite(o->theta)) return fail(nullptr, LB_EINVAL, "theta must be finite");
  if (o->equilibrium == LB_EQ_GUIDED && !(o->theta > 0.0 && o->theta < 1.0))
    return fail(nullptr, LB_EINVAL, "guided equilibrium needs 0 < theta < 1 (got %g)", o->theta);
  if (o->equilibrium == LB_EQ_POLY2 && std::fabs(o->theta - 1.0 / 3.0) > 1e-12)
    return fail(nullptr, LB_EINVAL, "polynomial equilibrium needs theta = 1/3 (got %.17g)", o->theta);
  if (o->storage != LB_F64 && (!is_finite(o->rho0) || !(o->rho0 > 0.0)))
    return fail(nullptr, LB_EINVAL, "rho0 must be finite and > 0 for shifted storage");
  if (o->fuse_steps < 0 || o->fuse_steps > 2)
    return fail(nullptr, LB_EINVAL, "fuse_steps must be 0, 1 or 2 (got %d)", o->fuse_steps);
  return LB_OK;
}

Coef64 make_coef(const lb_options& o) {
  const double th = (o.equilibrium == LB_EQ_POLY2) ? 1.0 / 3.0 : o.theta;
  Coef64 c;
  c.theta = th;
  c.a0 = 1.0 - th;
  c.a1 = 0.5 * th;
  c.kappa0 = (1.0 - 1.0 / o.tau) / (2.0 * th * th);
  c.omega = 1.0 / o.tau;
  c.rho0 = (o.storage == LB_F64) ? 0.0 : o.rho0;
  return c;
}

lb_status ensure_tmp(lb_lattice* h) {
  if (h->tmp) return LB_OK;
  HIP_TRY(h, hipMalloc((void**)&h->tmp, 3 * (size_t)h->geo.plane * sizeof(double)));
  return LB_OK;
}

lb_status check_handle(lb_lattice* h) {
  if (!h) return fail(nullptr, LB_EINVAL, "lattice handle is NULL");
  return LB_OK;
}

// Partial sums of lb_diagnostics_device_noalloc: one row of six per
// reduction workgroup, in a file-scope device array instead of an allocation.
// Every GPU the library runs on holds its own copy until the process ends.
// In host code `scratch` only names the symbol: its device address comes
// from hipGetSymbolAddress, once per device, and only that address is passed
// to kernels.
constexpr int kMaxScratchDevices = 64;
static __device__ __align__(256) double scratch[kDiagBlocks * 6];
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxScratchDevices] = {};

// Device address of `scratch` on `dev` (the current device), looked up on
// the first call for that device.
lb_status scratch_ptr(lb_lattice* h, int dev, double** out) {
  if (dev < 0 || dev >= kMaxScratchDevices)
    return fail(h, LB_EDEVICE, "device %d: no scratch slot (at most %d devices)", dev,
                kMaxScratchDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return hip_fail(h, e != hipSuccess ? e : hipErrorUnknown,
                                               "hipGetSymbolAddress(scratch)");
    g_scratch_ptr[dev] = p;
  }
  *out = static_cast<double*>(g_scratch_ptr[dev]);
  return LB_OK;
}

// The plan for a launch of exactly L steps (made on first use and kept: it
// depends on the lattice's size and storage only).
const StepPlan& step_plan(lb_lattice* h, int L) {
  if (L == h->best.levels) return h->best;
  StepPlan& p = h->exact[L];
  if (p.us == 0) {
    p = plan_levels(h->opt.storage, h->geo.nx, h->geo.ny, L, h->cus);
    if (p.us < 0) p.kind = StepKind::sweep;
  }
  return p;
}

lb_status finish_init(lb_lattice* h) {
  unsigned int bad = 0;
  HIP_TRY(h, hipMemcpyAsync(&bad, h->counter, sizeof bad, hipMemcpyDeviceToHost, h->stream));
  HIP_TRY(h, hipStreamSynchronize(h->stream));
  if (bad) {
    h->initialized = false;
    return fail(h, LB_EINVAL, "%u node(s) with a non-finite field or rho <= 0", bad);
  }
  h->initialized = true;
  h->t = 0;
  return LB_OK;
}

}  // namespace

extern "C" {

void lb_options_init(lb_options* o) {
  if (!o) return;
  std::memset(o, 0, sizeof *o);
  o->tau = 1.0;
  o->theta = 1.0 / 3.0;
  o->equilibrium = LB_EQ_GUIDED;
  o->storage = LB_F64;
  o->collision = LB_COLL_OREG;
  o->boundary_x = LB_BC_PERIODIC;
  o->rho0 = 1.0;
  o->stream = nullptr;
  o->use_stream = 0;
  o->device = -1;
  o->check_nonfinite = 0;
  o->fuse_steps = 0;
}

lb_status lb_create(int nx, int ny, double tau, double theta, lb_equilibrium eq,
                    lb_lattice** out) {
  lb_options o;
  lb_options_init(&o);
  o.nx = nx;
  o.ny = ny;
  o.tau = tau;
  o.theta = theta;
  o.equilibrium = eq;
  return lb_create_ex(&o, out);
}

lb_status lb_create_ex(const lb_options* opt, lb_lattice** out) {
  if (!out) return fail(nullptr, LB_EINVAL, "out pointer is NULL");
  *out = nullptr;
  lb_status st = validate(opt);
  if (st != LB_OK) return st;

  int ndev = 0;
  hipError_t e = hipGetDeviceCount(&ndev);
  if (e != hipSuccess || ndev < 1)
    return fail(nullptr, LB_EDEVICE, "no HIP device available (%s)",
                e != hipSuccess ? hipGetErrorString(e) : "count is 0");
  int dev = opt->device;
  if (dev < 0) {
    if (hipGetDevice(&dev) != hipSuccess) dev = 0;
  }
  if (dev >= ndev) return fail(nullptr, LB_EINVAL, "device %d out of range (%d devices)", dev, ndev);

  lb_lattice* h = new (std::nothrow) lb_lattice;
  if (!h) return fail(nullptr, LB_ENOMEM, "host allocation failed");
  h->opt = *opt;
  h->opt.device = dev;
  h->device = dev;
  h->elem = storage_bytes(opt->storage);
  h->geo.nx = opt->nx;
  h->geo.ny = opt->ny;
  h->geo.plane = (int64_t)opt->nx * (int64_t)opt->ny;
  h->coef = make_coef(*opt);
  h->theta_energy = h->coef.theta;

  DeviceScope ds(dev);
  if (!ds.ok) {
    delete h;
    return fail(nullptr, LB_EDEVICE, "cannot select device %d", dev);
  }
  auto cleanup = [&](lb_status s) {
    lb_destroy(h);
    return s;
  };
  if (opt->use_stream) {
    h->stream = static_cast<hipStream_t>(opt->stream);
  } else {
    e = hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking);
    if (e != hipSuccess) return cleanup(hip_fail(nullptr, e, "hipStreamCreateWithFlags"));
    h->own_stream = true;
  }
  const size_t bytes = 9 * (size_t)h->geo.plane * h->elem;
  for (int b = 0; b < 2; ++b) {
    e = hipMalloc(&h->buf[b], bytes);
    if (e != hipSuccess) return cleanup(hip_fail(nullptr, e, "hipMalloc(populations)"));
  }
  e = hipMalloc((void**)&h->aux, (kDiagBlocks * 6 + 8) * sizeof(double));
  if (e != hipSuccess) return cleanup(hip_fail(nullptr, e, "hipMalloc(aux)"));
  e = hipMalloc((void**)&h->counter, 3 * sizeof(unsigned int));
  if (e != hipSuccess) return cleanup(hip_fail(nullptr, e, "hipMalloc(counter)"));
  if (hipDeviceGetAttribute(&h->cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    h->cus = 256;
  h->strips = plan_strips(h->opt.storage, h->geo.nx, h->geo.ny, h->opt.collision, h->opt.boundary_x);
  h->numbers = h->strips && fused_numbers(h->opt.collision, h->opt.boundary_x, h->opt.storage);
  if (h->strips) {
    for (int L = 1; L <= fused_levels(h->opt.storage); ++L)
      if (fused_levels_available(h->opt.collision, h->opt.boundary_x, h->opt.storage, L))
        h->fused_rows[L] = fused_rows(h->strips, h->geo.nx, h->geo.ny,
                                      fused_shape(h->opt.storage, h->strips, L), L);
  } else {
    h->best = plan_best(h->opt.storage, h->geo.nx, h->geo.ny, h->cus);
  }
  *out = h;
  return LB_OK;
}

lb_status lb_init(lb_lattice* h, const double* rho, const double* ux, const double* uy) {
  if (check_handle(h) != LB_OK) return LB_EINVAL;
  if (!rho || !ux || !uy) return fail(h, LB_EINVAL, "field pointer is NULL");
  const int64_t n = h->geo.plane;
  const double* const u[2] = {ux, uy};
  for (int64_t i = first_suspect_fields(rho, u, n); i < n; ++i) {
    if (!is_finite(rho[i]) || !is_finite(ux[i]) || !is_finite(uy[i]) || !(rho[i] > 0.0))
      return fail(h, LB_EINVAL, "node %lld has a non-finite field or rho <= 0", (long long)i);
  }
  DeviceScope ds(h->device);
  if (!ds.ok) return fail(h, LB_EDEVICE, "cannot select device %d", h->device);
  lb_status st = ensure_tmp(h);
  if (st != LB_OK) return st;
  const size_t bytes = (size_t)n * sizeof(double);
  HIP_TRY(h, hipMemcpyAsync(h->tmp, rho, bytes, hipMemcpyHostToDevice, h->stream));
  HIP_TRY(h, hipMemcpyAsync(h->tmp + n, ux, bytes, hipMemcpyHostToDevice, h->stream));
  HIP_TRY(h, hipMemcpyAsync(h->tmp + 2 * n, uy, bytes, hipMemcpyHostToDevice, h->stream));
  HIP_TRY(h, hipMemsetAsync(h->counter, 0, sizeof(unsigned int), h->stream));
  HIP_TRY(h, launch_init(h->opt.equilibrium, h->opt.storage, h->tmp, h->tmp + n, h->tmp + 2 * n,
                         h->buf[h->cur], h->geo, h->coef, h->counter, h->fmt(h->cur), h->stream));
  return finish_init(h);
}

lb_status lb_init_device(lb_lattice* h, const double* rho, const double* ux, const double* uy) {
  if (check_handle(h) != LB_OK) return LB_EINVAL;
  if (!rho || !ux || !uy) return fail(h, LB_EINVAL, "field pointer is NULL");
  DeviceScope ds(h->device);
  if (!ds.ok) return fail(h, LB_EDEVICE, "cannot select device %d", h->device);
  HIP_TRY(h, hipMemsetAsync(h->counter, 0, sizeof(unsigned int), h->stream));
  HIP_TRY(h, launch_init(h->opt.equilibrium, h->opt.storage, rho, ux, uy, h->buf[h->cur], h->geo,
                         h->coef, h->counter, h->fmt(h->cur), h->stream));
  return finish_init(h);
}

lb_status lb_step(lb_lattice* h, int64_t n) {
  if (check_handle(h) != LB_OK) return LB_EINVAL;
  if (n < 0) return fail(h, LB_EINVAL, "n must be >= 0 (got %lld)", (long long)n);
  if (!h->initialized) return fail(h, LB_ESTATE, "lattice is not initialized");
  if (n == 0) return LB_OK;
  DeviceScope ds(h->device);
  if (!ds.ok) return fail(h, LB_EDEVICE, "cannot select device %d", h->device);
  int64_t left = n;
  auto done = [&](int L) {
    h->cur = 1 - h->cur;
    h->t += L;
    left -= L;
  };
  // Whether one launch advances L steps by the tile or block sweep (or L = 1),
  // and that launch.
  auto has_plan = [&](int L) { return L == 1 || step_plan(h, L).kind != StepKind::sweep; };
  auto planned = [&](int L) {
    const StepPlan& p = step_plan(h, L);
    const hipError_t e =
        p.kind == StepKind::tile
            ? launch_tile_sweep(h->opt.equilibrium, h->opt.collision, h->opt.boundary_x,
                                h->opt.storage, h->buf[h->cur], h->buf[1 - h->cur], h->geo, h->coef,
                                p.tile, L, h->stream)
            : launch_block_sweep(h->opt.equilibrium, h->opt.collision, h->opt.boundary_x,
                                 h->opt.storage, h->buf[h->cur], h->buf[1 - h->cur], h->geo, h->coef,
                                 p.block, L, h->stream);
    if (e == hipSuccess) done(L);
    return e;
  };
  auto strip = [&](int L) {
    const hipError_t e = launch_fused_sweep(
        h->opt.equilibrium, h->opt.collision, h->opt.boundary_x, h->opt.storage, h->buf[h->cur],
        h->buf[1 - h->cur], h->geo, h->coef, h->strips, h->fused_rows[L], L, h->fmt(h->cur),
        h->fmt(1 - h->cur), h->stream);
    if (e == hipSuccess) done(L);
    return e;
  };
  const int levels = fused_levels(h->opt.storage);
  auto has_strip = [&](int L) {
    return fused_levels_available(h->opt.collision, h->opt.boundary_x, h->opt.storage, L);
  };
  const bool swap = swaps_buffers(
      n, h->opt.fuse_steps == 2 || (h->opt.fuse_steps == 0 && h->geo.plane >= kFusedFrom), levels,
      has_strip(2));
  if (h->strips && (h->numbers || h->opt.fuse_steps != 1) && has_strip(2)) {
    // Strip launches of any length (periodic OReg).  Lattices stored as numbers
    // spread the steps evenly over the cheapest number of launches (4096^2: one of
    // seven and one of one step 876 us, two of four 662; 2048^2, twelve steps: four
    // launches 369 us, two 270).  The others take as many full launches as they can;
    // a single step of theirs runs by the single-step sweep.
    const int64_t K = h->opt.fuse_steps == 1 ? 1 : levels;
    int64_t launches = h->numbers ? number_launches(n, (int)K, h->geo.plane, swap) : (n + K - 1) / K;
    for (; launches > 0; --launches) {
      const int L = (int)(h->numbers ? (left + launches - 1) / launches : std::min(K, left));
      if (!has_strip(L)) break;
      HIP_TRY(h, strip(L));
    }
  } else if (h->strips && h->opt.fuse_steps != 1) {
    // Strip launches of K steps only.  The remainder runs as block launches, which
    // read and write the state once where single steps would do so per step, spread
    // over the fewest that end in the right buffer: one for an odd number of steps,
    // two for four, two of three for six, and two steps as single sweeps (4096^2, us
    // for 2 .. 6 steps, single steps : so: F64 BGK 859, 1290, 1720, 2150, 2590 : 860,
    // 577, 1139, 708, 1153; F32S BGK, 2 .. 5: 397, 596, 795, 993 : 397, 304, 644, 305;
    // F16S BGK 222, 333, 444, 555 : 223, 175, 311, 417).
    const bool swap_rest = swap != (((n / levels) & 1) != 0);
    while (left >= levels) HIP_TRY(h, strip(levels));
    int64_t launches = 1;
    for (; launches < left; ++launches) {
      const int L = (int)((left + launches - 1) / launches);
      if (((launches & 1) != 0) == swap_rest && has_plan(L) && has_plan((int)(left / launches)))
        break;
    }
    for (; left > launches; --launches) HIP_TRY(h, planned((int)((left + launches - 1) / launches)));
  } else if (h->opt.fuse_steps != 1 && h->best.us >= 0) {
    // Tile and block launches: the steps in as few launches as the best plan
    // needs, spread evenly over them.  Where the last one would leave the state in
    // the wrong buffer, one more or, where longer launches are cheaper, one fewer
    // (520^2 F64, seven steps: three launches 28.6 us, one 24).  In FP64 longer
    // launches of lattices that leave CUs idle have to be clearly cheaper: they take
    // the CUs of other lattices in flight (24 steps in four launches / two, one
    // lattice and three in flight: 128^2 26.9 / 24.5 us and 15.6 / 22.3, 200 x 300 39.8 /
    // 41.3 and 20.9 / 36.7; F32S 128^2 25.8 / 21.8 and 15.7 / 11.9).  On lattices of a
    // few rows or columns the model flatters long launches (42 steps, one more / one
    // fewer, us per step: F32S 14 x 32143 2.56 / 3.12, 400001 x 2 3.35 / 3.74).
    const double single = 2.5 + 18 * (double)h->elem * h->geo.plane / 5e6;  // us of a sweep at 5 TB/s
    const double gain = std::min(h->geo.nx, h->geo.ny) <= 36 ? 0
                        : h->opt.storage == LB_F64 && h->geo.plane < 262144 ? 0.9 : 1;
    auto us = [&](int L) {
      return L == 1 ? single : L <= kPlanLevels && has_plan(L) ? step_plan(h, L).us : -1.0;
    };
    int64_t launches = launches_for(n, (n + h->best.levels - 1) / h->best.levels, swap, us, gain);
    for (; left > launches; --launches) {
      const int L = (int)((left + launches - 1) / launches);
      if (!has_plan(L)) break;
      HIP_TRY(h, planned(L));
    }
  }
  while (left > 0) {
    HIP_TRY(h, launch_sweep(h->opt.equilibrium, h->opt.collision, h->opt.boundary_x,
                            h->opt.storage, h->buf[h->cur], h->buf[1 - h->cur], h->geo, h->coef,
                            h->stream));
    done(1);
  }
  if (h->opt.check_nonfinite) {
    double d[6];
    lb_status st = lb_diagnostics(h, d);
    if (st != LB_OK) return st;
    if (d[5] > 0) return fail(h, LB_ENONFINITE, "%.0f node(s) hold non-finite populations", d[5]);
  }
  return LB_OK;
}

lb_status lb_moments_device(lb_lattice* h, double* out_dev) {
  if (check_handle(h) != LB_OK) return LB_EINVAL;
  if (!out_dev) return fail(h, LB_EINVAL, "output pointer is NULL");
  if (!h->initialized) return fail(h, LB_ESTATE, "lattice is not initialized");
  DeviceScope ds(h->device);
  if (!ds.ok) return fail(h, LB_EDEVICE, "cannot select device %d", h->device);
  HIP_TRY(h, launch_moments(h->opt.equilibrium, h->opt.storage, h->buf[h->cur], out_dev, h->geo,
                           h->coef, h->fmt(h->cur), h->stream));
  return LB_OK;
}

lb_status lb_moments(lb_lattice* h, double* out) {
  if (check_handle(h) != LB_OK) return LB_EINVAL;
  if (!out) return fail(h, LB_EINVAL, "output pointer is NULL");
  if (!h->initialized) return fail(h, LB_ESTATE, "lattice is not initialized");
  DeviceScope ds(h->device);
  if (!ds.ok) return fail(h, LB_EDEVICE, "cannot select device %d", h->device);
  lb_status st = ensure_tmp(h);
  if (st != LB_OK) return st;
  HIP_TRY(h, launch_moments(h->opt.equilibrium, h->opt.storage, h->buf[h->cur], h->tmp, h->geo,
                           h->coef, h->fmt(h->cur), h->stream));
  const size_t bytes = 3 * (size_t)h->geo.plane * sizeof(double);
  HostTransfer copy(h->pieces, h->stream, bytes);
  HIP_TRY(h, copy.to_host(out, h->tmp, bytes));
  HIP_TRY(h, copy.finish());
  return LB_OK;
}

lb_status lb_populations(lb_lattice* h, double* out) {
  if (check_handle(h) != LB_OK) return LB_EINVAL;
  if (!out) return fail(h, LB_EINVAL, "output pointer is NULL");
  if (!h->initialized) return fail(h, LB_ESTATE, "lattice is not initialized");
  DeviceScope ds(h->device);
  if (!ds.ok) return fail(h, LB_EDEVICE, "cannot select device %d", h->device);
  lb_status st = ensure_tmp(h);
  if (st != LB_OK) return st;
  const int64_t n = h->geo.plane;
  HostTransfer copy(h->pieces, h->stream, 9 * (size_t)n * sizeof(double));
  for (int i = 0; i < 9; i += 3) {
    // The staging buffer holds three planes; the stream's order keeps them until
    // their copy is done.
    HIP_TRY(h, launch_export_planes(h->opt.equilibrium, h->opt.storage, i, 3, h->buf[h->cur], h->tmp,
                                    h->geo, h->coef, h->fmt(h->cur), h->stream));
    HIP_TRY(h, copy.to_host(out + (size_t)i * n, h->tmp, 3 * (size_t)n * sizeof(double)));
  }
  HIP_TRY(h, copy.finish());
  return LB_OK;
}

lb_status lb_set_populations(lb_lattice* h, const double* in) {
  if (check_handle(h) != LB_OK) return LB_EINVAL;
  if (!in) return fail(h, LB_EINVAL, "input pointer is NULL");
  const int64_t n = h->geo.plane;
  DeviceScope ds(h->device);
  if (!ds.ok) return fail(h, LB_EDEVICE, "cannot select device %d", h->device);
  lb_status st = ensure_tmp(h);
  if (st != LB_OK) return st;
  // The populations are checked on the device on their way into the buffer that
  // the next step overwrites, and take the place of the state once they are
  // known to be valid (512^2: 1130 us with the check on the host, 620 us).
  void* const next = h->buf[1 - h->cur];
  double* const sum = h->tmp + 2 * n;
  HIP_TRY(h, hipMemsetAsync(h->counter, 0, sizeof(unsigned int), h->stream));
  for (int i = 0; i < 9; i += 2) {
    const int count = i < 8 ? 2 : 1;
    HIP_TRY(h, hipMemcpyAsync(h->tmp, in + (size_t)i * n, (size_t)count * n * sizeof(double),
                              hipMemcpyHostToDevice, h->stream));
    HIP_TRY(h, launch_import_planes(h->opt.storage, i, count, h->tmp, next, sum, h->counter, h->geo,
                                    h->coef, h->stream));
  }
  unsigned int bad = 0;
  HostTransfer count(h->pieces, h->stream, sizeof bad);
  HIP_TRY(h, count.to_host(&bad, h->counter, sizeof bad));
  HIP_TRY(h, count.finish());
  if (bad) {
    for (int64_t c = 0; c < n; ++c) {
      double rho = 0.0;
      for (int i = 0; i < 9; ++i) {
        const double v = in[(size_t)i * n + c];
        if (!is_finite(v)) return fail(h, LB_EINVAL, "population %d of node %lld is not finite", i, (long long)c);
        rho += v;
      }
      if (!(rho > 0.0)) return fail(h, LB_EINVAL, "node %lld has sum_i f_i <= 0", (long long)c);
    }
    return fail(h, LB_EINVAL, "%u node(s) with invalid populations", bad);
  }
  HIP_TRY(h, hipMemcpyAsync(h->buf[h->cur], next, 9 * (size_t)n * h->elem, hipMemcpyDeviceToDevice,
                            h->stream));
  if (h->numbers)  // the buffer holds populations
    HIP_TRY(h, hipMemsetAsync(h->fmt(h->cur), 0, sizeof(unsigned int), h->stream));
  HIP_TRY(h, hipStreamSynchronize(h->stream));
  h->initialized = true;
  h->t = 0;
  return LB_OK;
}

lb_status lb_diagnostics(lb_lattice* h, double out[6]) {
  if (check_handle(h) != LB_OK) return LB_EINVAL;
  if (!out) return fail(h, LB_EINVAL, "output pointer is NULL");
  if (!h->initialized) return fail(h, LB_ESTATE, "lattice is not initialized");
  DeviceScope ds(h->device);
  if (!ds.ok) return fail(h, LB_EDEVICE, "cannot select device %d", h->device);
  double* result = h->aux + kDiagBlocks * 6;
  HIP_TRY(h, launch_diagnostics(h->opt.equilibrium, h->opt.storage, h->buf[h->cur], h->aux, result,
                                h->geo, h->coef, h->theta_energy, h->fmt(h->cur), h->stream));
  HostTransfer copy(h->pieces, h->stream, 6 * sizeof(double));
  HIP_TRY(h, copy.to_host(out, result, 6 * sizeof(double)));
  HIP_TRY(h, copy.finish());
  return LB_OK;
}

lb_status lb_diagnostics_device_noalloc(lb_lattice* h, double* out_dev) {
  if (check_handle(h) != LB_OK) return LB_EINVAL;
  if (!out_dev) return fail(h, LB_EINVAL, "output pointer is NULL");
  if (!h->initialized) return fail(h, LB_ESTATE, "lattice is not initialized");
  DeviceScope ds(h->device);
  if (!ds.ok) return fail(h, LB_EDEVICE, "cannot select device %d", h->device);
  double* partials = nullptr;
  lb_status st = scratch_ptr(h, h->device, &partials);
  if (st != LB_OK) return st;
  // The same two kernels as lb_diagnostics, in the same reduction order; every
  // partial is written before the final kernel reads it, so nothing is cleared.
  HIP_TRY(h, launch_diagnostics(h->opt.equilibrium, h->opt.storage, h->buf[h->cur], partials, out_dev,
                                h->geo, h->coef, h->theta_energy, h->fmt(h->cur), h->stream));
  return LB_OK;
}

lb_status lb_density_profile(lb_lattice* h, double* out) {
  if (check_handle(h) != LB_OK) return LB_EINVAL;
  if (!out) return fail(h, LB_EINVAL, "output pointer is NULL");
  if (!h->initialized) return fail(h, LB_ESTATE, "lattice is not initialized");
  DeviceScope ds(h->device);
  if (!ds.ok) return fail(h, LB_EDEVICE, "cannot select device %d", h->device);
  lb_status st = ensure_tmp(h);
  if (st != LB_OK) return st;
  HIP_TRY(h, launch_profile(h->opt.equilibrium, h->opt.storage, h->buf[h->cur], h->tmp,
                            h->tmp + h->geo.nx, h->geo, h->coef, h->fmt(h->cur), h->stream));
  const size_t bytes = (size_t)h->geo.nx * sizeof(double);
  HostTransfer copy(h->pieces, h->stream, bytes);
  HIP_TRY(h, copy.to_host(out, h->tmp, bytes));
  HIP_TRY(h, copy.finish());
  return LB_OK;
}

lb_status lb_sync(lb_lattice* h) {
  if (check_handle(h) != LB_OK) return LB_EINVAL;
  DeviceScope ds(h->device);
  if (!ds.ok) return fail(h, LB_EDEVICE, "cannot select device %d", h->device);
  HIP_TRY(h, hipStreamSynchronize(h->stream));
  return LB_OK;
}

int64_t lb_time(const lb_lattice* h) { return h ? h->t : -1; }

lb_status lb_get_options(const lb_lattice* h, lb_options* out) {
  if (!h || !out) return fail(nullptr, LB_EINVAL, "NULL argument");
  *out = h->opt;
  return LB_OK;
}

int64_t lb_device_bytes(const lb_lattice* h) {
  if (!h) return 0;
  int64_t b = 2 * 9 * h->geo.plane * (int64_t)h->elem;
  b += (kDiagBlocks * 6 + 8) * (int64_t)sizeof(double) + 3 * (int64_t)sizeof(unsigned int);
  if (h->tmp) b += 3 * h->geo.plane * (int64_t)sizeof(double);
  return b;
}

lb_status lb_destroy(lb_lattice* h) {
  if (!h) return LB_OK;
  lb_status st = LB_OK;
  {
    DeviceScope ds(h->device);
    if ((h->stream || !h->own_stream) && hipStreamSynchronize(h->stream) != hipSuccess)
      st = LB_EDEVICE;
    for (int b = 0; b < 2; ++b)
      if (h->buf[b]) (void)hipFree(h->buf[b]);
    if (h->tmp) (void)hipFree(h->tmp);
    h->pieces.release();
    if (h->aux) (void)hipFree(h->aux);
    if (h->counter) (void)hipFree(h->counter);
    if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
  }
  delete h;
  return st;
}

lb_status lb_copy_device(const void* src, void* dst, int64_t bytes, void* hip_stream) {
  if (!src || !dst) return fail(nullptr, LB_EINVAL, "lb_copy_device: NULL buffer");
  if (bytes < 0 || bytes % 16 != 0)
    return fail(nullptr, LB_EINVAL, "lb_copy_device: %lld bytes is not a multiple of 16",
                (long long)bytes);
  const uintptr_t a = reinterpret_cast<uintptr_t>(src), b = reinterpret_cast<uintptr_t>(dst);
  if ((a | b) % 16 != 0)
    return fail(nullptr, LB_EINVAL, "lb_copy_device: buffers must be 16-byte aligned");
  if (bytes > 0 && a < b + (uintptr_t)bytes && b < a + (uintptr_t)bytes)
    return fail(nullptr, LB_EINVAL, "lb_copy_device: buffers overlap");
  if (bytes == 0) return LB_OK;
  const hipError_t e = launch_copy(src, dst, bytes, static_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) return hip_fail(nullptr, e, "copy_kernel launch");
  return LB_OK;
}

const char* lb_status_string(lb_status s) {
  switch (s) {
    case LB_OK: return "LB_OK";
    case LB_EINVAL: return "LB_EINVAL: invalid argument";
    case LB_ENOMEM: return "LB_ENOMEM: device allocation failed";
    case LB_EDEVICE: return "LB_EDEVICE: HIP error or no device";
    case LB_ESTATE: return "LB_ESTATE: lattice not initialized";
    case LB_ENONFINITE: return "LB_ENONFINITE: non-finite populations";
    case LB_EAGAIN: return "LB_EAGAIN: not now, retry later";
  }
  return "unknown lb_status";
}

const char* lb_last_error(const lb_lattice* h) {
  if (h) return h->err.c_str();
  return t_err.c_str();
}

}  // extern "C"
