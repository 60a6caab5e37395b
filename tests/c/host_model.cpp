// The library's host code (pd_api.cpp, field.cpp) against a model of the HIP runtime and of the
// launches: device memory is host memory, a copy is a memcpy, a launch records what it was given
// (test_host_model.py builds and runs it).  For what the host side does with allocations, copies
// and pointers, where the device would show a mistake as a fault or not at all.  Prints one line
// per failed check and "host model ok"; the exit status is the number of failures.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <vector>

#include "pd_internal.h"

using namespace pdx;

static int failures = 0;
static void expect(bool cond, const char* what) {
  if (!cond) {
    std::printf("FAIL %s: %s\n", what, pd_last_error());
    ++failures;
  }
}

// ---- the runtime ----------------------------------------------------------------------

static std::set<void*> device_blocks;
static int host_pages = 0, host_allocs = 0, fills = 0, copies_of_n = 0;

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  *p = std::malloc(n ? n : 1);
  device_blocks.insert(*p);
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  device_blocks.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned int) {
  *p = std::malloc(n);
  ++host_pages;
  ++host_allocs;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::free(p);
  --host_pages;
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  if (n > sizeof(double)) ++copies_of_n;
  return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) {  // may return before it is done
  std::memset(d, v, n);
  ++fills;
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  std::memset(a, 0, sizeof *a);
  if (!device_blocks.count(const_cast<void*>(p))) return hipErrorInvalidValue;
  a->type = hipMemoryTypeDevice;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "model"; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = reinterpret_cast<hipEvent_t>(std::malloc(1));
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) {
  std::free(reinterpret_cast<void*>(e));
  return hipSuccess;
}
}

// ---- the launches ---------------------------------------------------------------------

static DensityOut last_density;
namespace pdx {
hipError_t launch_propagate(int, int, int, int, int, int, const SolveParams& p, hipStream_t) {
  for (long long i = 0; i < p.npts; ++i) p.n_out[i] = 1.0;
  return hipSuccess;
}
static hipError_t density(const DensityOut& o, long long npts) {
  last_density = o;
  if (!o.partial || !o.rho) return hipErrorInvalidValue;
  *o.rho = o.scale * (double)npts;
  if (o.rho_host) *o.rho_host = *o.rho;
  for (long long i = 0; o.n_copy && i < npts; ++i) o.n_copy[i] = 1.0;
  return hipSuccess;
}
hipError_t launch_snapshot(int, int, int, const SolveParams& p, const SnapshotParams&, const DensityOut& o,
                           hipStream_t) {
  for (long long i = 0; i < p.npts; ++i) p.n_out[i] = 1.0;
  return density(o, p.npts);
}
hipError_t launch_density(const double*, long long npts, const DensityOut& o, hipStream_t) { return density(o, npts); }
hipError_t static_scratch(int, double** out) {
  static std::vector<double> scratch(kStaticPartials + 1);
  *out = scratch.data();
  return hipSuccess;
}
long long density_partials(long long npts) { return (npts + 2047) / 2048; }
size_t state_values_per_point(int scheme) { return base_scheme(scheme) == PD_SCHEME_MIDPOINT ? 4 : 3; }
}  // namespace pdx

// ---- checks ---------------------------------------------------------------------------

static pd_field field() {
  pd_field f;
  std::memset(&f, 0, sizeof f);
  f.kind = PD_FIELD_SIN2;
  f.E0 = 0.2;
  f.omega = 0.6;
  f.cycles = 3;
  return f;
}

static pd_grid grid(int n = 40) {
  pd_grid g = nullptr;
  expect(pd_create_grid(n, n, -2.0, 2.0, -2.0, 2.0, PD_FP64, PD_SCHEME_STRANG, &g) == PD_OK, "grid");
  return g;
}

// What any of a new handle's allocations left missing, the next pd_set_field makes.
static void check_failed_allocations() {
  const pd_field f = field();
  for (int k = 1; k <= 4; ++k) {
    pd_grid g = grid();
    char spec[16];
    std::snprintf(spec, sizeof spec, "alloc@%d", k);
    double rho = 0.0;
    pd_set_fault(spec);
    expect(pd_set_field(g, &f, 500) == PD_ERR_NOMEM, spec);
    pd_set_fault(nullptr);
    expect(pd_set_field(g, &f, 500) == PD_OK, "field after a failed allocation");
    expect(g->d_table && g->d_n && g->d_partial && g->d_rho, "every buffer is there");
    if (g->d_rho) {
      expect(pd_propagate(g, -1, nullptr) == PD_OK && pd_density(g, nullptr, 0, &rho, nullptr) == PD_OK, "solve");
      expect(rho > 0.0, "rho");
    }
    pd_destroy_grid(g);
  }
  expect(fills == 0, "what is cleared is cleared by a copy, which waits");
}

// Handles one after another use one page; the pages of many are given back but for one.
static void check_slots() {
  const pd_field f = field();
  const int before = host_allocs;
  for (int i = 0; i < 20; ++i) {
    pd_grid g = grid();
    expect(pd_set_field(g, &f, 100) == PD_OK, "field");
    pd_destroy_grid(g);
  }
  expect(host_allocs <= before + 1, "one page for handles one after another");
  std::vector<pd_grid> many;
  std::set<double*> slots;
  for (int i = 0; i < 600; ++i) {
    many.push_back(grid(2));
    expect(pd_set_field(many.back(), &f, 100) == PD_OK, "field");
    slots.insert(many.back()->h_rho);
  }
  expect(slots.size() == 600 && !slots.count(nullptr), "a slot of its own for each");
  expect(host_pages == 3, "three pages for 600 handles");
  for (pd_grid g : many) pd_destroy_grid(g);
  expect(host_pages == 1, "one page stays");
}

// The buffers a handle keeps beside its field's samples do not grow with the step count.
static void check_kept_memory() {
  pd_field f = field();
  f.ellipticity = 0.5;
  pd_grid g = grid();
  for (long long n : {200000LL, 300000LL, 500LL, 400000LL, 400000LL}) {
    expect(pd_set_field(g, &f, n) == PD_OK, "field");
    expect(g->field.A_mid.size() == (size_t)n && g->field.Ay_mid.size() == (size_t)n, "the field's samples");
    expect(g->upload.capacity() + 8 * (g->spare_field.A_mid.capacity() + g->spare_field.Ay_mid.capacity()) <= 3 << 20,
           "at most 3 MiB beside them");
  }
  pd_set_fault("alloc@1");  // the table of a longer field: the buffers of a call that fails, too
  expect(pd_set_field(g, &f, 900000) == PD_ERR_NOMEM, "injected fault");
  pd_set_fault(nullptr);
  expect(g->upload.capacity() <= 1 << 20, "the upload of a failed call");
  pd_destroy_grid(g);
}

// n(p) for a device address: stored by the pass to memory of the device, copied to any other.
static void check_copy_of_n() {
  const pd_field f = field();
  pd_grid g = grid();
  const size_t m = 1600;
  void* device = nullptr;
  hipMalloc(&device, m * sizeof(double) + 8);
  std::vector<double> elsewhere(m);
  expect(pd_set_field(g, &f, 500) == PD_OK && pd_propagate(g, 250, nullptr) == PD_OK, "half of a solve");
  for (int call = 0; call < 3; ++call) {
    const auto density = [&](double* n) {
      double rho = 0.0;
      return call == 0   ? pd_snapshot(g, n, 1, &rho, nullptr)
             : call == 1 ? pd_density(g, n, 1, &rho, nullptr)
                         : pd_density_static(g, n, 1, &rho, nullptr);
    };
    if (call == 1) expect(pd_propagate(g, -1, nullptr) == PD_OK, "the rest");
    int copies = copies_of_n;
    expect(density(static_cast<double*>(device)) == PD_OK, "n to the device");
    expect(last_density.n_copy == device && copies_of_n == copies, "stored by the pass");
    elsewhere.assign(m, 0.0);
    expect(density(elsewhere.data()) == PD_OK, "n elsewhere");
    expect(!last_density.n_copy && copies_of_n == copies + 1 && elsewhere[m - 1] == 1.0, "copied");
    double* odd = reinterpret_cast<double*>(static_cast<char*>(device) + 4);
    device_blocks.insert(odd);
    expect(density(odd) == PD_OK && !last_density.n_copy, "an address that is no multiple of 8 is copied to");
    device_blocks.erase(odd);
  }
  hipFree(device);
  pd_destroy_grid(g);
}

// The kernel and the launch that a grid takes: by rows where columns would lose more to idle lanes
// than a new field costs by rows, and by columns every point of the grid in one lane of one wave.
static void check_strang_kernel() {
  struct {
    int nx, ny, precision, scheme;
    double ellipticity;
    bool columns;
  } grids[] = {{64, 64, PD_FP64, PD_SCHEME_STRANG, 0, true},         {64, 64, PD_FP32_FAST, PD_SCHEME_STRANG, 0, true},
               {512, 512, PD_FP32, PD_SCHEME_STRANG, 0, true},       {1500, 2047, PD_FP32, PD_SCHEME_STRANG, 0, true},
               {2048, 2048, PD_FP32_FAST, PD_SCHEME_STRANG, 0, true}, {1024, 1024, PD_FP32, PD_SCHEME_STRANG4, 0.5, true},
               {512, 512, PD_FP64, PD_SCHEME_STRANG4, 0, true},      {400, 300, PD_FP64, PD_SCHEME_STRANG, 0, true},
               {1184, 108, PD_FP32_FAST, PD_SCHEME_STRANG, 0, true},  {1403, 38, PD_FP32, PD_SCHEME_STRANG, 0.5, true},
               {28762, 35, PD_FP64, PD_SCHEME_STRANG, 0, false},      {18179, 129, PD_FP32, PD_SCHEME_STRANG4, 0.5, false},
               {64, 31, PD_FP64, PD_SCHEME_STRANG, 0, false}};
  pd_field f = field();
  for (const auto& q : grids) {
    pd_grid g = nullptr;
    expect(pd_create_grid(q.nx, q.ny, -2.0, 2.0, -2.0, 2.0, q.precision, q.scheme, &g) == PD_OK, "grid");
    f.ellipticity = q.ellipticity;
    expect(pd_set_field(g, &f, 4000) == PD_OK, "field");
    if ((g->series != 0) != q.columns) {
      std::printf("FAIL kernel of %d x %d precision %d scheme %d y component %g\n", q.nx, q.ny, q.precision, q.scheme,
                  q.ellipticity);
      ++failures;
    }
    pd_destroy_grid(g);
  }
  unsigned seed = 1;
  const auto pick = [&](int n) { return (int)((seed = seed * 1664525u + 1013904223u) >> 8) % n; };
  for (int trial = 0; trial < 300; ++trial) {
    Grid g;
    g.nx = 1 + pick(trial % 3 ? 70 : 300);
    g.ny = kColumnMinRows + pick(trial % 2 ? 40 : 500);
    const int precision = pick(3), stages = pick(2) ? 5 : 1, ell = pick(2), ppl = 1 << pick(4), waves = 1 << pick(3);
    const ColumnGeometry c = column_geometry(g, precision, stages, ell, ppl, pick(2) != 0);
    const int pair = precision == PD_FP64 ? 16 : 8, spaces = (1 << c.cshift) + ell, stride = c.chunk * stages + 16 / pair;
    expect(c.chunk >= 4 && c.chunk % 4 == 0 && spaces * stride * pair + 256 + 16 <= kColumnLdsWave, "the wave's LDS");
    std::vector<int> seen((size_t)g.nx * g.ny, 0);
    const int blocks = ((c.units + waves - 1) / waves + 7) / 8 * 8, shift = kColumnSuperShift - c.cshift;
    for (int unit = 0; unit < blocks * waves; ++unit) {  // as the kernel deals them
      const int super_units = c.segs << shift, super = unit / super_units, rest = unit % super_units;
      const int col0 = (super << kColumnSuperShift) + ((rest & ((1 << shift) - 1)) << c.cshift);
      if (unit >= c.units || col0 >= g.nx) continue;
      for (int lane = 0; lane < 64; ++lane)
        for (int q = 0; q < ppl; ++q) {
          const int col = col0 + (lane & ((1 << c.cshift) - 1));
          const long long row = (long long)((rest >> shift) * (64 >> c.cshift) + (lane >> c.cshift)) * ppl + q;
          if (col < g.nx && row < g.ny) ++seen[(size_t)row * g.nx + col];
        }
    }
    bool once = true;
    for (int n : seen) once = once && n == 1;
    expect(once, "every point in one lane");
  }
}

// The FP32 midpoint kernel of two terms holds 1/3 itself: no angle may ask it for another value.
void check_two_terms() {
  int two = 0;
  for (double x = 1e-6; x < 1e-2; x *= 1.01) {
    const pdx::TanPolynomial t = pdx::tan_polynomial(x, PD_FP32);
    if (t.terms != 2) continue;
    ++two;
    expect(t.c[2] == pdx::tan_series_coef(2), "two FP32 terms are the series' own");
    expect(pdx::tan_series_coef(3) * x * x <= 0x1p-27, "two FP32 terms hold to 2^-27");
  }
  expect(two > 100, "small angles take two FP32 terms");
}

int main() {
  check_two_terms();
  check_failed_allocations();
  check_slots();
  check_kept_memory();
  check_copy_of_n();
  check_strang_kernel();
  expect(device_blocks.empty(), "all device memory is given back");
  if (!failures) std::printf("host model ok\n");
  return failures;
}
