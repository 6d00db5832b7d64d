// vp_api.hip -- host side of the C ABI declared in include/vp.h: configuration
// checks, the context and its FP64 work fields, and the sequencing of the
// kernels of one step of Eq. (17) (Yoshikawa, Yoshida & Umemura, Sec. 2).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "vp.h"
#include "vp_internal.h"

using vp::Grid3;

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
int fail(int code, const char* fmt, ...)
{
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

bool debug_sync()
{
  static int v = -1;
  if (v < 0) {
    const char* e = getenv("VP_DEBUG_SYNC");
    v = (e && e[0] == '1') ? 1 : 0;
  }
  return v == 1;
}

}  // namespace

struct vp_ctx {
  vp_config cfg;
  void* f = nullptr;
  hipStream_t stream = nullptr;
  int device = 0;
  long long np = 0, nv3 = 0;
  double dx[3] = {0, 0, 0}, dv[3] = {0, 0, 0};
  Grid3 ng{};           // spatial grid
  Grid3 wg{};           // transform grid: ng (periodic) or 2 ng (isolated)
  double* rho = nullptr;
  double* phi = nullptr;      // (N+2)^3
  double* accel = nullptr;    // [3][np]
  double2* work = nullptr;    // wg cells
  double2* kspec = nullptr;   // Green's function spectrum (isolated, or a small grid)
  double2* tw[3] = {nullptr, nullptr, nullptr};
  double* s2[3] = {nullptr, nullptr, nullptr};   // sin^2(pi k / M) / dx^2 per axis
  double* part = nullptr;     // 2 * np
  double* red = nullptr;      // vp::RED_DOUBLES doubles on the device: results, then partials
  double* host = nullptr;     // 8 pinned doubles
  // reverse-mode work fields (allocated on first use)
  double* lphi = nullptr;     // (N+2)^3
  double* radj = nullptr;     // np
  double* dnu = nullptr;      // one value per line of a sweep
  long long dnu_len = 0;
  // workgroup sums of the x sweep (density without another pass over f);
  // null when the x sweep of this grid cannot produce them
  double* xsum = nullptr;
  // velocity cells per workgroup of the one-pass drift over all three axes (0:
  // none for this grid), and its sums, one per chunk and spatial cell
  int box3 = 0;
  bool small = false;         // gravity in one launch (gravity_small_supported)
  vp::SmallGravity sg{};      // its parts that do not change
  double* bsum = nullptr;
  // per-velocity-cell line coefficients of the one-pass T_z T_y (null when
  // the grid has no such pass)
  void* dtab = nullptr;
  // per-spatial-cell line coefficients of the kick passes (null when they work
  // them out themselves)
  void* ktab = nullptr;
  // position axes that share a pass of drift_pair: 1 for y and x, 2 for z and
  // y, 0 for none
  int pair = 0;
  // phase timing (vp_profile_*): pending event pairs per phase
  bool profiling = false;
  std::vector<hipEvent_t> ev_free;
  std::vector<std::pair<int, std::pair<hipEvent_t, hipEvent_t>>> ev_pending;
  double phase_ms[VP_NPHASE] = {};
  long long phase_n[VP_NPHASE] = {};
  // this device's address of the static scratch array (vp_sweep_adjoint_noalloc)
  double* scratch = nullptr;
};

// Scratch of vp_sweep_adjoint_noalloc: the per-line adjoint of the Courant
// number of one velocity sweep, one double per line, VP_NOALLOC_MAX_LINES lines
// (32 MiB). It is a static device array, so every device the library runs on
// holds its own copy from code-object load until the process ends. In host
// code the name is a host-side stand-in, never a device address: host code
// uses only the per-device address from hipGetSymbolAddress (scratch_address).
__device__ __align__(256) double scratch[VP_NOALLOC_MAX_LINES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_addr[kMaxDevices] = {};

// The current device's address of `scratch`, resolved once per device (the
// caller has made `device` current). Called from vp_init.
int scratch_address(int device, double** out)
{
  if (device < 0 || device >= kMaxDevices) return fail(VP_EUNSUPPORTED, "device index %d out of range", device);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_addr[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return fail(VP_EHIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
    g_scratch_addr[device] = static_cast<double*>(p);
  }
  *out = g_scratch_addr[device];
  return VP_OK;
}

}  // namespace

namespace {

#define HIP_TRY(expr)                                                                     \
  do {                                                                                    \
    hipError_t e_ = (expr);                                                               \
    if (e_ != hipSuccess) return fail(VP_EHIP, "%s: %s", #expr, hipGetErrorString(e_));   \
  } while (0)

int check_launch(vp_ctx* c, hipError_t e, const char* what)
{
  if (e != hipSuccess) return fail(VP_EHIP, "%s: %s", what, hipGetErrorString(e));
  if (debug_sync()) {
    e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return fail(VP_EHIP, "%s (sync): %s", what, hipGetErrorString(e));
  }
  return VP_OK;
}

#define LAUNCH(c, expr)                                 \
  do {                                                  \
    int r_ = check_launch((c), (expr), #expr);          \
    if (r_ != VP_OK) return r_;                         \
  } while (0)

// Gauss-Legendre rule of order n on [-1, 1]: nodes are the roots of P_n,
// found by Newton's method from the estimate cos(pi (i + 3/4) / (n + 1/2)),
// with P_n and P_n' from Bonnet's three-term recurrence; weights
// 2 / ((1 - x^2) P_n'(x)^2).
void gauss_legendre(int n, double* x, double* w)
{
  const double pi = 3.14159265358979323846;
  for (int i = 0; i < (n + 1) / 2; i++) {
    double z = std::cos(pi * (i + 0.75) / (n + 0.5)), dp = 0.0;
    for (int it = 0; it < 100; it++) {
      double p0 = 1.0, p1 = z;
      for (int k = 2; k <= n; k++) {
        const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
        p0 = p1;
        p1 = p2;
      }
      dp = n * (z * p1 - p0) / (z * z - 1.0);
      const double dz = p1 / dp;
      z -= dz;
      if (std::fabs(dz) < 1e-16) break;
    }
    x[i] = -z;
    x[n - 1 - i] = z;
    w[i] = w[n - 1 - i] = 2.0 / ((1.0 - z * z) * dp * dp);
  }
}

}  // namespace

// Integral of 1/|r| over the cell of widths dx, dy, dz centred on the origin: the
// potential of a unit-density cell at its own centre, which is the isolated
// kernel's value at zero offset. Since div(r/|r|) = 2/|r|, the divergence
// theorem makes the volume integral half the outward flux of r/|r|; on the two
// faces normal to axis l, r.n = h_l (the half width), so
//   I = sum_l h_l int_{face l} dA / |r|.
// Across one face coordinate the integrand has the antiderivative asinh, so
//   int_face dA/|r| = 4 int_0^{h_b} asinh(h_c / sqrt(h_l^2 + y^2)) dy,
// a smooth integrand (its nearest complex singularity is at y = i h_l),
// integrated with 16-point Gauss-Legendre panels no wider than h_l / 2.
double vp_cell_self_integral(double dx, double dy, double dz)
{
  g_err.clear();
  if (!(dx > 0.0) || !(dy > 0.0) || !(dz > 0.0) || !std::isfinite(dx + dy + dz)) {
    fail(VP_EINVAL, "cell widths must be finite and > 0");
    return NAN;
  }
  const int NG = 16;
  double gx[NG], gw[NG];
  gauss_legendre(NG, gx, gw);
  const double h[3] = {0.5 * dx, 0.5 * dy, 0.5 * dz};
  double total = 0.0;
  for (int l = 0; l < 3; l++) {
    const double hl = h[l];
    for (int t = 0; t < 2; t++) {  // (hb, hc) and (hc, hb): the face integral both ways, averaged
      const double hb = h[(l + 1 + t) % 3], hc = h[(l + 2 - t) % 3];
      const long panels = std::max(1L, (long)std::ceil(2.0 * hb / hl));
      const double width = hb / panels;
      double face = 0.0;
      for (long p = 0; p < panels; p++) {
        const double mid = (p + 0.5) * width;
        double acc = 0.0;
        for (int g = 0; g < NG; g++) {
          const double y = mid + 0.5 * width * gx[g];
          acc += gw[g] * std::asinh(hc / std::sqrt(hl * hl + y * y));
        }
        face += 0.5 * width * acc;
      }
      total += 0.5 * hl * 4.0 * face;
    }
  }
  return total;
}

namespace {

void release(vp_ctx* c)
{
  if (!c) return;
  hipFree(c->rho);
  hipFree(c->phi);
  hipFree(c->accel);
  hipFree(c->work);
  hipFree(c->kspec);
  for (auto& t : c->tw) hipFree(t);
  for (auto& t : c->s2) hipFree(t);
  hipFree(c->part);
  hipFree(c->xsum);
  hipFree(c->bsum);
  hipFree(c->dtab);
  hipFree(c->ktab);
  hipFree(c->red);
  hipFree(c->lphi);
  hipFree(c->radj);
  hipFree(c->dnu);
  if (c->host) hipHostFree(c->host);
  for (auto& p : c->ev_pending) {
    hipEventDestroy(p.second.first);
    hipEventDestroy(p.second.second);
  }
  for (auto e : c->ev_free) hipEventDestroy(e);
  delete c;
}

template <typename P>
int dalloc(P** p, size_t bytes, const char* what)
{
  hipError_t e = hipMalloc((void**)p, bytes ? bytes : 16);
  if (e != hipSuccess) {
    *p = nullptr;
    hipGetLastError();
    return fail(VP_ENOMEM, "hipMalloc(%s, %zu bytes): %s", what, bytes, hipGetErrorString(e));
  }
  return VP_OK;
}

long long prod3(const int m[3]) { return (long long)m[0] * m[1] * m[2]; }

hipEvent_t take_event(vp_ctx* c)
{
  if (!c->ev_free.empty()) {
    hipEvent_t e = c->ev_free.back();
    c->ev_free.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

// Brackets one phase with events when profiling is on.
struct PhaseScope {
  vp_ctx* c;
  int phase;
  hipEvent_t a = nullptr, b = nullptr;
  PhaseScope(vp_ctx* c_, int p) : c(c_), phase(p)
  {
    if (!c->profiling) return;
    a = take_event(c);
    b = take_event(c);
    if (a) hipEventRecord(a, c->stream);
  }
  ~PhaseScope()
  {
    if (!c->profiling || !a || !b) return;
    hipEventRecord(b, c->stream);
    c->ev_pending.push_back({phase, {a, b}});
  }
};

// Fold finished event pairs into the totals (synchronises the stream).
int drain_events(vp_ctx* c)
{
  HIP_TRY(hipStreamSynchronize(c->stream));
  for (auto& p : c->ev_pending) {
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, p.second.first, p.second.second));
    c->phase_ms[p.first] += ms;
    c->phase_n[p.first] += 1;
    c->ev_free.push_back(p.second.first);
    c->ev_free.push_back(p.second.second);
  }
  c->ev_pending.clear();
  return VP_OK;
}

// potential (with ghosts) of the density held in rho_in
int poisson_from(vp_ctx* c, const double* rho_in, double* phi_out)
{
  if (c->small) {
    vp::SmallGravity q = c->sg;
    q.rho = rho_in;
    q.phi = phi_out;
    LAUNCH(c, vp::launch_gravity_small(q, c->stream));
    return VP_OK;
  }
  const bool iso = c->cfg.bc == VP_BC_ISOLATED;
  LAUNCH(c, vp::launch_load_rho(c->work, c->wg, rho_in, c->ng, c->stream));
  for (int ax = 0; ax < 3; ax++) LAUNCH(c, vp::launch_dft_axis(c->work, c->wg, ax, -1, c->tw[ax], c->stream));
  if (iso)
    LAUNCH(c, vp::launch_mul_spectrum(c->work, c->kspec, prod3(c->wg.m), c->stream));
  else
    LAUNCH(c, vp::launch_green_periodic(c->work, c->wg, c->cfg.G, c->s2, c->stream));
  for (int ax = 0; ax < 3; ax++) LAUNCH(c, vp::launch_dft_axis(c->work, c->wg, ax, +1, c->tw[ax], c->stream));
  LAUNCH(c, vp::launch_extract_phi(phi_out, c->ng, c->work, c->wg, 1.0 / (double)prod3(c->wg.m), c->stream));
  return VP_OK;
}

// density -> rho, Poisson -> phi (with ghosts)
int potential_into(vp_ctx* c, double* phi_out)
{
  LAUNCH(c, vp::launch_density(c->f, c->cfg.dtype, c->rho, c->np, c->nv3,
                               c->dv[0] * c->dv[1] * c->dv[2], c->stream));
  return poisson_from(c, c->rho, phi_out);
}

// acceleration of the density held in c->rho
int accel_from_rho(vp_ctx* c)
{
  if (c->small) {
    vp::SmallGravity q = c->sg;
    q.rho = c->rho;
    q.accel = c->accel;
    LAUNCH(c, vp::launch_gravity_small(q, c->stream));
    return VP_OK;
  }
  int r = poisson_from(c, c->rho, c->phi);
  if (r != VP_OK) return r;
  LAUNCH(c, vp::launch_gradient(c->accel, c->phi, c->ng, c->dx[0], c->dx[1], c->dx[2], c->stream));
  return VP_OK;
}

int compute_accel(vp_ctx* c)
{
  PhaseScope scope(c, 6);
  LAUNCH(c, vp::launch_density(c->f, c->cfg.dtype, c->rho, c->np, c->nv3,
                               c->dv[0] * c->dv[1] * c->dv[2], c->stream));
  return accel_from_rho(c);
}

vp::SweepArgs sweep_args(vp_ctx* c, int axis, double tau)
{
  const auto& k = c->cfg;
  long long d[6] = {k.n[0], k.n[1], k.n[2], k.nv[0], k.nv[1], k.nv[2]};
  vp::SweepArgs a{};
  a.f = c->f;
  a.n = (int)d[axis];
  a.inner = 1;
  for (int q = 5; q > axis; q--) a.inner *= d[q];
  a.outer = 1;
  for (int q = 0; q < axis; q++) a.outer *= d[q];
  a.nlines = a.outer * a.inner;
  if (axis >= 3) {
    const int l = axis - 3;
    a.velocity = 1;
    a.periodic = 0;
    a.accel = c->accel + (long long)l * c->np;
    a.scale = tau / c->dv[l];
    a.sp_div = 1;
    for (int q = 3; q < axis; q++) a.sp_div *= d[q];
    a.j_div = 1;
    a.j_mod = 1;
  } else {
    a.velocity = 0;
    a.periodic = (k.bc == VP_BC_PERIODIC) ? 1 : 0;
    a.scale = tau / c->dx[axis];
    a.j_div = 1;
    for (int q = 5; q > axis + 3; q--) a.j_div *= d[q];
    a.j_mod = d[axis + 3];
    a.vmin = k.vmin[axis];
    a.dv = c->dv[axis];
    a.sp_div = 1;
  }
  return a;
}

int sweep(vp_ctx* c, int axis, double tau)
{
  const vp::SweepArgs a = sweep_args(c, axis, tau);
  PhaseScope scope(c, axis);
  LAUNCH(c, vp::launch_sweep(a, c->cfg.dtype, c->stream));
  return VP_OK;
}

// T_axis(tau) of the array at src, result written to dst (same layout, another array)
int sweep_to(vp_ctx* c, int axis, double tau, const void* src, void* dst)
{
  vp::SweepArgs a = sweep_args(c, axis, tau);
  a.f = const_cast<void*>(src);
  a.out = dst;
  PhaseScope scope(c, axis);
  LAUNCH(c, vp::launch_sweep(a, c->cfg.dtype, c->stream));
  return VP_OK;
}

// True when the x sweep can leave per-workgroup density sums: every
// workgroup's 256 lines lie in one spatial (y, z) column.
bool x_sweep_sums(vp_ctx* c)
{
  const vp::SweepArgs a = sweep_args(c, 0, 1.0);
  return c->nv3 % 256 == 0 && vp::sweep_part_supported(a, c->cfg.dtype);
}

// room for one value per line of a sweep (c->dnu)
int line_adjoints(vp_ctx* c, long long nlines)
{
  if (nlines <= c->dnu_len) return VP_OK;
  hipFree(c->dnu);
  c->dnu = nullptr;
  c->dnu_len = 0;
  int r = dalloc(&c->dnu, sizeof(double) * nlines, "line adjoints");
  if (r) return r;
  c->dnu_len = nlines;
  return VP_OK;
}

// lam <- J^T lam of T_axis(tau) at forward input fin; velocity axes add the
// acceleration adjoint to lam_a (if not null).
int sweep_adjoint(vp_ctx* c, int axis, double tau, const void* fin, void* lam, double* lam_a,
                  const double* rho_adj = nullptr)
{
  vp::SweepArgs a = sweep_args(c, axis, tau);
  if (rho_adj) {   // lam += dv^3 rho_adj(spatial cell) first: fused into the loads where supported
    const double dv3 = c->dv[0] * c->dv[1] * c->dv[2];
    a.addend = rho_adj;
    a.add_coef = dv3;
    a.add_stride = a.inner / c->nv3;
    a.add_div = c->nv3;
    if (axis >= 3 || a.inner % c->nv3 != 0 || !vp::adjoint_addend_supported(a)) {
      a.addend = nullptr;
      PhaseScope scope(c, 11);
      LAUNCH(c, vp::launch_broadcast_add(lam, c->cfg.dtype, rho_adj, c->np, c->nv3, dv3, c->stream));
    }
  }
  const bool want = axis >= 3 && lam_a;
  int r;
  if (want && (r = line_adjoints(c, a.nlines))) return r;
  PhaseScope scope(c, 10);
  LAUNCH(c, vp::launch_sweep_adjoint(a, c->cfg.dtype, fin, lam, want ? c->dnu : nullptr, c->stream));
  if (want) {
    const int l = axis - 3;
    LAUNCH(c, vp::launch_reduce_lines(lam_a + (long long)l * c->np, c->dnu, c->np, a.nlines / c->np,
                                      tau / c->dv[l], c->stream));
  }
  return VP_OK;
}

// lam <- adjoint of the half kick T_vz T_vy T_vx (tau) at forward input fin,
// with c->accel, in one pass; lam_a[l] gains the acceleration adjoint
int kick_adjoint(vp_ctx* c, double tau, const void* fin, void* lam, double* lam_a)
{
  vp::KickAdjArgs a{};
  a.fin = fin;
  a.lam = lam;
  a.np = c->np;
  for (int l = 0; l < 3; l++) {
    a.accel[l] = c->accel + (long long)l * c->np;
    a.scale[l] = tau / c->dv[l];
    a.lam_a[l] = lam_a ? lam_a + (long long)l * c->np : nullptr;
  }
  const int nv[3] = {c->cfg.nv[0], c->cfg.nv[1], c->cfg.nv[2]};
  PhaseScope scope(c, 13);
  LAUNCH(c, vp::launch_kick_adjoint(a, c->cfg.dtype, nv, c->stream));
  return VP_OK;
}

// the fields of density_adjoint
int density_adjoint_fields(vp_ctx* c)
{
  const long long ext = (long long)(c->cfg.n[0] + 2) * (c->cfg.n[1] + 2) * (c->cfg.n[2] + 2);
  int r;
  if (!c->small && !c->lphi && (r = dalloc(&c->lphi, sizeof(double) * ext, "potential adjoint"))) return r;
  if (!c->radj && (r = dalloc(&c->radj, sizeof(double) * c->np, "density adjoint"))) return r;
  return VP_OK;
}

// c->radj = G^T D^T lam_a: transpose of potential -> acceleration, per spatial
// cell (the density adjoint; lam then gains dv^3 times it)
int density_adjoint(vp_ctx* c, const double* lam_a)
{
  int r = density_adjoint_fields(c);
  if (r) return r;
  PhaseScope scope(c, 11);
  if (c->small) {
    vp::SmallGravity q = c->sg;
    q.lam_a = lam_a;
    q.radj = c->radj;
    LAUNCH(c, vp::launch_gravity_small(q, c->stream));
    return VP_OK;
  }
  LAUNCH(c, vp::launch_gradient_adj(c->lphi, lam_a, c->ng, c->dx[0], c->dx[1], c->dx[2], c->stream));
  if (c->cfg.bc == VP_BC_ISOLATED) {
    LAUNCH(c, vp::launch_load_ext(c->work, c->wg, c->lphi, c->ng, c->stream));
    for (int ax = 0; ax < 3; ax++) LAUNCH(c, vp::launch_dft_axis(c->work, c->wg, ax, -1, c->tw[ax], c->stream));
    LAUNCH(c, vp::launch_mul_spectrum(c->work, c->kspec, prod3(c->wg.m), c->stream));
    for (int ax = 0; ax < 3; ax++) LAUNCH(c, vp::launch_dft_axis(c->work, c->wg, ax, +1, c->tw[ax], c->stream));
    LAUNCH(c, vp::launch_extract_interior(c->radj, c->work, c->wg, c->ng, 1.0 / (double)prod3(c->wg.m), c->stream));
  } else {
    LAUNCH(c, vp::launch_fold_periodic(c->radj, c->lphi, c->ng, c->stream));
    LAUNCH(c, vp::launch_load_rho(c->work, c->wg, c->radj, c->ng, c->stream));
    for (int ax = 0; ax < 3; ax++) LAUNCH(c, vp::launch_dft_axis(c->work, c->wg, ax, -1, c->tw[ax], c->stream));
    LAUNCH(c, vp::launch_green_periodic(c->work, c->wg, c->cfg.G, c->s2, c->stream));
    for (int ax = 0; ax < 3; ax++) LAUNCH(c, vp::launch_dft_axis(c->work, c->wg, ax, +1, c->tw[ax], c->stream));
    LAUNCH(c, vp::launch_extract_interior(c->radj, c->work, c->wg, c->ng, 1.0 / (double)prod3(c->wg.m), c->stream));
  }
  return VP_OK;
}

// lam += dv^3 G^T D^T lam_a: transpose of density -> potential -> acceleration
int accel_adjoint(vp_ctx* c, const double* lam_a, void* lam)
{
  int r = density_adjoint(c, lam_a);
  if (r) return r;
  PhaseScope scope(c, 11);
  LAUNCH(c, vp::launch_broadcast_add(lam, c->cfg.dtype, c->radj, c->np, c->nv3, c->dv[0] * c->dv[1] * c->dv[2],
                                     c->stream));
  return VP_OK;
}

vp::KickArgs kick_args(vp_ctx* c, double tau, int reps, const void* src, void* dst)
{
  vp::KickArgs a{};
  a.tab = c->ktab;
  a.f = const_cast<void*>(src);
  a.out = dst;
  a.np = c->np;
  a.reps = reps;
  for (int l = 0; l < 3; l++) {
    a.a[l] = c->accel + (long long)l * c->np;
    a.scale[l] = tau / c->dv[l];
  }
  return a;
}

// True when the velocity block of a spatial cell has a one-pass half kick: in
// LDS (cubes with a kernel of their own, and other shapes where it pays) or,
// for FP64 32^3, in registers with one line per lane.
bool kick_one_pass(vp_ctx* c)
{
  const int* nv = c->cfg.nv;
  return vp::kick_fused_supported(c->cfg.dtype, nv) || vp::kick_lines_supported(c->cfg.dtype, nv) ||
         vp::kick_box_supported(c->cfg.dtype, nv, c->np);
}

// reps (1 or 2) half kicks in one pass, from src (over it, or to dst)
int kick_pass(vp_ctx* c, double tau, int reps, const void* src, void* dst)
{
  const int* nv = c->cfg.nv;
  const int dt = c->cfg.dtype;
  const vp::KickArgs a = kick_args(c, tau, reps, src, dst);
  PhaseScope scope(c, reps == 2 ? 8 : 7);
  if (vp::kick_fused_supported(dt, nv))
    LAUNCH(c, vp::launch_kick(a, dt, nv, c->stream));
  else if (vp::kick_lines_supported(dt, nv))
    LAUNCH(c, vp::launch_kick_lines(a, dt, nv, c->stream));
  else
    LAUNCH(c, vp::launch_kick_box(a, dt, nv, c->stream));
  return VP_OK;
}

// T_vz T_vy T_vx(tau), reps times in a row with the same acceleration: one
// pass over f when the velocity block fits on chip.
int kick_n(vp_ctx* c, double tau, int reps)
{
  if (kick_one_pass(c)) return kick_pass(c, tau, reps, c->f, nullptr);
  const int nv[3] = {c->cfg.nv[0], c->cfg.nv[1], c->cfg.nv[2]};
  int r;
  if (vp::kick_planes_supported(c->cfg.dtype, nv)) {   // T_vx | T_vy T_vz per half kick
    const vp::KickArgs a = kick_args(c, tau, 1, c->f, nullptr);
    if (reps == 2 && vp::kick_slices_supported(c->cfg.dtype, nv)) {   // T_vx T_vy | T_vz T_vx | T_vy T_vz
      for (int pass = 0; pass < 3; pass++) {
        PhaseScope scope(c, 12);
        LAUNCH(c, vp::launch_kick_slices(a, c->cfg.dtype, nv, pass, c->stream));
      }
      return VP_OK;
    }
    for (int i = 0; i < reps; i++) {
      if ((r = sweep(c, 3, tau))) return r;
      PhaseScope scope(c, 12);
      LAUNCH(c, vp::launch_kick_planes(a, c->cfg.dtype, nv, c->stream));
    }
    return VP_OK;
  }
  for (int i = 0; i < reps; i++)
    if ((r = sweep(c, 3, tau)) || (r = sweep(c, 4, tau)) || (r = sweep(c, 5, tau))) return r;
  return VP_OK;
}

int kick(vp_ctx* c, double tau) { return kick_n(c, tau, 1); }

// T_x T_y T_z(tau) over chunks of velocity cells (box.h), from src (over it, or
// to dst); with sums the chunks' density sums go to c->bsum
int drift_box(vp_ctx* c, double tau, bool sums, const void* src, void* dst)
{
  const auto& k = c->cfg;
  vp::DriftBoxArgs a{};
  a.f = src;
  a.out = dst;
  a.nv3 = c->nv3;
  a.periodic = (k.bc == VP_BC_PERIODIC) ? 1 : 0;
  a.part = sums ? c->bsum : nullptr;
  for (int l = 0; l < 3; l++) {
    a.n[l] = k.n[l];
    a.nv[l] = k.nv[l];
    a.vmin[l] = k.vmin[l];
    a.dv[l] = c->dv[l];
    a.scale[l] = tau / c->dx[l];
  }
  PhaseScope scope(c, 9);
  LAUNCH(c, vp::launch_drift_box(a, k.dtype, c->stream));
  return VP_OK;
}

// T_y T_z(tau) in one pass (drift_yz_supported), from src (over it, or to dst)
int drift_yz(vp_ctx* c, double tau, const void* src, void* dst)
{
  const auto& k = c->cfg;
  vp::DriftArgs a{};
  a.f = const_cast<void*>(src);
  a.out = dst;
  a.nx = k.n[0];
  a.nv3 = c->nv3;
  a.ny = k.n[1];
  a.nz = k.n[2];
  a.nvy = k.nv[1];
  a.nvz = k.nv[2];
  a.periodic = (k.bc == VP_BC_PERIODIC) ? 1 : 0;
  a.vmin_y = k.vmin[1];
  a.dv_y = c->dv[1];
  a.scale_y = tau / c->dx[1];
  a.vmin_z = k.vmin[2];
  a.dv_z = c->dv[2];
  a.scale_z = tau / c->dx[2];
  a.tab = c->dtab;
  PhaseScope scope(c, 9);
  LAUNCH(c, vp::launch_drift_yz(a, k.dtype, c->stream));
  return VP_OK;
}

// T_b T_a(tau) of two position axes in one pass (drift_pair_supported); with
// sums (b = 0, a = 1) the pass leaves density sums (c->xsum)
int drift_pair(vp_ctx* c, int a, int b, double tau, bool sums)
{
  const auto& k = c->cfg;
  const int o = 3 - a - b;
  const long long st[3] = {(long long)k.n[1] * k.n[2] * c->nv3, k.n[2] * c->nv3, c->nv3};
  auto axis = [&](int l) {
    vp::DriftPairAxis x{};
    x.j_div = l == 0 ? (long long)k.nv[1] * k.nv[2] : (l == 1 ? k.nv[2] : 1);
    x.j_mod = k.nv[l];
    x.vmin = k.vmin[l];
    x.dv = c->dv[l];
    x.scale = tau / c->dx[l];
    return x;
  };
  vp::DriftPairArgs q{};
  q.f = c->f;
  q.nv3 = c->nv3;
  q.sa = st[a];
  q.sb = st[b];
  q.so = st[o];
  q.nouter = k.n[o];
  q.periodic = (k.bc == VP_BC_PERIODIC) ? 1 : 0;
  q.a = axis(a);
  q.b = axis(b);
  q.part = sums ? c->xsum : nullptr;
  PhaseScope scope(c, b == 0 ? 0 : 9);
  LAUNCH(c, vp::launch_drift_pair(q, k.dtype, k.n[a], k.n[b], c->stream));
  return VP_OK;
}

// T_x T_y T_z(tau): in one pass when the whole spatial grid fits on chip with a
// chunk of velocity cells; else two axes in one pass when their plane does.
// With sums the last pass leaves density sums (c->bsum, c->xsum).
int drift(vp_ctx* c, double tau, bool x_sums = false)
{
  int r;
  const auto& k = c->cfg;
  if (c->box3) return drift_box(c, tau, x_sums, c->f, nullptr);
  if (c->pair == 1) {
    if ((r = sweep(c, 2, tau))) return r;
    return drift_pair(c, 1, 0, tau, x_sums);
  }
  if (c->pair == 2) {
    if ((r = drift_pair(c, 2, 1, tau, false))) return r;
  } else if (vp::drift_yz_supported(k.dtype, k.n[1], k.n[2], c->nv3, k.nv[2])) {
    if ((r = drift_yz(c, tau, c->f, nullptr))) return r;
  } else if ((r = sweep(c, 2, tau)) || (r = sweep(c, 1, tau))) {
    return r;
  }
  if (!x_sums) return sweep(c, 0, tau);
  vp::SweepArgs a = sweep_args(c, 0, tau);
  a.part = c->xsum;
  PhaseScope scope(c, 0);
  LAUNCH(c, vp::launch_sweep(a, c->cfg.dtype, c->stream));
  return VP_OK;
}

// Two position axes that share a pass (drift_pair) save one of the drift's
// passes over f: 10 to 29 % of a step (2 steps of 24 x 12 x 48 with 32^3 blocks FP32
// 6.41 -> 5.24 ms, 16 x 16 x 64 7.91 -> 6.12, 48 x 48 x 12 with 24 x 24 x 32 FP64 18.7 ->
// 15.5). Its tiles are serial, so the sweeps stay where workgroups, or wavefronts of
// an array that the last-level cache holds, are few: 288 workgroups over 256 CUs took
// 0.75 to 1.36 of the sweeps' time, 48 x 12 planes of six-cell vz rows 1.17 at 576. Of
// 2900 shapes of up to 2500 workgroups, those that the rule takes have 0.8 of the sweeps'
// time on average and 1.08 at most. The short z lines of FP32 planes of 6 or 12 x 48 cells stay
// too where their vz rows are shorter than 32 cells: a wavefront reads runs of half
// a vz row, as opposite velocities read their lines from opposite ends, and tiles
// of 72 KiB and six wavefronts, two to a CU, hide nothing of runs under 64 bytes (122
// shapes: 0.85 to 1.21 of the sweeps' time, 1.00 on average; 75 of longer rows 0.72 to
// 0.98, and 0.82). Square planes with
// a kernel of their own (drift_yz) keep it (16^3 x 16^3 FP32: 231 us, 251 with
// the pair), except the FP32 64-cell plane, whose half-line chunks run at half
// the copy rate (4 x 64 x 64 with 32^3: 7.36 -> 6.46 ms, with 16^3 the same).
// Where both pairs will do, that of the smaller plane goes together (8 x 48 x 4
// with 32^3 FP64: z and y 1.34 ms, y and x 1.47), or z and y where they are the
// same, which leaves the sums to the x sweep.
int pair_plan(const vp_ctx* c)
{
  const auto& k = c->cfg;
  const long long chunks = c->nv3 / 256;
  const long long bytes = c->np * c->nv3 * (k.dtype == VP_F32 ? 4 : 8);
  auto thin = [&](int a, int b) {
    return k.dtype == VP_F32 && a == 2 && k.nv[2] < 32 && k.n[2] < k.n[1] && vp::drift_pair_tile(k.dtype, k.n[2], k.n[1]) > 64 * 1024 &&
           vp::drift_pair_waves(k.dtype, k.n[2], k.n[1], 1, 256) <= 6;
  };
  auto pays = [&](int a, int b, int o) {
    const long long groups = k.n[o] * chunks;
    return vp::drift_pair_supported(k.dtype, k.n[a], k.n[b], c->nv3) && groups >= 320 &&
           (bytes >= (48LL << 20) || vp::drift_pair_waves(k.dtype, k.n[a], k.n[b], k.n[o], c->nv3) > 5 * 256) &&
           (k.n[a] * k.n[b] <= 320 || k.nv[2] >= 8 || groups > 600) && !thin(a, b);
  };
  const bool yx = c->xsum && pays(1, 0, 2);
  if (vp::drift_yz_supported(k.dtype, k.n[1], k.n[2], c->nv3, k.nv[2])) return yx && k.n[1] == 64 ? 1 : 0;
  const bool zy = pays(2, 1, 0);
  if (yx && zy) return k.n[0] < k.n[2] ? 1 : 2;
  return yx ? 1 : (zy ? 2 : 0);
}

// drift, then the acceleration of the drifted f (one step's middle): the x
// sweep sums its new values per workgroup when it can, which replaces the
// density pass over f by a reduction of those sums
int drift_accel(vp_ctx* c, double tau)
{
  if (c->box3) {
    int r = drift(c, tau, /*x_sums=*/true);
    if (r) return r;
    PhaseScope scope(c, 6);
    const long long nchunk = (c->nv3 + c->box3 - 1) / c->box3;
    vp::SmallGravity q = c->sg;
    q.part = c->bsum;
    q.nchunk = nchunk;
    q.accel = c->accel;
    if (c->small && vp::gravity_small_sums(q)) {
      LAUNCH(c, vp::launch_gravity_small(q, c->stream));
      return VP_OK;
    }
    LAUNCH(c, vp::launch_box_density(c->rho, c->bsum, c->np, nchunk, c->dv[0] * c->dv[1] * c->dv[2], c->stream));
    return accel_from_rho(c);
  }
  if (!c->xsum) {
    int r = drift(c, tau);
    return r ? r : compute_accel(c);
  }
  int r = drift(c, tau, /*x_sums=*/true);
  if (r) return r;
  PhaseScope scope(c, 6);
  vp::SmallGravity q = c->sg;
  q.part = c->xsum;
  q.xsums = 1;
  q.nchunk = c->nv3 / 256;
  q.accel = c->accel;
  if (c->small && vp::gravity_small_sums(q)) {
    LAUNCH(c, vp::launch_gravity_small(q, c->stream));
    return VP_OK;
  }
  const long long nyz = (long long)c->cfg.n[1] * c->cfg.n[2];
  LAUNCH(c, vp::launch_density_from_parts(c->rho, c->xsum, nyz, c->nv3 / 256, c->cfg.n[0],
                                          c->dv[0] * c->dv[1] * c->dv[2], c->stream));
  return accel_from_rho(c);
}

int check_ctx(vp_ctx* c)
{
  if (!c) return fail(VP_EINVAL, "null context");
  return VP_OK;
}

}  // namespace

extern "C" {

int vp_config_size(void) { return (int)sizeof(vp_config); }

int vp_config_validate(const vp_config* cfg)
{
  g_err.clear();
  if (!cfg) return fail(VP_EINVAL, "null config");
  for (int l = 0; l < 3; l++) {
    if (cfg->n[l] < 1 || cfg->nv[l] < 1) return fail(VP_EINVAL, "axis %d: cell counts must be >= 1", l);
    if (!vp::sweep_length_supported(cfg->n[l]))
      return fail(VP_EUNSUPPORTED, "n[%d] = %d is not a supported line length", l, cfg->n[l]);
    if (!vp::sweep_length_supported(cfg->nv[l]))
      return fail(VP_EUNSUPPORTED, "nv[%d] = %d is not a supported line length", l, cfg->nv[l]);
    if (!(std::isfinite(cfg->L[l]) && cfg->L[l] > 0)) return fail(VP_EINVAL, "L[%d] must be finite and > 0", l);
    if (!(std::isfinite(cfg->vmin[l]) && std::isfinite(cfg->vmax[l]) && cfg->vmax[l] > cfg->vmin[l]))
      return fail(VP_EINVAL, "velocity range of axis %d must be finite with vmax > vmin", l);
  }
  if (!(std::isfinite(cfg->G) && cfg->G >= 0)) return fail(VP_EINVAL, "G must be finite and >= 0");
  if (cfg->bc != VP_BC_PERIODIC && cfg->bc != VP_BC_ISOLATED) return fail(VP_EINVAL, "unknown bc %d", cfg->bc);
  if (cfg->dtype != VP_F32 && cfg->dtype != VP_F64) return fail(VP_EINVAL, "unknown dtype %d", cfg->dtype);
  if (cfg->flags != 0 || cfg->reserved != 0) return fail(VP_EINVAL, "flags and reserved must be 0");
  const double np = (double)cfg->n[0] * cfg->n[1] * cfg->n[2];
  const double nv = (double)cfg->nv[0] * cfg->nv[1] * cfg->nv[2];
  if (np * nv > 9.0e18 / 8) return fail(VP_EINVAL, "grid too large");
  if (np > 2.0e9 || nv > 2.0e9) return fail(VP_EINVAL, "spatial or velocity grid too large");
  if (cfg->bc == VP_BC_ISOLATED) {
    const double d0 = cfg->L[0] / cfg->n[0], d1 = cfg->L[1] / cfg->n[1], d2 = cfg->L[2] / cfg->n[2];
    if (std::fabs(d0 - d1) > 1e-12 * d0 || std::fabs(d0 - d2) > 1e-12 * d0)
      return fail(VP_EUNSUPPORTED, "isolated Poisson needs equal spacings");
  }
  return VP_OK;
}

int vp_init(const vp_config* cfg, void* f_dev, void* hip_stream, vp_ctx** out)
{
  g_err.clear();
  if (!out) return fail(VP_EINVAL, "null output pointer");
  *out = nullptr;
  int r = vp_config_validate(cfg);
  if (r != VP_OK) return r;
  if (!f_dev) return fail(VP_EINVAL, "null f pointer");
  if (reinterpret_cast<uintptr_t>(f_dev) % 16 != 0) return fail(VP_EINVAL, "f must be 16-byte aligned");
  vp_ctx* c = new (std::nothrow) vp_ctx;
  if (!c) return fail(VP_ENOMEM, "host allocation failed");
  c->cfg = *cfg;
  c->f = f_dev;
  c->stream = (hipStream_t)hip_stream;
  const hipError_t de = hipGetDevice(&c->device);
  if (de != hipSuccess) {
    delete c;
    return fail(VP_EHIP, "device query: %s", hipGetErrorString(de));
  }
  if ((r = scratch_address(c->device, &c->scratch))) {
    delete c;
    return r;
  }
  for (int l = 0; l < 3; l++) {
    c->dx[l] = cfg->L[l] / cfg->n[l];
    c->dv[l] = (cfg->vmax[l] - cfg->vmin[l]) / cfg->nv[l];
    c->ng.m[l] = cfg->n[l];
    c->wg.m[l] = cfg->bc == VP_BC_ISOLATED ? 2 * cfg->n[l] : cfg->n[l];
  }
  c->np = prod3(c->ng.m);
  c->nv3 = (long long)cfg->nv[0] * cfg->nv[1] * cfg->nv[2];
  const long long ext = (long long)(cfg->n[0] + 2) * (cfg->n[1] + 2) * (cfg->n[2] + 2);
  const long long wn = prod3(c->wg.m);
  if ((r = dalloc(&c->rho, sizeof(double) * c->np, "rho")) ||
      (r = dalloc(&c->phi, sizeof(double) * ext, "phi")) ||
      (r = dalloc(&c->accel, sizeof(double) * 3 * c->np, "accel")) ||
      (r = dalloc(&c->work, sizeof(double2) * wn, "transform work")) ||
      (r = dalloc(&c->part, sizeof(double) * 2 * c->np, "partials")) ||
      (r = dalloc(&c->red, sizeof(double) * vp::RED_DOUBLES, "reduction"))) {
    release(c);
    return r;
  }
  for (int ax = 0; ax < 3; ax++) {
    if ((r = dalloc(&c->tw[ax], sizeof(double2) * c->wg.m[ax], "twiddles")) ||
        (r = dalloc(&c->s2[ax], sizeof(double) * c->wg.m[ax], "Green's function"))) {
      release(c);
      return r;
    }
  }
  c->small = vp::gravity_small_supported(c->wg);
  if ((c->small || cfg->bc == VP_BC_ISOLATED) && (r = dalloc(&c->kspec, sizeof(double2) * wn, "green spectrum"))) {
    release(c);
    return r;
  }
  c->box3 = vp::drift_box_cells(cfg->dtype, cfg->n, c->nv3);
  if (c->box3) {
    const long long nsum = (c->nv3 + c->box3 - 1) / c->box3 * c->np;
    if ((r = dalloc(&c->bsum, sizeof(double) * nsum, "drift sums"))) {
      release(c);
      return r;
    }
  } else if (x_sweep_sums(c)) {   // n_x sums per 256 lines of the x sweep
    const long long nsum = (long long)cfg->n[1] * cfg->n[2] * (c->nv3 / 256) * cfg->n[0];
    if ((r = dalloc(&c->xsum, sizeof(double) * nsum, "x sweep sums"))) {
      release(c);
      return r;
    }
  }
  c->pair = c->box3 ? 0 : pair_plan(c);
  {
    const int nv[3] = {cfg->nv[0], cfg->nv[1], cfg->nv[2]};
    if (vp::kick_wants_table(cfg->dtype, nv, c->np) &&
        (r = dalloc(&c->ktab, vp::kick_table_bytes(cfg->dtype, c->np), "kick coefficients"))) {
      release(c);
      return r;
    }
  }
  if (vp::drift_yz_supported(cfg->dtype, cfg->n[1], cfg->n[2], c->nv3, cfg->nv[2]) &&
      (r = dalloc(&c->dtab, vp::drift_table_bytes(cfg->dtype, c->nv3), "drift coefficients"))) {
    release(c);
    return r;
  }
  hipError_t he = hipHostMalloc((void**)&c->host, sizeof(double) * 8, hipHostMallocDefault);
  if (he != hipSuccess) {
    c->host = nullptr;
    release(c);
    return fail(VP_ENOMEM, "hipHostMalloc: %s", hipGetErrorString(he));
  }
  for (int ax = 0; ax < 3; ax++) {
    if ((r = check_launch(c, vp::launch_twiddles(c->tw[ax], c->s2[ax], c->wg.m[ax], c->dx[ax], c->stream), "twiddles"))) {
      release(c);
      return r;
    }
  }
  if (c->small) {
    vp::SmallGravity& q = c->sg;
    q.n = c->ng;
    q.g = c->wg;
    q.isolated = cfg->bc == VP_BC_ISOLATED;
    for (int l = 0; l < 3; l++) {
      q.d[l] = c->dx[l];
      q.tw[l] = c->tw[l];
    }
    q.kspec = c->kspec;
    q.dv3 = c->dv[0] * c->dv[1] * c->dv[2];
    vp::gravity_small_plan(q);
    if (cfg->bc == VP_BC_PERIODIC &&
        (r = check_launch(c, vp::launch_green_table(c->kspec, c->wg, cfg->G, c->s2, c->stream), "green"))) {
      release(c);
      return r;
    }
  }
  if (cfg->bc == VP_BC_ISOLATED) {
    const double self = -cfg->G * vp_cell_self_integral(c->dx[0], c->dx[1], c->dx[2]);
    r = check_launch(c, vp::launch_green_isolated(c->kspec, c->wg, cfg->G, c->dx[0], c->dx[1], c->dx[2], self,
                                                  c->stream), "green");
    for (int ax = 0; ax < 3 && r == VP_OK; ax++)
      r = check_launch(c, vp::launch_dft_axis(c->kspec, c->wg, ax, -1, c->tw[ax], c->stream), "green dft");
    if (r != VP_OK) {
      release(c);
      return r;
    }
  }
  r = compute_accel(c);
  if (r != VP_OK) {
    hipStreamSynchronize(c->stream);
    release(c);
    return r;
  }
  *out = c;
  return VP_OK;
}

int vp_sweep(vp_ctx* c, int32_t axis, double tau)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (axis < 0 || axis > 5) return fail(VP_EINVAL, "axis must be 0..5");
  if (!std::isfinite(tau)) return fail(VP_EINVAL, "tau must be finite");
  return sweep(c, axis, tau);
}

int vp_step(vp_ctx* c, double dt)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (!(std::isfinite(dt) && dt > 0)) return fail(VP_EINVAL, "dt must be finite and > 0");
  const double h = 0.5 * dt;
  if ((r = kick(c, h)) || (r = drift_accel(c, dt)) || (r = kick(c, h))) return r;
  return VP_OK;
}

int vp_run(vp_ctx* c, int32_t nsteps, double dt)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (nsteps < 0) return fail(VP_EINVAL, "nsteps must be >= 0");
  if (!(std::isfinite(dt) && dt > 0)) return fail(VP_EINVAL, "dt must be finite and > 0");
  if (nsteps == 0) return VP_OK;
  // the closing half kick of a step and the opening half kick of the next use
  // the same acceleration and run back to back: one pass does both
  const double h = 0.5 * dt;
  if ((r = kick(c, h))) return r;
  for (int i = 0; i < nsteps; i++) {
    if ((r = drift_accel(c, dt))) return r;
    if ((r = kick_n(c, h, i + 1 < nsteps ? 2 : 1))) return r;
  }
  return VP_OK;
}

int vp_kick(vp_ctx* c, double tau)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (!std::isfinite(tau)) return fail(VP_EINVAL, "tau must be finite");
  return kick(c, tau);
}

int vp_drift(vp_ctx* c, double tau)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (!std::isfinite(tau)) return fail(VP_EINVAL, "tau must be finite");
  return drift(c, tau);
}

int vp_accel(vp_ctx* c)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  return compute_accel(c);
}

int vp_get_accel(vp_ctx* c, double* a_dev)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (!a_dev) return fail(VP_EINVAL, "null pointer");
  HIP_TRY(hipMemcpyAsync(a_dev, c->accel, sizeof(double) * 3 * c->np, hipMemcpyDeviceToDevice, c->stream));
  return VP_OK;
}

int vp_set_accel(vp_ctx* c, const double* a_dev)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (!a_dev) return fail(VP_EINVAL, "null pointer");
  HIP_TRY(hipMemcpyAsync(c->accel, a_dev, sizeof(double) * 3 * c->np, hipMemcpyDeviceToDevice, c->stream));
  return VP_OK;
}

int vp_density(vp_ctx* c, double* rho_dev)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (!rho_dev) return fail(VP_EINVAL, "null pointer");
  LAUNCH(c, vp::launch_density(c->f, c->cfg.dtype, rho_dev, c->np, c->nv3, c->dv[0] * c->dv[1] * c->dv[2],
                               c->stream));
  return VP_OK;
}

int vp_moment(vp_ctx* c, const void* a_dev, const double* w_dev, double scale, double* out_dev)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (!a_dev || !w_dev || !out_dev) return fail(VP_EINVAL, "null pointer");
  if (!std::isfinite(scale)) return fail(VP_EINVAL, "scale must be finite");
  LAUNCH(c, vp::launch_weighted_moment(a_dev, c->cfg.dtype, w_dev, out_dev, c->np, c->nv3, scale, c->stream));
  return VP_OK;
}

int vp_potential(vp_ctx* c, double* phi_dev)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (!phi_dev) return fail(VP_EINVAL, "null pointer");
  return potential_into(c, phi_dev);
}

int vp_energy(vp_ctx* c, double out_host[4])
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (!out_host) return fail(VP_EINVAL, "null pointer");
  vp::VelGrid vg{};
  for (int l = 0; l < 3; l++) {
    vg.nv[l] = c->cfg.nv[l];
    vg.vmin[l] = c->cfg.vmin[l];
    vg.dv[l] = c->dv[l];
  }
  LAUNCH(c, vp::launch_energy_partials(c->f, c->cfg.dtype, c->part, c->rho, c->np, vg, c->stream));
  if ((r = poisson_from(c, c->rho, c->phi))) return r;
  LAUNCH(c, vp::launch_energy_final(c->red, c->part, c->rho, c->phi, c->ng, c->dx[0] * c->dx[1] * c->dx[2],
                                    c->dv[0] * c->dv[1] * c->dv[2], c->stream));
  HIP_TRY(hipMemcpyAsync(c->host, c->red, sizeof(double) * 4, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  for (int i = 0; i < 4; i++) out_host[i] = c->host[i];
  for (int i = 0; i < 4; i++)
    if (!std::isfinite(out_host[i])) return fail(VP_ENONFINITE, "diagnostic %d is not finite", i);
  return VP_OK;
}

int vp_dt(vp_ctx* c, double cfl, double* dt_host)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (!dt_host) return fail(VP_EINVAL, "null pointer");
  if (!(std::isfinite(cfl) && cfl > 0)) return fail(VP_EINVAL, "cfl must be finite and > 0");
  // the maximum goes straight to the pinned page that the host reads
  LAUNCH(c, vp::launch_accel_max(c->red, c->host, c->accel, c->np, 1.0 / c->dv[0], 1.0 / c->dv[1], 1.0 / c->dv[2],
                                 c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  double dtp = INFINITY;
  for (int l = 0; l < 3; l++) {
    const double vm = std::fmax(std::fabs(c->cfg.vmin[l]), std::fabs(c->cfg.vmax[l]));
    if (vm > 0) dtp = std::fmin(dtp, c->dx[l] / vm);
  }
  const double amax = c->host[0];
  const double dtv = amax > 0 ? 1.0 / amax : INFINITY;
  *dt_host = cfl * std::fmin(dtp, dtv);
  return VP_OK;
}

int vp_sweep_adjoint(vp_ctx* c, int32_t axis, double tau, const void* f_in_dev, void* lam_dev,
                     double* lam_accel_dev)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (axis < 0 || axis > 5) return fail(VP_EINVAL, "axis must be 0..5");
  if (!std::isfinite(tau)) return fail(VP_EINVAL, "tau must be finite");
  if (!f_in_dev || !lam_dev) return fail(VP_EINVAL, "null pointer");
  return sweep_adjoint(c, axis, tau, f_in_dev, lam_dev, lam_accel_dev);
}

int vp_kick_adjoint(vp_ctx* c, double tau, const void* f_in_dev, void* lam_dev, double* lam_accel_dev)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (!std::isfinite(tau)) return fail(VP_EINVAL, "tau must be finite");
  if (!f_in_dev || !lam_dev) return fail(VP_EINVAL, "null pointer");
  const int nv[3] = {c->cfg.nv[0], c->cfg.nv[1], c->cfg.nv[2]};
  // the grids of this entry point's contract (vp_grad uses the pass on more)
  const bool offered = c->cfg.dtype == VP_F32 ? nv[0] <= 24 : nv[0] == 8;
  if (!offered || !vp::kick_adjoint_supported(c->cfg.dtype, nv))
    return fail(VP_EUNSUPPORTED, "no one-pass reverse half kick for this velocity grid");
  return kick_adjoint(c, tau, f_in_dev, lam_dev, lam_accel_dev);
}

int vp_sweep_adjoint_noalloc(vp_ctx* c, int32_t axis, double tau, const void* f_in_dev, void* lam_dev,
                             double* lam_accel_dev)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (axis < 0 || axis > 5) return fail(VP_EINVAL, "axis must be 0..5");
  if (!std::isfinite(tau)) return fail(VP_EINVAL, "tau must be finite");
  if (!f_in_dev || !lam_dev) return fail(VP_EINVAL, "null pointer");
  const vp::SweepArgs a = sweep_args(c, axis, tau);
  const bool want = axis >= 3 && lam_accel_dev;
  if (want && a.nlines > VP_NOALLOC_MAX_LINES)
    return fail(VP_EINVAL, "velocity sweep of %lld lines exceeds the %d-line device scratch of the "
                           "allocation-free reverse sweep", a.nlines, VP_NOALLOC_MAX_LINES);
  if (want && !c->scratch) return fail(VP_EHIP, "device scratch address not resolved");
  // every line writes its own entry before the reduction reads it, so the
  // scratch needs no clearing; no phase timing here (it would create events)
  LAUNCH(c, vp::launch_sweep_adjoint(a, c->cfg.dtype, f_in_dev, lam_dev, want ? c->scratch : nullptr, c->stream));
  if (want) {
    const int l = axis - 3;
    LAUNCH(c, vp::launch_reduce_lines(lam_accel_dev + (long long)l * c->np, c->scratch, c->np, a.nlines / c->np,
                                      tau / c->dv[l], c->stream));
  }
  return VP_OK;
}

int vp_accel_adjoint(vp_ctx* c, const double* lam_accel_dev, void* lam_dev)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (!lam_accel_dev || !lam_dev) return fail(VP_EINVAL, "null pointer");
  return accel_adjoint(c, lam_accel_dev, lam_dev);
}

namespace {

constexpr size_t kGradSpare = size_t(1) << 30;   // device memory that vp_grad's optional array leaves free

struct GradWork {
  vp_ctx* c;
  std::vector<void*> bufs;
  std::vector<double*> dbufs;
  // the caller's state array and the context's acceleration, which stand in
  // for others during the call: put back however it ends
  void* user_f;
  double* user_accel;
  bool small;
  int pair;
  explicit GradWork(vp_ctx* c_) : c(c_), user_f(c_->f), user_accel(c_->accel), small(c_->small), pair(c_->pair) {}
  ~GradWork()
  {
    c->f = user_f;
    c->accel = user_accel;
    c->small = small;
    c->pair = pair;
    for (void* p : bufs) hipFree(p);
    for (double* p : dbufs) hipFree(p);
  }
  int f(void** p, size_t bytes)
  {
    int r = dalloc(p, bytes, "gradient work");
    if (!r) bufs.push_back(*p);
    return r;
  }
  int d(double** p, size_t bytes)
  {
    int r = dalloc(p, bytes, "gradient work");
    if (!r) dbufs.push_back(*p);
    return r;
  }
};

int copy_f(vp_ctx* c, void* dst, const void* src, size_t bytes)
{
  HIP_TRY(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, c->stream));
  return VP_OK;
}

// dst = T_vz T_vy T_vx(tau) src (dst may not alias src): one pass when the
// velocity block fits on chip (in LDS, or in registers for FP64 32^3), else a
// copy and the kick in place. c->f is left pointing at dst.
int kick_to(vp_ctx* c, double tau, const void* src, void* dst, size_t fbytes)
{
  if (kick_one_pass(c)) {
    c->f = dst;
    return kick_pass(c, tau, 1, src, dst);
  }
  int r = copy_f(c, dst, src, fbytes);
  if (r) return r;
  c->f = dst;
  return kick(c, tau);
}

// T_axis(tau) in place on the array at buf (left as c->f)
int sweep_on(vp_ctx* c, int axis, double tau, void* buf)
{
  c->f = buf;
  return sweep(c, axis, tau);
}

// dst = T_y T_z(tau) src (another array): one pass where the plane has one, else
// two sweeps. c->f is left pointing at dst.
int zy_to(vp_ctx* c, double tau, const void* src, void* dst)
{
  c->f = dst;
  if (vp::drift_yz_supported(c->cfg.dtype, c->cfg.n[1], c->cfg.n[2], c->nv3, c->cfg.nv[2]))
    return drift_yz(c, tau, src, dst);
  int r = sweep_to(c, 2, tau, src, dst);
  return r ? r : sweep(c, 1, tau);
}

// Reverse mode of nsteps steps of Eq. (17) with checkpoints; see vp.h.
//
// Device memory: every k-th state of the forward run (ceil(nsteps/k) copies of
// f), the other k-1 states of the segment being reversed, and three work arrays
// in which the inputs of a step's nine sweeps are regenerated from the step's
// start x0, in the order the reverse sweeps need them:
//   in3 = kick(x0) in b1, in5 = T_y T_z in3 in b2, in6 = T_x in5 in b3;
//   closing half kick (a_{n+1}):  one pass at in6 that rebuilds in7 = T_vx in6
//                                 and in8 = T_vy in7 on chip (kick_adjoint);
//   drift:                        at in5, then at in4 = T_z in3 (in b3), at in3;
//   opening half kick (a_n):      one pass at x0.
// Velocity blocks without that pass regenerate in8 and in7 in b2 (and in5 again
// after them), in1 = T_vx x0 in b1 and in2 = T_vy in1 in b2. Where the device
// has no room for b3, in6 is formed in b1, and in3 and in5 are formed again
// after the closing half kick. Every regenerated input is computed by the
// kernels of the forward run, so it is the forward input bit for bit.
//
// The kicks read and drift_accel writes the acceleration of step n where it is
// kept (c->accel points there meanwhile).
int grad_impl(vp_ctx* c, int nsteps, double dt, int k, void* lam, double* loss)
{
  const size_t fb = (size_t)c->np * (size_t)c->nv3 * (c->cfg.dtype == VP_F32 ? 4 : 8);
  const size_t ab = sizeof(double) * 3 * (size_t)c->np;
  const int nck = (nsteps + k - 1) / k;
  void* user_f = c->f;
  GradWork w(c);
  // ck: every k-th state of the forward run; st[1..k-1]: the other states of
  // one segment, recomputed; b1, b2, b3: regenerated sweep inputs of one step
  std::vector<void*> ck(nck), st(k, nullptr);
  void *b1 = nullptr, *b2 = nullptr, *b3 = nullptr;
  double *ahist = nullptr, *lam_p = nullptr;
  int r;
  for (int i = 0; i < nck; i++)
    if ((r = w.f(&ck[i], fb))) return r;
  for (int i = 1; i < k; i++)
    if ((r = w.f(&st[i], fb))) return r;
  if ((r = w.f(&b1, fb)) || (r = w.f(&b2, fb))) return r;
  if ((r = w.d(&ahist, ab * (size_t)(nsteps + 1))) || (r = w.d(&lam_p, ab))) return r;
  // FP32: the separate gravity kernels and the x sweep's density sums, whose
  // roundings FP32 gradients keep. A last bit of an acceleration can move the
  // FP32 rounding of a line's alpha, and a corrector switch behind it: with the one-
  // launch solve one gradient of 16^3 x 24^3 in twelve (16 steps) came out 1.1e-9 from
  // that of the separate kernels, the others the same bits. The final state then
  // differs from vp_run's by that rounding (vp.h).
  if (c->cfg.dtype == VP_F32) {
    c->small = false;
    c->pair = 0;
  }
  const int nv[3] = {c->cfg.nv[0], c->cfg.nv[1], c->cfg.nv[2]};
  const bool fused_adj = vp::kick_adjoint_supported(c->cfg.dtype, nv);
  // all that the reverse pass cannot do without, before f changes and before b3
  const int vmin = std::min(nv[0], std::min(nv[1], nv[2]));
  if ((r = density_adjoint_fields(c))) return r;
  if (nsteps > 0 && !fused_adj && (r = line_adjoints(c, c->np * (c->nv3 / vmin)))) return r;
  // b3 where the device has room for it and for what the runtime itself takes at
  // a first launch (code objects, register spill space)
  size_t dev_free = 0, dev_total = 0;
  if (nsteps > 0 && hipMemGetInfo(&dev_free, &dev_total) != hipSuccess) hipGetLastError();
  if (nsteps > 0 && dev_free >= fb + kGradSpare && w.f(&b3, fb)) {
    b3 = nullptr;
    g_err.clear();
  }
  auto A = [&](int n) { return ahist + (size_t)n * 3 * c->np; };

  // forward pass from f0, keeping checkpoints and every step's acceleration
  if ((r = copy_f(c, A(0), w.user_accel, ab))) return r;
  c->accel = A(0);
  const double h = 0.5 * dt;
  // between checkpoints the closing half kick of step n-1 and the opening one
  // of step n (same acceleration) run as one pass, as in vp_run
  bool closing = false;   // the closing half kick of the previous step is still due
  for (int n = 0; n < nsteps; n++) {
    if (n % k == 0) {
      if (closing && (r = kick(c, h))) return r;
      closing = false;
      if ((r = copy_f(c, ck[n / k], user_f, fb))) return r;
    }
    if ((r = kick_n(c, h, closing ? 2 : 1))) return r;
    c->accel = A(n + 1);
    if ((r = drift_accel(c, dt))) return r;
    closing = true;
  }
  if (closing && (r = kick(c, h))) return r;
  // user_f now holds the final state; the reverse pass leaves it alone
  // loss = -U of the final state, seed lam = dL/df = -dx^3 dv^3 phi(x)
  if ((r = potential_into(c, c->phi))) return r;
  const double dx3 = c->dx[0] * c->dx[1] * c->dx[2], dv3 = c->dv[0] * c->dv[1] * c->dv[2];
  LAUNCH(c, vp::launch_potential_energy(c->red, c->rho, c->phi, c->ng, dx3, c->stream));
  HIP_TRY(hipMemcpyAsync(c->host, c->red, sizeof(double), hipMemcpyDeviceToHost, c->stream));
  LAUNCH(c, vp::launch_seed(lam, c->cfg.dtype, c->phi, c->ng, c->nv3, -dx3 * dv3, c->stream));
  // lam_p: the adjoint of the acceleration in hand, from the half kicks that use it
  HIP_TRY(hipMemsetAsync(lam_p, 0, ab, c->stream));

  for (int seg = nck - 1; seg >= 0; seg--) {
    const int s0 = seg * k, s1 = (s0 + k < nsteps) ? s0 + k : nsteps;
    st[0] = ck[seg];
    for (int n = s0; n + 1 < s1; n++) {   // recompute the segment's states
      c->accel = A(n);
      if ((r = kick_to(c, h, st[n - s0], st[n - s0 + 1], fb))) return r;
      c->accel = A(n + 1);                // written again, with the same values
      if ((r = drift_accel(c, dt)) || (r = kick(c, h))) return r;
    }
    for (int n = s1 - 1; n >= s0; n--) {
      void* x0 = st[n - s0];
      c->accel = A(n);
      if ((r = kick_to(c, h, x0, b1, fb))) return r;              // b1 = in3
      void* in6 = b3 ? b3 : b1;
      if (b3 && c->box3 && !fused_adj) {   // in5 is not kept
        if ((r = drift_box(c, dt, false, b1, b3))) return r;
      } else if (b3) {
        if ((r = zy_to(c, dt, b1, b2)) || (r = sweep_to(c, 0, dt, b2, b3))) return r;   // b2 = in5, b3 = in6
      } else if ((r = drift(c, dt))) {                            // b1 = in6
        return r;
      }
      // closing half kick, acceleration a_{n+1}
      c->accel = A(n + 1);
      bool have5 = b3 != nullptr;
      if (fused_adj) {
        if ((r = kick_adjoint(c, h, in6, lam, lam_p))) return r;
      } else {
        if ((r = sweep_to(c, 3, h, in6, b2)) || (r = sweep_on(c, 4, h, b2))) return r;
        if ((r = sweep_adjoint(c, 5, h, b2, lam, lam_p))) return r;          // at in8
        if ((r = sweep_to(c, 3, h, in6, b2)) || (r = sweep_adjoint(c, 4, h, b2, lam, lam_p))) return r;   // at in7
        if ((r = sweep_adjoint(c, 3, h, in6, lam, lam_p))) return r;         // at in6
        have5 = false;
      }
      // a_{n+1} = A(state after the drift): the density adjoint's contribution
      // to lam rides on the loads of the reverse x sweep that follows
      if ((r = density_adjoint(c, lam_p))) return r;
      HIP_TRY(hipMemsetAsync(lam_p, 0, ab, c->stream));
      // drift, then the opening half kick with a_n
      c->accel = A(n);
      if (!b3 && (r = kick_to(c, h, x0, b1, fb))) return r;       // b1 = in3
      if (!have5 && (r = zy_to(c, dt, b1, b2))) return r;         // b2 = in5
      if ((r = sweep_adjoint(c, 0, dt, b2, lam, nullptr, c->radj))) return r;
      void* in4 = b3 ? b3 : b2;
      if ((r = sweep_to(c, 2, dt, b1, in4)) || (r = sweep_adjoint(c, 1, dt, in4, lam, nullptr))) return r;
      if ((r = sweep_adjoint(c, 2, dt, b1, lam, nullptr))) return r;         // at in3
      if (fused_adj) {
        if ((r = kick_adjoint(c, h, x0, lam, lam_p))) return r;
        continue;
      }
      if ((r = sweep_to(c, 3, h, x0, b1)) || (r = sweep_to(c, 4, h, b1, b2))) return r;   // in1, in2
      if ((r = sweep_adjoint(c, 5, h, b2, lam, lam_p)) || (r = sweep_adjoint(c, 4, h, b1, lam, lam_p)) ||
          (r = sweep_adjoint(c, 3, h, x0, lam, lam_p)))
        return r;
    }
  }
  c->f = user_f;
  // a_0 = A(f0)
  if ((r = accel_adjoint(c, lam_p, lam))) return r;
  if ((r = copy_f(c, w.user_accel, A(nsteps), ab))) return r;
  HIP_TRY(hipStreamSynchronize(c->stream));
  *loss = -c->host[0];
  return VP_OK;
}

}  // namespace

int vp_grad(vp_ctx* c, int32_t nsteps, double dt, int32_t ckpt_every, void* grad_f0_dev, double* loss_host)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (nsteps < 0) return fail(VP_EINVAL, "nsteps must be >= 0");
  if (!(std::isfinite(dt) && dt > 0)) return fail(VP_EINVAL, "dt must be finite and > 0");
  if (ckpt_every < 1) return fail(VP_EINVAL, "ckpt_every must be >= 1");
  if (!grad_f0_dev || !loss_host) return fail(VP_EINVAL, "null pointer");
  if (reinterpret_cast<uintptr_t>(grad_f0_dev) % 16 != 0) return fail(VP_EINVAL, "gradient must be 16-byte aligned");
  r = grad_impl(c, nsteps, dt, ckpt_every, grad_f0_dev, loss_host);
  if (r) hipStreamSynchronize(c->stream);
  return r;
}

int vp_profile_enable(vp_ctx* c, int32_t on)
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if ((r = drain_events(c))) return r;
  c->profiling = on != 0;
  if (c->profiling) {
    for (int i = 0; i < VP_NPHASE; i++) {
      c->phase_ms[i] = 0;
      c->phase_n[i] = 0;
    }
  }
  return VP_OK;
}

int vp_profile_read(vp_ctx* c, double ms_out[VP_NPHASE], int64_t count_out[VP_NPHASE])
{
  g_err.clear();
  int r = check_ctx(c);
  if (r) return r;
  if (!ms_out || !count_out) return fail(VP_EINVAL, "null pointer");
  if ((r = drain_events(c))) return r;
  for (int i = 0; i < VP_NPHASE; i++) {
    ms_out[i] = c->phase_ms[i];
    count_out[i] = c->phase_n[i];
  }
  return VP_OK;
}

int vp_stream_copy(const void* src, void* dst, int64_t nbytes, void* hip_stream)
{
  g_err.clear();
  if (!src || !dst) return fail(VP_EINVAL, "null pointer");
  if (nbytes < 0 || nbytes % 16 != 0) return fail(VP_EINVAL, "nbytes must be a non-negative multiple of 16");
  const uintptr_t a = reinterpret_cast<uintptr_t>(src), b = reinterpret_cast<uintptr_t>(dst);
  if (a % 16 != 0 || b % 16 != 0) return fail(VP_EINVAL, "pointers must be 16-byte aligned");
  if (nbytes > 0 && a < b + (uintptr_t)nbytes && b < a + (uintptr_t)nbytes)
    return fail(VP_EINVAL, "source and destination overlap");
  const hipError_t e = vp::launch_copy16(src, dst, nbytes / 16, static_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) return fail(VP_EHIP, "copy: %s", hipGetErrorString(e));
  return VP_OK;
}

int vp_free(vp_ctx* c)
{
  g_err.clear();
  if (!c) return VP_OK;
  hipStreamSynchronize(c->stream);
  release(c);
  return VP_OK;
}

const char* vp_last_error(void) { return g_err.c_str(); }

}  // extern "C"
