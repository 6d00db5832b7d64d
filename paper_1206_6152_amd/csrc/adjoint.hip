// adjoint.hip -- reverse mode of the directional PFC sweep (not in the paper;
// it gives gradients of the final field energy for the C ABI's vp_grad).
//
// For one line with forward input f (the sweep's input state), Courant number
// nu = s + sign * alpha and output adjoint lam_out, the lane recomputes the
// forward quantities (f_inf and its first argmax, the one-sided differences
// and which bound of each corrector clamp is active) and runs the flux form
// backwards, in the same mirrored register view as the forward update:
//   lam_g_k = lam_out_{k+s}                     (transpose of the shift)
//   lam_F_k = lam_g_{k+1} - lam_g_k             (F_k leaves cell k, enters k+1)
//   F_k = alpha * (f_k + c1 Lp_k + c2 Lm_k):
//     lam_f_k += alpha lam_F_k, lam_Lp = c1 alpha lam_F_k, lam_Lm = c2 alpha lam_F_k,
//     lam_alpha += lam_F_k (f_k + c1 Lp_k + c2 Lm_k + alpha (c1' Lp_k + c2' Lm_k)),
//     c1' = (2 alpha - 3)/6, c2' = -alpha/3;
//   Lp = clamp(f_{k+1} - f_k, 2 f_k - 2 f_inf, 2 f_k) and
//   Lm = clamp(f_k - f_{k-1}, -2 f_k, 2 f_inf - 2 f_k) pass their adjoint to
//   the operands of the active branch (a bound is active only when the
//   difference is strictly beyond it), f_inf passes its adjoint to the first
//   cell holding the maximum, and lam_nu = sign * lam_alpha.
// A velocity sweep's nu = a_l(x) tau / dv_l sends lam_nu to the acceleration;
// the per-line values are reduced per spatial cell in a fixed order.
#include "adj_line.h"
#include "vec16.h"
#include "vp_internal.h"

namespace vp {
namespace {

// Reverse of pfc_line + store_shifted for one line; returns d<lam_out, out>/d nu.
// `at(r)` is the offset of storage cell r of the lane's line from both bases,
// la(r, x) the lam value of cell r from its stored value x. The view runs along
// the transport direction: view cell i is storage cell i (nu >= 0) or N-1-i
// (nu < 0). The lane's forward line is mirrored into the view with selects, so
// every lane follows the same instruction stream whatever its sign. In the
// view the shift's transpose is lam_g_k = lam_out_{k+m} (zero beyond an outflow
// end, wrapped if periodic): where the line has a whole-cell shift, lam_g is
// read straight into view order, each view cell from the storage cell that the
// mirror and the transposed shift name.
template <typename T, int N, bool ALPHA, typename AT, typename LA>
__device__ __forceinline__ double adj_line(const T* fin, T* lam, double nu, bool periodic, AT at, LA la)
{
  const AdjCoef<T> k = adj_coef<T, N>(nu, periodic);
  const bool neg = k.neg;
  T w[N], l[N];
#pragma unroll
  for (int r = 0; r < N; r++) w[r] = fin[at(r)];
  auto straight = [&]() __attribute__((always_inline)) {   // storage order, then the mirror
#pragma unroll
    for (int r = 0; r < N; r++) l[r] = la(r, lam[at(r)]);
#pragma unroll
    for (int i = 0; i < N / 2; i++) {
      const T p = l[i], q = l[N - 1 - i];
      l[i] = neg ? q : p;
      l[N - 1 - i] = neg ? p : q;
    }
  };
  // Short FP32 lines are read before the branch on the shift (8 cells: 2 to 4 % of
  // the pass), longer ones would hold their registers through it (24 cells: 6 to
  // 11 % more).
  constexpr bool EARLY = sizeof(T) == 4 && N <= 12;
  if constexpr (EARLY) {
    straight();
#pragma unroll
    for (int r = 0; r < N; r++) asm volatile("" : "+v"(l[r]));   // not sunk into the branch
  }
  if (k.shift != 0) {
    int m = k.shift;
    asm volatile("" : "+v"(m));               // the places below stay inside this rarely taken branch
#pragma unroll
    for (int i = 0; i < N; i++) {
      int j = i + m;
      if (periodic && j >= N) j -= N;
      const bool in = j < N;                  // else past an outflow end: zero
      const int rs = in ? (neg ? N - 1 - j : j) : 0;
      const T x = la(rs, lam[at(rs)]);
      l[i] = in ? x : T(0);
    }
  } else if constexpr (!EARLY) {
    straight();
  }
  // f_inf and the first storage cell that holds it (none on an empty line)
  T finf = T(0);
#pragma unroll
  for (int r = 0; r < N; r++) finf = max_(finf, w[r]);
  int am = -1;
#pragma unroll
  for (int r = N - 1; r >= 0; r--) am = w[r] == finf ? r : am;
  if (!(finf > T(0))) am = -1;
#pragma unroll
  for (int i = 0; i < N / 2; i++) {
    const T x = w[i], y = w[N - 1 - i];
    w[i] = neg ? y : x;
    w[N - 1 - i] = neg ? x : y;
  }
  T lfinf, lalpha;
  adj_core<T, N, ALPHA>(w, l, finf, k, periodic, lfinf, lalpha);
  // back to storage order
#pragma unroll
  for (int i = 0; i < N / 2; i++) {
    const T p = l[i], q = l[N - 1 - i];
    l[i] = neg ? q : p;
    l[N - 1 - i] = neg ? p : q;
  }
#pragma unroll
  for (int r = 0; r < N; r++) lam[at(r)] = r == am ? l[r] + lfinf : l[r];
  return neg ? -(double)lalpha : (double)lalpha;
}

template <typename T, int N, bool ALPHA, typename AT>
__device__ __forceinline__ double adj_line(const T* fin, T* lam, double nu, bool periodic, AT at)
{
  return adj_line<T, N, ALPHA>(fin, lam, nu, periodic, at, [](int, T x) { return x; });
}

__device__ __forceinline__ double adj_line_nu(const SweepArgs& a, long long o, long long c)
{
  if (a.velocity) return a.accel[o / a.sp_div] * a.scale;
  const long long j = (c / a.j_div) % a.j_mod;
  return (a.vmin + ((double)j + 0.5) * a.dv) * a.scale;
}

// NARROW: the workgroup's first line is the uniform base and a lane's cells sit
// at base + r*inner + off with a 32-bit offset (the host checks that they fit),
// as in the forward strided sweep; otherwise 64-bit addressing per lane.
// ALPHA: the lines' adjoints of nu are wanted (dnu). Position sweeps have no use
// for them, and without them a line takes seven instructions per cell less.
template <typename T, int N, bool ALPHA, bool NARROW, bool ADD = false>
__global__ __launch_bounds__(256) void sweep_adj_kernel(SweepArgs a, const T* fin, T* lam, double* dnu)
{
  const long long gid = (long long)blockIdx.x * 256 + threadIdx.x;
  if (gid >= a.nlines) return;
  double d;
  if constexpr (NARROW) {
    const long long gid0 = (long long)blockIdx.x * 256;
    const unsigned t = threadIdx.x;
    const long long o0 = gid0 / a.inner;
    const unsigned inner = (unsigned)a.inner;
    const unsigned c0 = (unsigned)(gid0 - o0 * a.inner);
    const unsigned cc = c0 + t;
    const unsigned dov = cc / inner;
    const unsigned c = cc - dov * inner;
    const unsigned off = dov * (unsigned)(N * inner) + c - c0;
    const long long b0 = o0 * N * (long long)inner + c0;
    double nu;
    if (a.velocity) {
      const long long q0 = o0 / a.sp_div;
      const unsigned r0 = (unsigned)(o0 - q0 * a.sp_div);
      nu = a.accel[q0 + (r0 + dov) / (unsigned)a.sp_div] * a.scale;
    } else {
      const unsigned j = (c / (unsigned)a.j_div) % (unsigned)a.j_mod;
      nu = (a.vmin + ((double)j + 0.5) * a.dv) * a.scale;
    }
    // uniform row base (r * inner) plus the lane's 32-bit offset
    if constexpr (ADD) {
      const long long o = o0 + dov;
      const double* add = a.addend + c / (unsigned)a.add_div;
      d = adj_line<T, N, ALPHA>(fin + b0, lam + b0, nu, a.periodic != 0,
                         [&](int r) { return (long long)r * inner + off; },
                         [&](int r, T x) { return (T)((double)x + a.add_coef * add[(o * N + r) * a.add_stride]); });
    } else {
      d = adj_line<T, N, ALPHA>(fin + b0, lam + b0, nu, a.periodic != 0,
                         [&](int r) { return (long long)r * inner + off; });
    }
  } else {
    const long long o = gid / a.inner;
    const long long c = gid - o * a.inner;
    const long long base = o * (long long)N * a.inner + c;
    const long long inner = a.inner;
    d = adj_line<T, N, ALPHA>(fin + base, lam + base, adj_line_nu(a, o, c), a.periodic != 0,
                       [&](int r) { return (long long)r * inner; });
  }
  if constexpr (ALPHA) dnu[gid] = d;
}

// Contiguous lines (inner == 1, the vz sweep): a workgroup stages LINES
// consecutive lines of the forward input and of lam through LDS with coalesced
// loads (rows padded to N + 1), each lane runs the reverse update of one line
// there, and lam goes back the same way.
template <typename T, int N>
struct AdjContig {
  static constexpr int P = N + 1;
  static constexpr int LINES = (2 * 256 * P * (int)sizeof(T) <= 65536) ? 256
                               : (2 * 128 * P * (int)sizeof(T) <= 65536) ? 128 : 64;
};

template <typename T, int N, bool ALPHA>
__global__ __launch_bounds__((AdjContig<T, N>::LINES)) void sweep_adj_contig(SweepArgs a, const T* fin, T* lam,
                                                                             double* dnu)
{
  using S = AdjContig<T, N>;
  constexpr int LINES = S::LINES, P = S::P;
  __shared__ T tf[LINES * P];
  __shared__ T tl[LINES * P];
  const int tid = threadIdx.x;
  const long long line0 = (long long)blockIdx.x * LINES;
  const long long left = a.nlines - line0;
  const int nl = left < LINES ? (int)left : LINES;
  const T* gf = fin + line0 * N;
  T* gl = lam + line0 * N;
  if (nl == LINES) {
    T xf[N], xl[N];
#pragma unroll
    for (int k = 0; k < N; k++) {
      xf[k] = gf[tid + k * LINES];
      xl[k] = gl[tid + k * LINES];
    }
#pragma unroll
    for (int k = 0; k < N; k++) {
      const int e = tid + k * LINES;
      tf[(e / N) * P + (e % N)] = xf[k];
      tl[(e / N) * P + (e % N)] = xl[k];
    }
  } else {
    for (int e = tid; e < nl * N; e += LINES) {
      tf[(e / N) * P + (e % N)] = gf[e];
      tl[(e / N) * P + (e % N)] = gl[e];
    }
  }
  __syncthreads();
  if (tid < nl) {
    const long long line = line0 + tid;
    const double nu = a.velocity ? a.accel[line / a.sp_div] * a.scale
                                 : (a.vmin + 0.5 * a.dv) * a.scale;   // one velocity cell on this axis
    const double d = adj_line<T, N, ALPHA>(tf + tid * P, tl + tid * P, nu, a.periodic != 0, [&](int r) { return r; });
    if constexpr (ALPHA) dnu[line] = d;
  }
  __syncthreads();
  if (nl == LINES) {
#pragma unroll
    for (int k = 0; k < N; k++) {
      const int e = tid + k * LINES;
      gl[e] = tl[(e / N) * P + (e % N)];
    }
  } else {
    for (int e = tid; e < nl * N; e += LINES) gl[e] = tl[(e / N) * P + (e % N)];
  }
}

// lam_a[s] += scale * sum of dnu over the lines of spatial cell s (a
// contiguous run of `per` line indices), fixed-order tree per workgroup.
__global__ __launch_bounds__(256) void reduce_lines_kernel(double* lam_a, const double* dnu, long long per,
                                                           double scale)
{
  __shared__ double sh[256];
  const long long s = blockIdx.x;
  double acc = 0.0;
  for (long long i = threadIdx.x; i < per; i += 256) acc += dnu[s * per + i];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) lam_a[s] += scale * sh[0];
}

// LDS that a workgroup of a strided FP32 velocity sweep asks for without using it,
// so that only two share a CU: on arrays beyond the last-level cache the long lines
// of two arrays, read and written by every wave that the registers allow, cost more
// than the waves hide (vx lines of 24 cells, 1.7 GB, us: seven workgroups on a CU
// 1088, two 964; without alpha's adjoint 1029 and 914; 32 cells, 0.8 GB, 482 and 426).
// Smaller arrays, shorter lines and position sweeps lose up to 14 % by it.
static unsigned adj_spare_lds(const SweepArgs& a, int es)
{
  return a.velocity && es == 4 && a.n >= 24 && a.nlines * a.n * es >= (1LL << 28) ? 79 * 1024 : 0;
}

template <typename T, int N, bool ALPHA>
hipError_t launch_adj_a(const SweepArgs& a, const T* fin, T* lam, double* dnu, hipStream_t s)
{
  if (a.inner == 1) {
    if (a.addend) return hipErrorInvalidValue;
    constexpr int LINES = AdjContig<T, N>::LINES;
    hipLaunchKernelGGL((sweep_adj_contig<T, N, ALPHA>), dim3((unsigned)((a.nlines + LINES - 1) / LINES)), dim3(LINES),
                       0, s, a, fin, lam, dnu);
    return hipGetLastError();
  }
  const dim3 blocks((unsigned)((a.nlines + 255) / 256));
  const unsigned spare = adj_spare_lds(a, (int)sizeof(T));
  if (a.addend) {
    if (!narrow_ok(a, N)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((sweep_adj_kernel<T, N, ALPHA, true, true>), blocks, dim3(256), 0, s, a, fin, lam, dnu);
  } else if (narrow_ok(a, N))
    hipLaunchKernelGGL((sweep_adj_kernel<T, N, ALPHA, true>), blocks, dim3(256), spare, s, a, fin, lam, dnu);
  else
    hipLaunchKernelGGL((sweep_adj_kernel<T, N, ALPHA, false>), blocks, dim3(256), spare, s, a, fin, lam, dnu);
  return hipGetLastError();
}

template <typename T, int N>
hipError_t launch_adj_n(const SweepArgs& a, const void* fin, void* lam, double* dnu, hipStream_t s)
{
  if (a.nlines <= 0) return hipSuccess;
  const T* f = static_cast<const T*>(fin);
  T* l = static_cast<T*>(lam);
  return dnu ? launch_adj_a<T, N, true>(a, f, l, dnu, s) : launch_adj_a<T, N, false>(a, f, l, dnu, s);
}

template <typename T>
hipError_t launch_adj_t(const SweepArgs& a, const void* fin, void* lam, double* dnu, hipStream_t s)
{
  switch (a.n) {
    case 1: return launch_adj_n<T, 1>(a, fin, lam, dnu, s);
    case 2: return launch_adj_n<T, 2>(a, fin, lam, dnu, s);
    case 3: return launch_adj_n<T, 3>(a, fin, lam, dnu, s);
    case 4: return launch_adj_n<T, 4>(a, fin, lam, dnu, s);
    case 6: return launch_adj_n<T, 6>(a, fin, lam, dnu, s);
    case 8: return launch_adj_n<T, 8>(a, fin, lam, dnu, s);
    case 12: return launch_adj_n<T, 12>(a, fin, lam, dnu, s);
    case 16: return launch_adj_n<T, 16>(a, fin, lam, dnu, s);
    case 24: return launch_adj_n<T, 24>(a, fin, lam, dnu, s);
    case 32: return launch_adj_n<T, 32>(a, fin, lam, dnu, s);
    case 48: return launch_adj_n<T, 48>(a, fin, lam, dnu, s);
    case 64: return launch_adj_n<T, 64>(a, fin, lam, dnu, s);
    case 96: return launch_adj_n<T, 96>(a, fin, lam, dnu, s);
    case 128: return launch_adj_n<T, 128>(a, fin, lam, dnu, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

bool adjoint_addend_supported(const SweepArgs& a)
{
  return a.inner > 1 && a.add_div > 0 && narrow_ok(a, a.n);
}

hipError_t launch_sweep_adjoint(const SweepArgs& a, int dtype, const void* fin, void* lam, double* dnu,
                                hipStream_t s)
{
  return dtype == 0 ? launch_adj_t<float>(a, fin, lam, dnu, s) : launch_adj_t<double>(a, fin, lam, dnu, s);
}

hipError_t launch_reduce_lines(double* lam_a, const double* dnu, long long np, long long per, double scale,
                               hipStream_t s)
{
  if (np <= 0) return hipSuccess;
  hipLaunchKernelGGL(reduce_lines_kernel, dim3((unsigned)np), dim3(256), 0, s, lam_a, dnu, per, scale);
  return hipGetLastError();
}

}  // namespace vp
