// box.h -- several directional sweeps of Eq. (17) in one pass over f for
// grids of any accepted axis lengths (Sec. 2.1 of Yoshikawa, Yoshida &
// Umemura): a box of lines is held in LDS and swept along its axes in turn,
// with the axis lengths as run-time values. Included by box_f32.hip and
// box_f64.hip, one per storage type. gfx950.
//
//   kick_box   the velocity block of one spatial cell: T_vx, T_vy, T_vz (once
//              or twice) for blocks that fit the LDS and have no kernel of
//              their own (kick.hip has cubes of 8, 16, 24, 32)
//   drift_box  W consecutive velocity cells of a whole spatial grid: T_z, T_y,
//              T_x, with the density sums of the new f (FP64)
//
// A line's length has to be a constant where the line is held in registers, so
// a sweep branches once (uniformly) to the code of its length; a kernel is
// built for the lengths up to NMAX, which sets its register count. All axes go
// through the same code, which keeps it short: a small grid runs each sweep
// once or twice per workgroup, and fetching straight-line code that is used
// once costs more than its arithmetic. Strides are run-time values: one
// address addition per access, against which sweeping a line from its far end
// (nu < 0) costs nothing. The line update is that of sweep.hip (pfc_line.h),
// so every pass rounds like the single sweeps.
#pragma once

#include "pfc_line.h"
#include "vec16.h"
#include "vp_internal.h"

namespace vp {
namespace {

// Coefficients of a line in the direction of its motion: |nu| = shift + alpha.
// meta holds 2 shift + neg: 0 <= shift < n (periodic) or <= n; neg: nu < 0, the
// line is swept from its far end.
template <typename T>
struct alignas(16) BoxCoef {
  T alpha, c1, c2;
  int meta;
  __device__ __forceinline__ int shift() const { return meta >> 1; }
  __device__ __forceinline__ bool neg() const { return meta & 1; }
};

// line_coef for a run-time length
template <typename T>
__device__ __forceinline__ BoxCoef<T> box_coef(double nu, int n, bool periodic)
{
  const double a = fabs(nu), fl = floor(a);
  const LineCoef<T> k = line_coef<T, 1>(a - fl, false);
  int m;
  if (fl >= (double)n) m = periodic ? (int)fmod(fl, (double)n) : n;
  else m = (int)fl;
  return BoxCoef<T>{k.alpha, k.c1, k.c2, 2 * m + (nu < 0.0 ? 1 : 0)};
}

// u / d for 0 <= u < 2^24, d >= 1, inv = 1.0f / d
__device__ __forceinline__ int quot(int u, int d, float inv)
{
  int q = (int)((float)u * inv);
  q += ((q + 1) * d <= u) ? 1 : 0;
  q -= (q * d > u) ? 1 : 0;
  return q;
}

// One line of N cells in LDS, cell i (in its direction of motion) at p + i d;
// the result is written at its shifted place.
template <typename T, int N>
__device__ __forceinline__ void box_line(T* L, int p, int d, const BoxCoef<T>& c, bool periodic)
{
  T v[N];
#pragma unroll
  for (int r = 0; r < N; r++) v[r] = L[p + r * d];
  pfc_core<T, N>(v, c.alpha, c.c1, c.c2, periodic);
  // long lines: the places are computed again, not kept in N registers
  if constexpr (N >= 24) asm volatile("" : "+v"(p), "+v"(d));
  int m = c.shift();
  if (m == 0) {
#pragma unroll
    for (int r = 0; r < N; r++) L[p + r * d] = v[r];
    return;
  }
  asm volatile("" : "+v"(m));   // the places below stay inside this rarely taken branch
#pragma unroll
  for (int r = 0; r < N; r++) {
    int i = r + m;
    if (periodic && i >= N) i -= N;
    if (i < N) L[p + i * d] = v[r];
  }
  if (!periodic)
    for (int i = 0; i < m; i++) L[p + i * d] = T(0);
}

// Sweep of all lines of a box along one axis: nl lines of n cells (stride st),
// line li = (i nj + j) 2^lgw + w at i si + j sj + w, coefficients cf[w].
template <typename T, int N>
__device__ __forceinline__ void box_lines(T* L, int st, int nl, int lgw, int nj, int si, int sj,
                                          const BoxCoef<T>* cf, bool periodic)
{
  const float rj = 1.0f / (float)nj;
  for (int li = threadIdx.x; li < nl; li += blockDim.x) {
    const int w = li & ((1 << lgw) - 1), q = li >> lgw;
    const int i = quot(q, nj, rj), j = q - i * nj;
    const BoxCoef<T> c = cf[w];
    const int base = i * si + j * sj + w;
    box_line<T, N>(L, c.neg() ? base + (N - 1) * st : base, c.neg() ? -st : st, c, periodic);
  }
}

constexpr int kBoxRed = 512;   // split lines: at most this many lanes

// The same sweep with each line split over n / S lanes, S consecutive cells
// each: for boxes with too few lines to fill the workgroup, where one lane per
// line is a chain of n cells (128 FP64 cells: 6 us of the 1D-1V kick's 20). All
// reads and the cells' part of the line maximum come before a barrier (red: one
// value per lane), the update after it recomputes the flux that enters the
// first cell. nl n / S lanes at most take part. The arithmetic of each cell is
// pfc_core's.
template <typename T, int S>
__device__ __forceinline__ void box_split(T* L, T* red, int n, int st, int nl, int lgw, int nj, int si, int sj,
                                          const BoxCoef<T>* cf, bool periodic)
{
#pragma clang fp contract(off)
  const int P = n / S, it = threadIdx.x;
  const bool on = it < nl * P;
  const float rp = 1.0f / (float)P, rj = 1.0f / (float)nj;
  const int line = quot(it, P, rp), k0 = (it - line * P) * S;
  const int w = line & ((1 << lgw) - 1), q = line >> lgw;
  const int i = quot(q, nj, rj), j = q - i * nj;
  T v[S + 3];            // cells k0 - 2 .. k0 + S
  BoxCoef<T> c{};
  int p = 0, d = 0;
  if (on) {
    c = cf[w];
    const int base = i * si + j * sj + w;
    p = c.neg() ? base + (n - 1) * st : base;
    d = c.neg() ? -st : st;
    T m = T(0);
#pragma unroll
    for (int r = 0; r < S + 3; r++) {
      int k = k0 + r - 2;
      if (periodic) k += k < 0 ? n : (k >= n ? -n : 0);
      v[r] = k >= 0 && k < n ? L[p + k * d] : T(0);
    }
#pragma unroll
    for (int r = 0; r < S; r++) m = max_(m, v[r + 2]);
    red[it] = m;
  }
  __syncthreads();
  if (on) {
    T finf = T(0);
    for (int k = 0; k < P; k++) finf = max_(finf, red[line * P + k]);
    const T twoinf = finf + finf;
    T qprev = T(0);
    T dm = v[1] - v[0];
#pragma unroll
    for (int r = 1; r < S + 2; r++) {
      const T f0 = v[r], dp = v[r + 1] - f0, h = f0 + f0, rr = twoinf - h;
      const T lp = clamp_ordered(dp, -rr, h), lm = clamp_ordered(dm, -h, rr);
      T qk = fma_(c.c2, lm, fma_(c.c1, lp, f0));
      if (r == 1 && !periodic && k0 == 0) qk = T(0);   // nothing enters an outflow line
      if (r > 1) {
        int k = k0 + r - 2 + c.shift();
        if (periodic && k >= n) k -= n;
        const T g = fma_(c.alpha, qprev - qk, f0);
        if (k < n) L[p + k * d] = g;
        if (!periodic && k0 + r - 2 < c.shift()) L[p + (k0 + r - 2) * d] = T(0);
      }
      qprev = qk;
      dm = dp;
    }
  }
}

template <typename T, int NMAX>
__device__ __forceinline__ void box_sweep(T* L, T* red, int n, int st, int nl, int lgw, int nj, int si, int sj,
                                          const BoxCoef<T>* cf, bool periodic)
{
  const int most = (int)blockDim.x < kBoxRed ? (int)blockDim.x : kBoxRed;
  if (n >= 16 && nl * (n / 8) <= most) {   // uniform; lengths from 16 on are multiples of 8
    if (nl * (n / 4) <= most)
      box_split<T, 4>(L, red, n, st, nl, lgw, nj, si, sj, cf, periodic);
    else
      box_split<T, 8>(L, red, n, st, nl, lgw, nj, si, sj, cf, periodic);
    return;
  }
#define VP_BOX_LEN(N) \
  case N: box_lines<T, N>(L, st, nl, lgw, nj, si, sj, cf, periodic); break
  if constexpr (NMAX == 16) {
    switch (n) {
      VP_BOX_LEN(1); VP_BOX_LEN(2); VP_BOX_LEN(3); VP_BOX_LEN(4); VP_BOX_LEN(6); VP_BOX_LEN(8); VP_BOX_LEN(12);
      VP_BOX_LEN(16);
    }
  } else if constexpr (NMAX == 32) {
    switch (n) {
      VP_BOX_LEN(1); VP_BOX_LEN(2); VP_BOX_LEN(3); VP_BOX_LEN(4); VP_BOX_LEN(6); VP_BOX_LEN(8); VP_BOX_LEN(12);
      VP_BOX_LEN(16); VP_BOX_LEN(24); VP_BOX_LEN(32);
    }
  } else if constexpr (NMAX == 48) {
    switch (n) {
      VP_BOX_LEN(1); VP_BOX_LEN(2); VP_BOX_LEN(3); VP_BOX_LEN(4); VP_BOX_LEN(6); VP_BOX_LEN(8); VP_BOX_LEN(12);
      VP_BOX_LEN(16); VP_BOX_LEN(24); VP_BOX_LEN(32); VP_BOX_LEN(48);
    }
  } else if constexpr (NMAX == 64) {
    switch (n) {
      VP_BOX_LEN(1); VP_BOX_LEN(2); VP_BOX_LEN(3); VP_BOX_LEN(4); VP_BOX_LEN(6); VP_BOX_LEN(8); VP_BOX_LEN(12);
      VP_BOX_LEN(16); VP_BOX_LEN(24); VP_BOX_LEN(32); VP_BOX_LEN(48); VP_BOX_LEN(64);
    }
  } else {
    switch (n) {
      VP_BOX_LEN(1); VP_BOX_LEN(2); VP_BOX_LEN(3); VP_BOX_LEN(4); VP_BOX_LEN(6); VP_BOX_LEN(8); VP_BOX_LEN(12);
      VP_BOX_LEN(16); VP_BOX_LEN(24); VP_BOX_LEN(32); VP_BOX_LEN(48); VP_BOX_LEN(64); VP_BOX_LEN(96);
      VP_BOX_LEN(128);
    }
  }
#undef VP_BOX_LEN
}

// Workgroup sizes: 16 waves hold lines of up to 64 FP32 or 32 FP64 cells
// without spilling, eight waves longer ones.
constexpr int box_threads_most(int nmax, int es) { return nmax * es <= 256 ? 1024 : 512; }

template <typename T, int NMAX>
constexpr int box_threads()
{
  return box_threads_most(NMAX, (int)sizeof(T));
}

// ---- velocity blocks -----------------------------------------------------------
// LDS: [vx][vy][vz] with rows of SY = nz or nz + 1 elements (odd, so that the
// vz lines of a wave, one row apart, take distinct banks).
template <typename T, int NMAX>
__global__ __launch_bounds__((box_threads<T, NMAX>())) void kick_box(KickArgs a, int nx, int ny, int nz)
{
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  T* L = reinterpret_cast<T*>(lds_raw);
  __shared__ BoxCoef<T> cf[3];
  __shared__ T red[kBoxRed];
  constexpr int V = Vec16<T>::n;
  using VT = typename Vec16<T>::type;
  const int tid = threadIdx.x, nth = blockDim.x;
  const int sy = nz | 1, sx = ny * sy, nv3 = nx * ny * nz;
  const T* g = static_cast<const T*>(a.f) + (long long)blockIdx.x * nv3;
  T* go = static_cast<T*>(a.out ? a.out : a.f) + (long long)blockIdx.x * nv3;
  const float rz = 1.0f / (float)nz;
  // in, four loads in flight per lane; whole 16-byte vectors where they make up
  // the vz rows (each row then starts on 16 bytes, as f does). Row vx ny + vy
  // lies at (vx ny + vy) SY in LDS.
  const double nux = a.a[0][blockIdx.x] * a.scale[0], nuy = a.a[1][blockIdx.x] * a.scale[1],
               nuz = a.a[2][blockIdx.x] * a.scale[2];
  const bool vec = nz % V == 0;
  const int nvec = vec ? nv3 / V : 0;
  const VT* gv = reinterpret_cast<const VT*>(g);
  VT x[4];
  auto fetch = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 4; k++)
      if (e0 + k * nth < nvec) x[k] = gv[e0 + k * nth];
  };
  fetch(tid);
  // the coefficients while the first loads are in flight
  if (tid < 3)
    cf[tid] = box_coef<T>(tid == 0 ? nux : (tid == 1 ? nuy : nuz), tid == 0 ? nx : (tid == 1 ? ny : nz), false);
  for (int e0 = tid; e0 < nvec; e0 += 4 * nth) {
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const int e = (e0 + k * nth) * V;
      if (e >= nv3) break;
      const int row = quot(e, nz, rz), at = row * sy + (e - row * nz);
#pragma unroll
      for (int q = 0; q < V; q++) L[at + q] = lane_of<VT, T>(x[k], q);
    }
    fetch(e0 + 4 * nth);
  }
  if (!vec) {
    for (int e = tid; e < nv3; e += nth) {
      const int row = quot(e, nz, rz);
      L[row * sy + (e - row * nz)] = g[e];
    }
  }
  __syncthreads();
#pragma unroll 1
  for (int k = 0; k < 3 * a.reps; k++) {
    const int ax = k >= 3 ? k - 3 : k;
    // lines (i, j): vx lines (vy, vz), vy lines (vx, vz), vz lines (vx, vy)
    const int n = ax == 0 ? nx : (ax == 1 ? ny : nz), st = ax == 0 ? sx : (ax == 1 ? sy : 1);
    const int nl = ax == 0 ? ny * nz : (ax == 1 ? nx * nz : nx * ny);
    box_sweep<T, NMAX>(L, red, n, st, nl, 0, ax == 2 ? ny : nz, ax == 0 ? sy : sx, ax == 2 ? sy : 1, cf + ax, false);
    __syncthreads();
  }
  if (vec) {
    for (int e = tid * V; e < nv3; e += nth * V) {
      const int row = quot(e, nz, rz), at = row * sy + (e - row * nz);
      VT x;
      T* xs = reinterpret_cast<T*>(&x);
#pragma unroll
      for (int q = 0; q < V; q++) xs[q] = L[at + q];
      *reinterpret_cast<VT*>(go + e) = x;
    }
  } else {
    for (int e = tid; e < nv3; e += nth) {
      const int row = quot(e, nz, rz);
      go[e] = L[row * sy + (e - row * nz)];
    }
  }
}

template <typename T, int NMAX>
hipError_t launch_kick_box_n(const KickArgs& a, const int nv[3], hipStream_t st)
{
  const size_t lds = (size_t)nv[0] * nv[1] * (nv[2] | 1) * sizeof(T);
  int th = kick_box_threads(sizeof(T) == 4 ? 0 : 1, nv, a.np);
  if (th > box_threads<T, NMAX>()) th = box_threads<T, NMAX>();   // NMAX may be a class above the longest axis
  hipLaunchKernelGGL((kick_box<T, NMAX>), dim3((unsigned)a.np), dim3(th), lds, st, a, nv[0], nv[1], nv[2]);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_kick_box_t(const KickArgs& a, const int nv[3], hipStream_t st)
{
  if (a.np <= 0) return hipSuccess;
  int m = nv[0] > nv[1] ? nv[0] : nv[1];
  m = nv[2] > m ? nv[2] : m;
  if (m <= 16) return launch_kick_box_n<T, 16>(a, nv, st);
  if (m <= 32) return launch_kick_box_n<T, 32>(a, nv, st);
  if (m <= 48) return launch_kick_box_n<T, 48>(a, nv, st);
  if (m <= 64) return launch_kick_box_n<T, 64>(a, nv, st);
  return launch_kick_box_n<T, 128>(a, nv, st);
}

// ---- spatial boxes ---------------------------------------------------------------
// A workgroup holds W = 2^lgw consecutive velocity cells of all n0 x n1 x n2
// spatial cells, LDS [x][y][z][w]. Rows (one y)
// are padded to SY = W (mod the 64 banks), so that the lines of a wave take
// distinct banks in every direction. With part set the W new values of each
// spatial cell are summed in FP64, in a fixed order, as they leave:
// part[chunk np + cell], from which the density follows without another pass
// over f.
struct DriftBoxShape {
  int n[3];
  int lgw;
  int sy, sx;          // LDS strides in elements
  int periodic;
  int nvy, nvz, nv3, nchunk;
  double v0[3], dv[3], scale[3];   // v0: vmin
  int xcd_group;       // > 1: that many workgroups that share cache lines on one XCD (see drift.hip)
};

constexpr int kBoxW = 32;   // most velocity cells per workgroup

template <typename T, int NMAX>
__global__ __launch_bounds__((box_threads<T, NMAX>())) void drift_box(const T* fin, T* fout, DriftBoxShape s,
                                                                      double* part)
{
  static_assert(sizeof(T) == 8, "drift_box_cells offers FP64 only");
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  T* L = reinterpret_cast<T*>(lds_raw);
  __shared__ BoxCoef<T> cf[3][kBoxW];
  __shared__ T red[kBoxRed];
  constexpr int V = Vec16<T>::n;
  using VT = typename Vec16<T>::type;
  const int tid = threadIdx.x, nth = blockDim.x, lgw = s.lgw, W = 1 << lgw;
  unsigned b = blockIdx.x;
  if (s.xcd_group > 1) {             // blocks 8 (G m + q) + x: q-th chunk of line group 8 m + x
    const unsigned G = s.xcd_group, x = b & 7, k = b >> 3, m = k / G;
    b = (8 * m + x) * G + (k - m * G);
  }
  const int chunk = (int)b;
  const int j0 = chunk << lgw;
  const int nw = s.nv3 - j0 < W ? s.nv3 - j0 : W;   // the last chunk may be narrower
  const bool periodic = s.periodic != 0;
  const int n0 = s.n[0], n1 = s.n[1], n2 = s.n[2], np = n0 * n1 * n2;
  const long long nv3 = s.nv3;
  const T* g = fin + j0;
  T* go = fout + j0;
  const float r1 = 1.0f / (float)n1, r2 = 1.0f / (float)n2;
  const int sx = s.sx, sy = s.sy;
  auto place = [=](int cell) {       // LDS place of a spatial cell
    const int row = quot(cell, n2, r2), x = quot(row, n1, r1);
    return x * sx + (row - x * n1) * sy + ((cell - row * n2) << lgw);
  };
  // whole 16-byte vectors where the runs start on 16 bytes (f does)
  const bool vec = nv3 % V == 0 && W % V == 0;
  constexpr int lgv = V == 4 ? 2 : 1;
  const int lq = lgw - lgv, nvec = vec ? np << lq : 0;
  VT x[4];
  auto fetch = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const int e = e0 + k * nth, w = (e & ((1 << lq) - 1)) << lgv;
      if (e < nvec && w < nw) x[k] = *reinterpret_cast<const VT*>(g + (long long)(e >> lq) * nv3 + w);
    }
  };
  fetch(tid);
  // the coefficients while the first loads are in flight, by 3 W lanes (every
  // workgroup has at least 3 kBoxW)
  if (tid < 3 * W) {
    const unsigned nvy = s.nvy, nvz = s.nvz;
    const int l = tid >> lgw, w = tid & (W - 1);
    const unsigned j = (unsigned)(j0 + (w < nw ? w : 0)), jr = j / nvz, jx = jr / nvy;
    const double nux = (s.v0[0] + ((double)jx + 0.5) * s.dv[0]) * s.scale[0];
    const double nuy = (s.v0[1] + ((double)(jr - jx * nvy) + 0.5) * s.dv[1]) * s.scale[1];
    const double nuz = (s.v0[2] + ((double)(j - jr * nvz) + 0.5) * s.dv[2]) * s.scale[2];
    cf[l][w] = box_coef<T>(l == 2 ? nuz : (l == 1 ? nuy : nux), l == 2 ? n2 : (l == 1 ? n1 : n0), periodic);
  }
  // A periodic line of one cell keeps its value: what enters is what leaves. Its
  // sweep can be left out but for values near overflow or not finite, where the
  // difference of the two fluxes is not zero.
  const bool ones = periodic && (n0 == 1 || n1 == 1 || n2 == 1);
  bool huge = false;
  auto look = [&](T v) { huge = huge || !(fabs(v) < T(0x1p1000)); };
  for (int e0 = tid; e0 < nvec; e0 += 4 * nth) {
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const int e = e0 + k * nth, w = (e & ((1 << lq) - 1)) << lgv;
      if (e < nvec && w < nw) {
        *reinterpret_cast<VT*>(L + place(e >> lq) + w) = x[k];
#pragma unroll
        for (int q = 0; q < V; q++) look(lane_of<VT, T>(x[k], q));
      }
    }
    fetch(e0 + 4 * nth);
  }
  if (!vec) {
    for (int e = tid; e < np << lgw; e += nth) {
      const int w = e & (W - 1);
      if (w < nw) {
        const T v = g[(long long)(e >> lgw) * nv3 + w];
        L[place(e >> lgw) + w] = v;
        look(v);
      }
    }
  }
  if (nw < W) {                      // the columns past the end take part in the sweeps as zeros
    for (int e = tid; e < np << lgw; e += nth) {
      const int w = e & (W - 1);
      if (w >= nw) L[place(e >> lgw) + w] = T(0);
    }
  }
  const bool skip = ones && __syncthreads_or(huge ? 1 : 0) == 0;
  if (!ones) __syncthreads();
#pragma unroll 1
  for (int ax = 2; ax >= 0; ax--) {
    // lines (i, j): x lines (y, z), y lines (x, z), z lines (x, y)
    if (skip && (ax == 0 ? n0 : (ax == 1 ? n1 : n2)) == 1) continue;
    const int n = ax == 0 ? n0 : (ax == 1 ? n1 : n2), st = ax == 0 ? sx : (ax == 1 ? sy : W);
    const int nq = ax == 0 ? n1 * n2 : (ax == 1 ? n0 * n2 : n0 * n1);
    box_sweep<T, NMAX>(L, red, n, st, nq << lgw, lgw, ax == 2 ? n1 : n2, ax == 0 ? sy : sx, ax == 2 ? sy : W, cf[ax],
                       periodic);
    __syncthreads();
  }
  if (vec) {
    const int lanes = 1 << lq;
    const int rounds = (nvec + nth - 1) / nth;
    for (int k = 0; k < rounds; k++) {
      const int e = tid + k * nth, w = (e & (lanes - 1)) << lgv;
      double acc = 0.0;
      if (e < nvec && w < nw) {
        const VT x = *reinterpret_cast<const VT*>(L + place(e >> lq) + w);
        *reinterpret_cast<VT*>(go + (long long)(e >> lq) * nv3 + w) = x;
#pragma unroll
        for (int q = 0; q < V; q++) acc += (double)lane_of<VT, T>(x, q);
      }
      if (part) {
        for (int o = lanes >> 1; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
        if (e < nvec && w == 0) part[(long long)chunk * np + (e >> lq)] = acc;
      }
    }
  } else {
    for (int e = tid; e < np << lgw; e += nth) {
      const int w = e & (W - 1);
      if (w < nw) go[(long long)(e >> lgw) * nv3 + w] = L[place(e >> lgw) + w];
    }
    if (part) {
      for (int cell = tid; cell < np; cell += nth) {
        const T* p = L + place(cell);
        double acc = 0.0;
        for (int w = 0; w < nw; w++) acc += (double)p[w];
        part[(long long)chunk * np + cell] = acc;
      }
    }
  }
}

// LDS row stride of nz cells of w values: = w (mod the 64 banks)
inline int box_sy(int nz, int w, int es)
{
  const int banks = 64 * 4 / es;   // elements of this size over the 64 banks
  const int s0 = nz * w;
  return s0 + (((w - s0) % banks) + banks) % banks;
}

inline size_t box_lds(int n0, int n1, int n2, int w, int es) { return (size_t)n0 * n1 * box_sy(n2, w, es) * es; }

template <typename T, int NMAX>
hipError_t launch_drift_box_n(const DriftBoxArgs& a, const DriftBoxShape& s, long long blocks, hipStream_t st)
{
  const size_t lds = box_lds(s.n[0], s.n[1], s.n[2], 1 << s.lgw, (int)sizeof(T));
  // two workgroups or more per CU where their boxes fit (one loads while
  // another sweeps), 16 waves where only one does
  int th = lds <= 16 * 1024 ? 256 : (lds <= 80 * 1024 ? 512 : 1024);
  if (th > box_threads<T, NMAX>()) th = box_threads<T, NMAX>();
  hipLaunchKernelGGL((drift_box<T, NMAX>), dim3((unsigned)blocks), dim3(th), lds, st, static_cast<const T*>(a.f),
                     static_cast<T*>(a.out ? a.out : const_cast<void*>(a.f)), s, a.part);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_drift_box_t(const DriftBoxArgs& a, int w, hipStream_t st)
{
  DriftBoxShape s{};
  for (int l = 0; l < 3; l++) s.n[l] = a.n[l];
  while ((1 << s.lgw) < w) s.lgw++;
  s.sy = box_sy(a.n[2], w, (int)sizeof(T));
  s.sx = a.n[1] * s.sy;
  s.periodic = a.periodic;
  s.nvy = a.nv[1];
  s.nvz = a.nv[2];
  s.nv3 = (int)a.nv3;
  s.nchunk = (int)((a.nv3 + w - 1) / w);
  for (int l = 0; l < 3; l++) {
    s.v0[l] = a.vmin[l];
    s.dv[l] = a.dv[l];
    s.scale[l] = a.scale[l];
  }
  const long long blocks = s.nchunk;
  const int G = w * (int)sizeof(T) >= 128 ? 1 : 128 / (w * (int)sizeof(T));
  s.xcd_group = G > 1 && blocks % (8 * G) == 0 ? G : 0;
  int m = s.n[0] > s.n[1] ? s.n[0] : s.n[1];
  m = s.n[2] > m ? s.n[2] : m;
  if (m <= 16) return launch_drift_box_n<T, 16>(a, s, blocks, st);
  if (m <= 32) return launch_drift_box_n<T, 32>(a, s, blocks, st);
  if (m <= 48) return launch_drift_box_n<T, 48>(a, s, blocks, st);
  if (m <= 64) return launch_drift_box_n<T, 64>(a, s, blocks, st);
  return launch_drift_box_n<T, 128>(a, s, blocks, st);
}

}  // namespace
}  // namespace vp
