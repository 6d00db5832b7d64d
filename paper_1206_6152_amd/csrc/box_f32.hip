// box_f32.hip -- the run-time-shaped passes of box.h for FP32-stored f, the
// rules that choose them, and the reduction of their density sums.
#include "box.h"

namespace vp {

hipError_t launch_kick_box_f64(const KickArgs& a, const int nv[3], hipStream_t s);
hipError_t launch_drift_box_f64(const DriftBoxArgs& a, int w, hipStream_t s);

namespace {

hipError_t launch_kick_box_f32(const KickArgs& a, const int nv[3], hipStream_t s)
{
  return launch_kick_box_t<float>(a, nv, s);
}

hipError_t launch_drift_box_f32(const DriftBoxArgs& a, int w, hipStream_t s)
{
  return launch_drift_box_t<float>(a, w, s);
}

// rho[cell] = dv3 sum_k part[k np + cell]: a workgroup takes 32 cells, its
// eight rows of lanes every eighth chunk; the eight sums are added in order.
__global__ __launch_bounds__(256) void box_density_kernel(double* rho, const double* part, long long np,
                                                          long long nchunk, double dv3)
{
  __shared__ double sh[8][32];
  const int c = threadIdx.x & 31, g = threadIdx.x >> 5;
  const long long cell = (long long)blockIdx.x * 32 + c;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  if (cell < np) {
    const double* p = part + cell;
    long long k = g;
    for (; k + 24 < nchunk; k += 32) {
      s0 += p[k * np];
      s1 += p[(k + 8) * np];
      s2 += p[(k + 16) * np];
      s3 += p[(k + 24) * np];
    }
    for (; k < nchunk; k += 8) s0 += p[k * np];
  }
  sh[g][c] = (s0 + s1) + (s2 + s3);
  __syncthreads();
  if (g == 0 && cell < np) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < 8; i++) t += sh[i][c];
    rho[cell] = t * dv3;
  }
}

constexpr int kLdsMost = 152 * 1024;   // of 160 KiB, less the coefficients and the split lines' maxima

}  // namespace

bool kick_box_supported(int dtype, const int nv[3])
{
  return (size_t)nv[0] * nv[1] * (nv[2] | 1) * (dtype == 0 ? 4 : 8) <= (size_t)kLdsMost;
}

hipError_t launch_kick_box(const KickArgs& a, int dtype, const int nv[3], hipStream_t s)
{
  if (!kick_box_supported(dtype, nv) || (a.reps != 1 && a.reps != 2)) return hipErrorInvalidValue;
  return dtype == 0 ? launch_kick_box_f32(a, nv, s) : launch_kick_box_f64(a, nv, s);
}

// Velocity cells per workgroup of the one-pass drift of the grid n; 0 if the
// single sweeps (or the one-pass T_y T_z) are the better choice. The pass is
// bound by vector issue and LDS latency, so several workgroups have to share a
// CU: boxes of up to 40 KiB, with runs of 128 bytes, or of 64 that share their
// lines with a neighbour on the same XCD. 8^3 x 32^3 FP32: 50 us with 64-byte
// runs (37 KiB), 56 with 128 (73 KiB), 69 for the three sweeps; 12^3 x 24^3 in
// one workgroup per CU (110 KiB) 97 us against 87. Launches of at most 512
// workgroups are bound by latency and not by their lines: 32-byte runs and up to
// 80 KiB serve them (8^3 x 16^3 FP32: 11.4 us against 13.7, and two launches
// fewer in a step).
//
// FP64 only: the pass sums the density in another order than the x sweep, whose
// sums FP32 gradients were differentiated with. A last bit of the acceleration
// can move the rounding of a line's alpha to FP32, and a corrector switch behind
// it; and at 8^3 x 16^3 FP32 the pass with its sums took what the three sweeps
// take (15 + 4.5 us against 17 + 2.6).
int drift_box_cells(int dtype, const int n[3], long long nv3)
{
  if (dtype == 0) return 0;
  const int es = dtype == 0 ? 4 : 8;
  for (int run = 128; run >= 32; run /= 2) {
    const int w = run / es;
    const size_t lds = box_lds(n[0], n[1], n[2], w, es);
    const long long blocks = (nv3 + w - 1) / w;
    if (lds <= 40 * 1024 && run >= 64 && blocks >= 256) return w;
    if (lds <= 80 * 1024 && blocks <= 512 && (blocks >= 256 || run == 32)) return w;
  }
  return 0;
}

hipError_t launch_drift_box(const DriftBoxArgs& a, int dtype, hipStream_t s)
{
  const int w = drift_box_cells(dtype, a.n, a.nv3);
  if (w == 0) return hipErrorInvalidValue;
  return dtype == 0 ? launch_drift_box_f32(a, w, s) : launch_drift_box_f64(a, w, s);
}

hipError_t launch_box_density(double* rho, const double* part, long long np, long long nchunk, double dv3,
                              hipStream_t s)
{
  if (np <= 0) return hipSuccess;
  hipLaunchKernelGGL(box_density_kernel, dim3((unsigned)((np + 31) / 32)), dim3(256), 0, s, rho, part, np, nchunk, dv3);
  return hipGetLastError();
}

}  // namespace vp
