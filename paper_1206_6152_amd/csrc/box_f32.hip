// box_f32.hip -- the run-time-shaped kick of box.h for FP32-stored f, the rules that
// choose the passes of box.h, and the reduction of their density sums.
#include <algorithm>

#include "box.h"

namespace vp {

hipError_t launch_kick_box_f64(const KickArgs& a, const int nv[3], hipStream_t s);
hipError_t launch_drift_box_f64(const DriftBoxArgs& a, int w, hipStream_t s);

namespace {

hipError_t launch_kick_box_f32(const KickArgs& a, const int nv[3], hipStream_t s)
{
  return launch_kick_box_t<float>(a, nv, s);
}

// rho[cell] = dv3 sum_k part[k np + cell]: a workgroup takes four cells (there
// are few: drift_box_cells takes up to 512), its 256 groups of lanes every 256th chunk with four sums
// in flight; the groups' sums are added in a tree. 64 cells of 6912 chunks took
// 43 us with eight groups and 32 cells per workgroup.
__global__ __launch_bounds__(1024) void box_density_kernel(double* rho, const double* part, int np, int nchunk,
                                                           double dv3)
{
  constexpr int G = 256;
  __shared__ double sh[G][4];
  const int c = threadIdx.x & 3, g = threadIdx.x >> 2, cell = blockIdx.x * 4 + c;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  if (cell < np) {
    const double* p = part + cell;
    int k = g;
    for (; k + 3 * G < nchunk; k += 4 * G) {
      s0 += p[(long long)k * np];
      s1 += p[(long long)(k + G) * np];
      s2 += p[(long long)(k + 2 * G) * np];
      s3 += p[(long long)(k + 3 * G) * np];
    }
    for (; k < nchunk; k += G) s0 += p[(long long)k * np];
  }
  sh[g][c] = (s0 + s1) + (s2 + s3);
  __syncthreads();
  for (int w = G / 2; w > 0; w >>= 1) {
    if (g < w) sh[g][c] += sh[g + w][c];
    __syncthreads();
  }
  if (g == 0 && cell < np) rho[cell] = sh[0][c] * dv3;
}

constexpr int kLdsMost = 152 * 1024;   // of 160 KiB, less the coefficients and the split lines' maxima

}  // namespace

// Lanes per velocity block: a line or two per lane, in whole waves; 16 waves where
// one block fills a CU. With no more blocks than CUs nothing else would use the
// other lanes: 1 x 32 x 64 FP32 on one cell took 12.3 us with one wave (three
// sweeps: 11.4) and takes 7.4 with four.
int kick_box_threads(int dtype, const int nv[3], long long np)
{
  const int es = dtype == 0 ? 4 : 8, nv3 = nv[0] * nv[1] * nv[2];
  const long long lds = (long long)nv[0] * nv[1] * (nv[2] | 1) * es;
  const int most = box_threads_most(std::max(nv[0], std::max(nv[1], nv[2])), es);
  int th = 1024;
  if (nv3 <= 2048) th = np <= 512 && nv3 >= 512 ? 256 : 64;
  else if (nv3 <= 6144) th = np <= 256 ? 512 : 256;
  else if (lds <= 80 * 1024 && np > 256) th = 512;
  return std::min(th, most);
}

// Cells that the busiest lane updates in a half kick (box_sweep's choices)
static int kick_box_chain(const int nv[3], int threads)
{
  const int nv3 = nv[0] * nv[1] * nv[2], most = std::min(threads, kBoxRed);
  int cells = 0;
  for (int l = 0; l < 3; l++) {
    const int n = nv[l], nl = nv3 / n;
    if (n >= 16 && nl * (n / 8) <= most) cells += nl * (n / 4) <= most ? 4 + 2 : 8 + 2;   // and the cells of the edges
    else cells += (nl + threads - 1) / threads * n;
  }
  return cells;
}

// Where the one-pass kick is the better choice than the three sweeps (us, three
// sweeps -> one pass; 3000 shapes of random axes and cells were timed, and none
// that this rule takes is more than 5 % slower):
// - A workgroup is started for every block, however small: on many cells of tiny
//   blocks that is the time (131 072 blocks of 2^3 FP32 14 -> 64, 49 152 of 4^3 FP64
//   26 -> 42; 8192 of either, and any number of blocks from 192 cells on, less).
// - On a few cells the sweeps take three launches' time, the pass that of a lane's
//   chain of cells (8 x 32 x 128 FP32 on two cells 13.7 -> 18.3 at 256, up to 1.5 times
//   the sweeps; up to 128 cells at most 1.05 of them, from 32 cells on 0.7 on average).
// - Lines of 96 and 128 cells that are not split over lanes leave most lanes without a
//   line and spill in FP64: 128 x 96 x 1 FP64 on 24^3 cells 1940 -> 2600, 12 x 2 x 128 FP32
//   on 24 576 368 -> 519; split ones take half of the sweeps' time on few cells, but the
//   kernel's registers hold eight blocks on a CU: 1 x 96 x 3 FP32 on 262 144 668 -> 859.
bool kick_box_supported(int dtype, const int nv[3], long long np)
{
  if ((size_t)nv[0] * nv[1] * (nv[2] | 1) * (dtype == 0 ? 4 : 8) > (size_t)kLdsMost) return false;
  if (nv[0] * nv[1] * nv[2] < 192 && np > 8192) return false;
  if (np >= 32 && np <= 256) return true;
  const int chain = kick_box_chain(nv, kick_box_threads(dtype, nv, np));
  if (np < 32) return chain <= 128;
  return std::max(nv[0], std::max(nv[1], nv[2])) <= 64 || (chain <= 64 && np <= 16384);
}

hipError_t launch_kick_box(const KickArgs& a, int dtype, const int nv[3], hipStream_t s)
{
  if (!kick_box_supported(dtype, nv, a.np) || (a.reps != 1 && a.reps != 2)) return hipErrorInvalidValue;
  return dtype == 0 ? launch_kick_box_f32(a, nv, s) : launch_kick_box_f64(a, nv, s);
}

// Velocity cells per workgroup of the one-pass drift of the grid n; 0 if the
// single sweeps (or the one-pass T_y T_z) are the better choice. The pass is
// bound by vector issue (index decoding and run-time strides) and LDS latency,
// so several workgroups have to share a CU: boxes of up to 40 KiB, with runs of
// 128 bytes, or of 64 that share their lines with a neighbour on the same XCD; up
// to 64 KiB where one or two workgroups per CU are all there are (8 x 8 x 6 x 4096
// cells FP64, us a drift, three sweeps -> one pass: 22.5 -> 16.9, with half the run
// 19.9; 8^3, 72 KiB, 22.2 -> 20.2, with half the run 18.0). FP64: 4^3 x 24^3 10.8 us
// (16.6), 8^3 x 32^3 97 (121), 6^3 x 48^3 144 (166). The sweeps it is left to:
// - beyond 256 MiB (8^3 x 64^3, two steps: 6.2 ms against 5.9), and longer axes from a
//   MiB on (8 x 12 x 4 x 48^3 347 against 312, 64 x 4 x 4 x 12^3 37 against 33);
// - more than 2304 workgroups of fewer than 48 cells each, whose start is the time
//   (96^3 on one cell 18 -> 110, on 2^3 67 -> 167, on 2 x 3 x 6 the same);
// - under a MiB, where latency is all (1D-1V 128 x 128: 6 us against three launches of
//   3 to 12) and 32-byte runs and up to 80 KiB serve: long axes with more than 384
//   cells, whose lines one or two workgroups take in turn (12^3 of one value 9.6 ->
//   14.3, 3 x 6 x 128 of two 15.6 -> 32).
//
// FP64 only: at 8^3 x 16^3 FP32 the pass with its sums took what the three sweeps
// take (15 + 4.5 us against 17 + 2.6).
int drift_box_cells(int dtype, const int n[3], long long nv3)
{
  if (dtype == 0) return 0;
  const int es = 8;
  const long long np = (long long)n[0] * n[1] * n[2];
  const long long bytes = np * nv3 * es;
  if ((n[0] > 8 || n[1] > 8 || n[2] > 8) && (bytes >= (1 << 20) || np > 384)) return 0;
  if (bytes > (1 << 28)) return 0;
  for (int run = 128; run >= 32; run /= 2) {
    const int w = run / es;
    const size_t lds = box_lds(n[0], n[1], n[2], w, es);
    const long long blocks = (nv3 + w - 1) / w;
    if (blocks > 2304 && np < 48) continue;
    if (lds <= 40 * 1024 && run >= 64 && blocks >= 256) return w;
    if (lds <= (run == 32 ? 80 : 64) * 1024 && blocks <= 512 && (blocks >= 256 || run == 32)) return w;
  }
  return 0;
}

hipError_t launch_drift_box(const DriftBoxArgs& a, int dtype, hipStream_t s)
{
  const int w = drift_box_cells(dtype, a.n, a.nv3);
  if (w == 0) return hipErrorInvalidValue;
  return launch_drift_box_f64(a, w, s);
}

hipError_t launch_box_density(double* rho, const double* part, long long np, long long nchunk, double dv3,
                              hipStream_t s)
{
  if (np <= 0) return hipSuccess;
  hipLaunchKernelGGL(box_density_kernel, dim3((unsigned)((np + 3) / 4)), dim3(1024), 0, s, rho, part, (int)np,
                     (int)nchunk, dv3);
  return hipGetLastError();
}

}  // namespace vp
