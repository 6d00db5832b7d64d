// kick_adjoint.hip -- the reverse of one half kick T_vz T_vy T_vx in one pass
// over the velocity blocks (the reverse line update is that of adj_line.h, its
// formulas are stated in adjoint.hip). gfx950.
#include "adj_line.h"
#include "vec16.h"
#include "vp_internal.h"

namespace vp {
namespace {

// The adjoint of T_vz T_vy T_vx (tau) for velocity blocks that fit the LDS, one
// copy at a time. Each lane holds one line of the forward state (w) and of the
// adjoint (l) in registers; the block's one LDS buffer only changes their
// orientation (rows padded to N + 1, planes to SX = N (mod 64)):
//   x (vx lines, from HBM) -> T_vx -> LDS -> T_vy -> LDS -> w along vz
//   lam (from HBM)         -> LDS -> l along vz; vz reverse -> LDS -> l along vy
//   x (vx lines, from L2)  -> T_vx -> LDS -> w along vy; vy reverse
//   l                      -> LDS -> l along vx; w = x (vx lines, from L2);
//                             vx reverse -> HBM
// against twelve passes over HBM for two regenerated states and three separate
// reverse sweeps. Holding both blocks in LDS left one workgroup on a CU (9 waves
// on 4 SIMDs for 24^3 FP32); with one buffer two share it, and one's loads and
// barriers run under the other's arithmetic.
//
// All lines of a block along one axis move with one Courant number: its
// coefficients are worked out once per block (three lanes, while the first
// loads are in flight), and each axis is held in LDS in the orientation of its
// motion, so that the updates need no selects for the direction and a
// whole-cell shift is a uniform branch. 16^3 x 24^3 FP32 takes 0.376 ms instead of
// 0.50. The vector units are busy for 0.62 of that (162 instructions per cell for six
// sweeps); what is left are the loads and LDS accesses between the barriers, which
// two workgroups on a CU hide in part. The per-line results are the same bits as those
// of the single reverse sweeps, and the nu adjoints are added per axis in the order of
// reduce_lines_kernel.
template <typename T, int N>
struct AdjKickShape {
  static constexpr int SY = N + 1;
  static constexpr int SX0 = N * SY;
  static constexpr int SX = SX0 + ((((N - SX0) % 64) + 64) % 64);
  static constexpr int ELEMS = N * SX;
  static constexpr int LINES = N * N;
  // at least 256 lanes: the reduction below runs the 256-lane tree of reduce_lines_kernel
  static constexpr int THREADS = (LINES + 63) / 64 * 64 > 256 ? (LINES + 63) / 64 * 64 : 256;
  // the block, or at the end the line adjoints and their tree
  static constexpr int RED = (3 * LINES + 3 * 256) * 8;
  static constexpr int BYTES = ELEMS * (int)sizeof(T) > RED ? ELEMS * (int)sizeof(T) : RED;
  static constexpr bool fits = BYTES <= 156 * 1024 && THREADS <= 1024 && N % (16 / (int)sizeof(T)) == 0;
};

template <typename T>
__device__ __forceinline__ AdjCoef<T> uniform(const AdjCoef<T>& c)
{
  AdjCoef<T> k;
  k.alpha = uniform(c.alpha);
  k.c1 = uniform(c.c1);
  k.c2 = uniform(c.c2);
  k.dc1 = uniform(c.dc1);
  k.dc2 = uniform(c.dc2);
  k.shift = uniform(c.shift);
  k.neg = false;
  return k;
}

// f_inf of a line in view order and the first storage cell that holds it, as a
// view index (neg: storage order is the reverse of the view); -1 on an empty line
template <typename T, int N>
__device__ __forceinline__ int first_max(const T (&w)[N], bool neg, T& finf)
{
  finf = T(0);
#pragma unroll
  for (int r = 0; r < N; r++) finf = max_(finf, w[r]);
  int am = 0;
  if (neg) {
#pragma unroll
    for (int r = 0; r < N; r++) am = w[r] == finf ? r : am;
  } else {
#pragma unroll
    for (int r = N - 1; r >= 0; r--) am = w[r] == finf ? r : am;
  }
  return finf > T(0) ? am : -1;
}

// The shift's transpose in view order, lam_g_r = lam_out_{r+m}, zero past the
// outflow end, of a line at p + r st in LDS. A shift is uniform over the block.
template <typename T, int N>
__device__ __forceinline__ void read_lam(T (&l)[N], const T* p, int st, int m)
{
  if (m == 0) {
#pragma unroll
    for (int r = 0; r < N; r++) l[r] = p[r * st];
  } else {
#pragma unroll
    for (int r = 0; r < N; r++) {
      const int j = r + m < N ? r + m : N - 1;
      const T x = p[j * st];
      l[r] = r + m < N ? x : T(0);
    }
  }
}

template <typename T, int N>
__global__ __launch_bounds__((AdjKickShape<T, N>::THREADS)) void kick_adj_block(KickAdjArgs a)
{
  using S = AdjKickShape<T, N>;
  using VT = typename Vec16<T>::type;
  constexpr int V = Vec16<T>::n;
  constexpr int NVEC = N * N * N / V;
  constexpr int SX = S::SX, SY = S::SY;
  __shared__ __align__(16) char lds[S::BYTES];
  __shared__ LineCoef<T> fc[3];      // forward coefficients (with |nu|)
  __shared__ AdjCoef<T> rc[3];
  T* L = reinterpret_cast<T*>(lds);
  const int tid = threadIdx.x;
  const long long s = blockIdx.x;
  const T* xg = static_cast<const T*>(a.fin) + s * (long long)(N * N * N);
  T* lg = static_cast<T*>(a.lam) + s * (long long)(N * N * N);
  const double nux = a.accel[0][s] * a.scale[0], nuy = a.accel[1][s] * a.scale[1], nuz = a.accel[2][s] * a.scale[2];
  const bool rx = nux < 0.0, ry = nuy < 0.0, rz = nuz < 0.0;
  const bool on = tid < S::LINES;    // the lanes with a line
  const int o = tid / N, i = tid - o * N;
  const int px = (ry ? N - 1 - o : o) * SY + (rz ? N - 1 - i : i);   // vx line of storage (vy, vz) = (o, i), its LDS place
  const int py = o * SX + i, pz = o * SX + i * SY;                   // vy line of LDS (vx, vz), vz line of LDS (vx, vy)
  // the vx line of storage (o, i), in the order of its motion
  auto load_x = [&](T (&v)[N]) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < N; r++) v[r] = xg[(rx ? N - 1 - r : r) * (N * N) + tid];
  };
  auto forward_x = [&]() __attribute__((always_inline)) {            // T_vx of x, to LDS
    T v[N];
    load_x(v);
    pfc_core<T, N>(v, uniform(fc[0].alpha), uniform(fc[0].c1), uniform(fc[0].c2), false);
    store_shifted<T, N>(v, uniform(fc[0].shift), false, [&](int r, T x) { L[px + r * SX] = x; });
  };
  if (tid < 3) {
    const double nu = tid == 0 ? nux : (tid == 1 ? nuy : nuz);
    fc[tid] = line_coef<T, N>(fabs(nu), false);
    rc[tid] = adj_coef<T, N>(nu, false);
  }
  __syncthreads();
  if (on) forward_x();
  __syncthreads();
  if (on) {
    T v[N];
#pragma unroll
    for (int r = 0; r < N; r++) v[r] = L[py + r * SY];
    pfc_core<T, N>(v, uniform(fc[1].alpha), uniform(fc[1].c1), uniform(fc[1].c2), false);
    store_shifted<T, N>(v, uniform(fc[1].shift), false, [&](int r, T x) { L[py + r * SY] = x; });
  }
  __syncthreads();
  T w[N], l[N], finf, lfinf, lalpha;
  double dnx = 0.0, dny = 0.0, dnz = 0.0;
  if (on) {
#pragma unroll
    for (int r = 0; r < N; r++) w[r] = L[pz + r];
  }
  __syncthreads();
  // lam to LDS, 16 bytes per load and up to four loads in flight per lane (w
  // occupies N registers meanwhile)
  {
    constexpr int PER = (NVEC + S::THREADS - 1) / S::THREADS, U = PER < 4 ? PER : 4;
    const int dz = rz ? -1 : 1;
#pragma unroll
    for (int j0 = 0; j0 < PER; j0 += U) {
      VT x[U];
#pragma unroll
      for (int j = 0; j < U; j++) {
        const int k = tid + (j0 + j) * S::THREADS;
        if (j0 + j < PER && k < NVEC) x[j] = reinterpret_cast<const VT*>(lg)[k];
      }
#pragma unroll
      for (int j = 0; j < U; j++) {
        const int k = tid + (j0 + j) * S::THREADS;
        if (j0 + j < PER && k < NVEC) {
          const int e = k * V, jz = e % N, jy = (e / N) % N, jx = e / (N * N);
          T* p = L + (rx ? N - 1 - jx : jx) * SX + (ry ? N - 1 - jy : jy) * SY + (rz ? N - 1 - jz : jz);
#pragma unroll
          for (int q = 0; q < V; q++) p[q * dz] = lane_of<VT, T>(x[j], q);
        }
      }
    }
  }
  __syncthreads();
  if (on) {   // vz reverse
    const AdjCoef<T> k = uniform(rc[2]);
    read_lam<T, N>(l, L + pz, 1, k.shift);
    const int am = first_max<T, N>(w, rz, finf);
    adj_core<T, N>(w, l, finf, k, false, lfinf, lalpha);
    dnz = rz ? -(double)lalpha : (double)lalpha;
#pragma unroll
    for (int r = 0; r < N; r++) L[pz + r] = l[r];
    if (am >= 0) L[pz + am] += lfinf;
  }
  __syncthreads();
  if (on) read_lam<T, N>(l, L + py, SY, uniform(rc[1].shift));
  __syncthreads();
  if (on) forward_x();
  __syncthreads();
  if (on) {   // vy reverse
#pragma unroll
    for (int r = 0; r < N; r++) w[r] = L[py + r * SY];
    const int am = first_max<T, N>(w, ry, finf);
    adj_core<T, N>(w, l, finf, uniform(rc[1]), false, lfinf, lalpha);
    dny = ry ? -(double)lalpha : (double)lalpha;
    // the line's own places, which no other lane reads
#pragma unroll
    for (int r = 0; r < N; r++) L[py + r * SY] = l[r];
    if (am >= 0) L[py + am * SY] += lfinf;
  }
  __syncthreads();
  if (on) {   // vx reverse, straight to HBM
    load_x(w);
    const AdjCoef<T> k = uniform(rc[0]);
    read_lam<T, N>(l, L + px, SX, k.shift);
    const int am = first_max<T, N>(w, rx, finf);
    adj_core<T, N>(w, l, finf, k, false, lfinf, lalpha);
    dnx = rx ? -(double)lalpha : (double)lalpha;
#pragma unroll
    for (int r = 0; r < N; r++) lg[(rx ? N - 1 - r : r) * (N * N) + tid] = r == am ? l[r] + lfinf : l[r];
  }
  // lam_a[l][s] += scale_l * sum of the block's line adjoints, in the order of
  // reduce_lines_kernel: lane t < 256 adds lines t, t + 256, ... (in storage
  // order), then a tree (the three axes' trees side by side, with the same
  // pairs as each alone)
  if (!a.lam_a[0]) return;   // uniform: no acceleration adjoint wanted
  __syncthreads();
  double* dn = reinterpret_cast<double*>(lds);             // [3][LINES]
  double* sh = dn + 3 * S::LINES;                          // [3][256]
  if (on) {
    const int so = rx ? N - 1 - o : o;                     // storage vx of the vy and vz lines
    dn[tid] = dnx;
    dn[S::LINES + so * N + (rz ? N - 1 - i : i)] = dny;
    dn[2 * S::LINES + so * N + (ry ? N - 1 - i : i)] = dnz;
  }
  __syncthreads();
  if (tid < 256) {
#pragma unroll
    for (int q = 0; q < 3; q++) {
      double acc = 0.0;
      for (int j = tid; j < S::LINES; j += 256) acc += dn[q * S::LINES + j];
      sh[q * 256 + tid] = acc;
    }
  }
  __syncthreads();
  for (int w2 = 128; w2 > 0; w2 >>= 1) {
    if (tid < w2) {
#pragma unroll
      for (int q = 0; q < 3; q++) sh[q * 256 + tid] += sh[q * 256 + tid + w2];
    }
    __syncthreads();
  }
  if (tid < 3) a.lam_a[tid][s] += a.scale[tid] * sh[tid * 256];
}

template <typename T, int N>
hipError_t launch_kick_adj_n(const KickAdjArgs& a, hipStream_t s)
{
  using S = AdjKickShape<T, N>;
  static_assert(S::fits, "the velocity block does not fit the LDS");
  if (a.np <= 0) return hipSuccess;
  hipLaunchKernelGGL((kick_adj_block<T, N>), dim3((unsigned)a.np), dim3(S::THREADS), 0, s, a);
  return hipGetLastError();
}

}  // namespace

// Cubic velocity blocks that fit the LDS: FP32 up to 32^3, FP64 up to 24^3.
bool kick_adjoint_supported(int dtype, const int nv[3])
{
  if (nv[0] != nv[1] || nv[1] != nv[2]) return false;
  const int n = nv[0];
  return n == 8 || n == 16 || n == 24 || (dtype == 0 && n == 32);
}

hipError_t launch_kick_adjoint(const KickAdjArgs& a, int dtype, const int nv[3], hipStream_t s)
{
  if (!kick_adjoint_supported(dtype, nv)) return hipErrorInvalidValue;
  if (dtype == 0) {
    switch (nv[0]) {
      case 8: return launch_kick_adj_n<float, 8>(a, s);
      case 16: return launch_kick_adj_n<float, 16>(a, s);
      case 24: return launch_kick_adj_n<float, 24>(a, s);
      default: return launch_kick_adj_n<float, 32>(a, s);
    }
  }
  switch (nv[0]) {
    case 8: return launch_kick_adj_n<double, 8>(a, s);
    case 16: return launch_kick_adj_n<double, 16>(a, s);
    default: return launch_kick_adj_n<double, 24>(a, s);
  }
}

}  // namespace vp
