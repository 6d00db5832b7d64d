// drift_pair.h -- two of the three position sweeps of Eq. (17) (Sec. 2.1 of
// Yoshikawa, Yoshida & Umemura) in one pass over f, for planes of two unequal
// or small axes. The line update is that of sweep.hip (pfc_line.h), so the pass
// rounds like the single sweeps. gfx950.
#pragma once
#include "vp_internal.h"

#include "pfc_line.h"

namespace vp {
namespace {

// A tile is W consecutive velocity cells of every cell of the (A, B) plane, at
// one index of the third axis. Lane (i, w) of the S x W lanes, S the shorter
// axis, holds the A lines of its velocity cell w at b = i, i + S, ..: they come
// from HBM in the orientation of their sweep, are updated in registers and
// parked in LDS at their b place in the orientation of the B sweep; after a
// barrier the lane takes the B lines of the same velocity cell at a' = i,
// i + S, .., updates them and writes them back. The lane keeps its velocity
// cell, so each tile's coefficients are worked out once per lane, under the
// loads. With sums (B = x) the new values go back to LDS in storage order and each
// (x, y) row of W values is added up in FP64 in a fixed order, over the 256
// velocity cells of a workgroup: the sums of sweep_strided<.., true>.
//
// Bound by loads in flight: 24 x 12 planes (32 x 24 x 16 cells, FP32, 0.68 GB)
// take 0.274 ms, a copy 0.22, the two single sweeps 0.49; 64 x 4 planes (64^3
// cells, 17.2 GB) 7.9 ms, where 64 KiB tiles leave two wavefronts on a SIMD.
// Wavefronts count for more than anything each has under way: with the next
// tile's lines prefetched under the B sweeps, and the registers for that, the
// first takes 0.38 ms and the second the same 7.9; one-line rows (W = 32) 0.30
// and 8.3.
// rows of one wave where two tiles of them fit a CU, else of one cache line
constexpr int pair_row(int es, int cells) { return es == 4 && cells <= 320 ? 64 : (cells <= 320 ? 256 : 128) / es; }
// rows of lanes: the shorter axis, in whole waves
constexpr int pair_rows(int least, int w) { return least * w % 64 == 0 ? least : (2 * least * w % 64 == 0 ? 2 * least : 4 * least); }

template <typename T, int NA, int NB>
struct PairShape {
  static constexpr int CELLS = NA * NB;
  static constexpr int W = pair_row(sizeof(T), CELLS);
  static constexpr int BYTES = CELLS * W * (int)sizeof(T);
  static constexpr int MIN = NA < NB ? NA : NB;
  static constexpr int S = pair_rows(MIN, W);
  static constexpr int THREADS = S * W;
  static constexpr int TILES = 256 / W;
  static constexpr int KA = (NB + S - 1) / S, KB = (NA + S - 1) / S;   // lines per lane
  // waves per SIMD: what the registers of one set of lines and the LDS allow
  static constexpr int LIVE = (KA * NA > KB * NB ? KA * NA : KB * NB) * (int)sizeof(T) / 4;
  // and what a wave needs beside them (measured): FP64 temporaries, and the more of
  // them the more lines a lane holds
  static constexpr bool EVEN = NA % S == 0 && NB % S == 0;
  static constexpr int TEMPS =
      sizeof(T) == 8 ? (KA * KB > 1 ? 64 + 3 * LIVE / 4 : 72) : (LIVE >= 32 && !EVEN ? 88 : 64);
  static constexpr int REGW = 512 / (LIVE + TEMPS), LDSW = 160 * 1024 / BYTES * THREADS / 256;
  static constexpr int WAVES = REGW < LDSW ? REGW : LDSW;
  static constexpr int LEAST = (THREADS + 255) / 256;                  // one workgroup
  static constexpr int WPE = WAVES < LEAST ? LEAST : (WAVES > 8 ? 8 : WAVES);
  // P lanes share a row's sum
  static constexpr int P0 = THREADS / CELLS;
  static constexpr int P = P0 >= 16 ? 16 : P0 >= 8 ? 8 : P0 >= 4 ? 4 : P0 >= 2 ? 2 : 1;
  static constexpr int RS = THREADS / P;                               // rows at a time
  static constexpr int R = (CELLS + RS - 1) / RS;
  static constexpr bool fits = BYTES <= 80 * 1024 && THREADS <= 1024;
};

template <typename T, int N>
__device__ __forceinline__ LineCoef<T> pair_coef(const DriftPairAxis& x, unsigned c, bool periodic, bool& neg)
{
  const unsigned j = (c / (unsigned)x.j_div) % (unsigned)x.j_mod;
  const double nu = (x.vmin + ((double)j + 0.5) * x.dv) * x.scale;
  neg = nu < 0.0;
  return line_coef<T, N>(fabs(nu), periodic);
}

template <typename T, int NA, int NB>
__global__ __launch_bounds__((PairShape<T, NA, NB>::THREADS))
__attribute__((amdgpu_waves_per_eu(PairShape<T, NA, NB>::WPE)))
void drift_pair(DriftPairArgs p)
{
  using H = PairShape<T, NA, NB>;
  constexpr int W = H::W, S = H::S;
  __shared__ T L[H::CELLS * W];   // [b][a][w]
  const int tid = threadIdx.x, i0 = W == 64 ? uniform(tid / W) : tid / W, w = tid - i0 * W;
  const unsigned nch = (unsigned)(p.nv3 / 256);
  const unsigned o = blockIdx.x / nch, ch = blockIdx.x - o * nch;
  const bool periodic = p.periodic != 0;
  T* row0 = static_cast<T*>(p.f) + o * p.so + ch * 256LL;
  // a wave that is one row whose velocity cells all move one way has one scalar
  // address per row; else the lanes carry their own
  auto one_way = [&](bool neg) {
    const unsigned long long m = __ballot(neg);
    return W == 64 && (m == 0 || m == ~0ull);
  };
  double acc[H::R];
#pragma unroll
  for (int k = 0; k < H::R; k++) acc[k] = 0.0;

  T v[H::KA][NA];
  auto load = [&](int t) {
    // only the sign of this tile's A sweep is needed to address its lines
    const unsigned c = ch * 256u + (unsigned)(t * W + w);
    const unsigned j = (c / (unsigned)p.a.j_div) % (unsigned)p.a.j_mod;
    const bool neg = (p.a.vmin + ((double)j + 0.5) * p.a.dv) * p.a.scale < 0.0;
    auto rows = [&](const T* q, long long st, auto at) {
      const long long jump = S * p.sb - NA * st;
#pragma unroll
      for (int k = 0; k < H::KA; k++) {
        if (NB % S != 0 && i0 + k * S >= NB) break;
#pragma unroll
        for (int r = 0; r < NA; r++) {
          v[k][r] = at(q);
          q += st;
        }
        q += jump;
      }
    };
    const T* q = row0 + t * W + i0 * p.sb;
    if (one_way(neg)) {
      const bool n = uniform((int)neg) != 0;
      rows(q + (n ? (NA - 1) * p.sa : 0), n ? -p.sa : p.sa, [&](const T* x) { return x[(unsigned)w]; });
    } else {
      rows(q + (neg ? (NA - 1) * p.sa : 0) + w, neg ? -p.sa : p.sa, [&](const T*& x) {
        const T y = *x;
        asm volatile("" : "+v"(x));   // one running address, not one per cell
        return y;
      });
    }
  };
#pragma unroll 1
  for (int t = 0; t < H::TILES; t++) {
    load(t);
    const unsigned c = ch * 256u + (unsigned)(t * W + w);
    bool na, nb;
    const LineCoef<T> ca = pair_coef<T, NA>(p.a, c, periodic, na);
    const LineCoef<T> cb = pair_coef<T, NB>(p.b, c, periodic, nb);
    const bool one = one_way(na) && one_way(nb);
#pragma unroll
    for (int k = 0; k < H::KA; k++) {
      const int b = i0 + k * S;
      if (NB % S != 0 && b >= NB) break;
      __builtin_amdgcn_sched_barrier(0);   // one line's temporaries at a time
      pfc_core<T, NA>(v[k], ca.alpha, ca.c1, ca.c2, periodic);
      T* l = L + (nb ? NB - 1 - b : b) * (NA * W) + w;
      store_shifted<T, NA>(v[k], ca.shift, periodic, [&](int r, T x) { l[r * W] = x; });
    }
    __syncthreads();
    T u[H::KB][NB];
#pragma unroll
    for (int k = 0; k < H::KB; k++) {
      const int a = i0 + k * S;
      if (NA % S != 0 && a >= NA) break;
#pragma unroll
      for (int r = 0; r < NB; r++) u[k][r] = L[(r * NA + a) * W + w];
    }
    __syncthreads();   // LDS takes the new values, or the next tile
#pragma unroll
    for (int k = 0; k < H::KB; k++) {
      const int a = i0 + k * S;
      if (NA % S != 0 && a >= NA) break;
      __builtin_amdgcn_sched_barrier(0);
      pfc_core<T, NB>(u[k], cb.alpha, cb.c1, cb.c2, periodic);
      const int ay = na ? NA - 1 - a : a;
      T* q = row0 + t * W + ay * p.sa + (nb ? (NB - 1) * p.sb : 0);
      const long long st = nb ? -p.sb : p.sb;
      if (one && cb.shift == 0) {
        T* x = row0 + t * W + (uniform((int)na) ? NA - 1 - a : a) * p.sa + (uniform((int)nb) ? (NB - 1) * p.sb : 0);
        const long long xs = uniform((int)nb) ? -p.sb : p.sb;
#pragma unroll
        for (int r = 0; r < NB; r++) {
          x[(unsigned)w] = u[k][r];
          x += xs;
        }
      } else if (cb.shift == 0) {
        q += w;
#pragma unroll
        for (int r = 0; r < NB; r++) {
          *q = u[k][r];
          q += st;
          asm volatile("" : "+v"(q));
        }
      } else {
        store_shifted<T, NB>(u[k], cb.shift, periodic, [&](int r, T x) { q[r * st + w] = x; });
      }
      if (p.part) {
        T* l = L + ((nb ? (NB - 1) * NA : 0) + ay) * W + w;
        const int ls = nb ? -NA * W : NA * W;
        store_shifted<T, NB>(u[k], cb.shift, periodic, [&](int r, T x) { l[r * ls] = x; });
      }
    }
    if (p.part) {
      __syncthreads();
      int rot = tid;                    // no two lanes of a wave on one bank
      asm volatile("" : "+v"(rot));     // places worked out here, not kept over the loop
#pragma unroll
      for (int k = 0; k < H::R; k++) {
        const int row = tid / H::P + k * H::RS;
        if (row < H::CELLS) {
#pragma unroll 8
          for (int j = 0; j < W / H::P; j++) acc[k] += (double)L[row * W + ((j * H::P + rot) & (W - 1))];
        }
      }
      __syncthreads();
    }
  }
  if (p.part) {
#pragma unroll
    for (int k = 0; k < H::R; k++) {
#pragma unroll
      for (int s = H::P / 2; s > 0; s >>= 1) acc[k] += __shfl_xor(acc[k], s, 64);
      const int row = tid / H::P + k * H::RS;
      if (row < H::CELLS && tid % H::P == 0) {
        const int b = row / NA, a = row - b * NA;
        p.part[((long long)(a * p.nouter + (int)o) * nch + ch) * NB + b] = acc[k];
      }
    }
  }
}

template <typename T, int NA, int NB>
hipError_t launch_pair(const DriftPairArgs& p, hipStream_t s)
{
  using H = PairShape<T, NA, NB>;
  static_assert(H::fits && 256 % H::W == 0 && H::THREADS % 64 == 0 && 64 % H::P == 0, "tile");
  hipLaunchKernelGGL((drift_pair<T, NA, NB>), dim3((unsigned)(p.nouter * (p.nv3 / 256))), dim3(H::THREADS), 0, s, p);
  return hipGetLastError();
}

// The planes with a kernel: up to 576 cells (two tiles of 128-byte runs on a
// CU) of two of these lengths, but FP64 of 6 and 64, where a lane's lines leave room
// for one wave on a SIMD (384 to 1152 workgroups: 0.9 to 1.4 times the two sweeps).
constexpr bool pair_plane(int es, int na, int nb)
{
  return na * nb <= 576 && !(es == 8 && na * nb == 384 && (na == 64 || nb == 64));
}

template <typename T, int NA>
hipError_t launch_a(const DriftPairArgs& p, int nb, hipStream_t s)
{
  switch (nb) {
#define CASE(N) \
  case N: \
    if constexpr (pair_plane(sizeof(T), NA, N)) return launch_pair<T, NA, N>(p, s); \
    break;
    CASE(4) CASE(6) CASE(8) CASE(12) CASE(16) CASE(24) CASE(32) CASE(48) CASE(64)
#undef CASE
    default: break;
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_pair_t(const DriftPairArgs& p, int na, int nb, hipStream_t s)
{
  switch (na) {
#define CASE(N) \
  case N: return launch_a<T, N>(p, nb, s);
    CASE(4) CASE(6) CASE(8) CASE(12) CASE(16) CASE(24) CASE(32) CASE(48) CASE(64)
#undef CASE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_drift_pair_f32(const DriftPairArgs& p, int na, int nb, hipStream_t s);
hipError_t launch_drift_pair_f64(const DriftPairArgs& p, int na, int nb, hipStream_t s);

}  // namespace vp
