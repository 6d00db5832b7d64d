// adj_line.h -- the reverse of the one-line PFC update, shared by the reverse
// sweeps and the one-pass reverse half kick (the formulas are stated in
// adjoint.hip). Device code only.
#pragma once

#include "pfc_line.h"

namespace vp {
namespace {

// Coefficients of a reverse line update in the direction of its motion, |nu| =
// shift + alpha: c1, c2 as in the forward update, dc1 = d c1/d alpha and dc2 =
// d c2/d alpha.
template <typename T>
struct AdjCoef {
  T alpha, c1, c2, dc1, dc2;
  int shift;   // >= 0, below N when periodic
  bool neg;
};

template <typename T, int N>
__device__ __forceinline__ AdjCoef<T> adj_coef(double nu, bool periodic)
{
  const LineCoef<T> c = line_coef<T, N>(nu, periodic);
  const double a = fabs(nu), al = a - floor(a);
  return AdjCoef<T>{c.alpha, c.c1, c.c2, (T)((2.0 * al - 3.0) / 6.0), (T)(-al / 3.0), c.neg ? -c.shift : c.shift,
                    c.neg};
}

// One line in view order (along its motion): w the forward line, l in: the
// adjoint of the updated line before its shift (lam_g), out: the adjoint of w
// without f_inf's share. lfinf and lalpha receive f_inf's and alpha's adjoints
// (lalpha with ALPHA only).
// A corrector bound is active where the difference lies outside it. Cell i
// sends its own terms to out_i, its Lp interior-branch term to out_{i+1} and
// its Lm interior-branch term to out_{i-1}, so out_{i-1} is written once cell i
// is known. Every rounding step is written out, so all kernels agree bit for
// bit. 36 vector instructions per FP32 cell with alpha's adjoint, seven less without;
// a pass of its own for alpha's adjoint and a product per term took 41. Products
// merged per line (c1 alpha and the like) would leave 29, but other roundings: FP32
// gradients moved by up to 6e-9.
template <typename T, int N, bool ALPHA = true>
__device__ __forceinline__ void adj_core(const T (&w)[N], T (&l)[N], T finf, const AdjCoef<T>& k, bool periodic,
                                         T& lfinf, T& lalpha)
{
#pragma clang fp contract(off)
  const T twoinf = finf + finf;
  const T lg0 = l[0];
  T dm = periodic ? w[0] - w[N - 1] : w[0];
  T carry = T(0), pending = T(0), wrap_back = T(0);
  lfinf = T(0);
  lalpha = T(0);
#pragma unroll
  for (int i = 0; i < N; i++) {
    const T f0 = w[i];
    const T fr = (i + 1 < N) ? w[i + 1 < N ? i + 1 : 0] : (periodic ? w[0] : T(0));
    const T dp = fr - f0;
    const T h = f0 + f0;
    const T r = twoinf - h;
    const T lp = clamp_ordered(dp, -r, h);
    const T lm = clamp_ordered(dm, -h, r);
    const T lgi = l[i];
    const T lgn = (i + 1 < N) ? l[i + 1 < N ? i + 1 : 0] : (periodic ? lg0 : T(0));
    const T lF = lgn - lgi;                      // lam_F_i = lam_g_{i+1} - lam_g_i
    const T q = fma_(k.c2, lm, fma_(k.c1, lp, f0));
    if constexpr (ALPHA) lalpha = lalpha + lF * (q + k.alpha * (k.dc1 * lp + k.dc2 * lm));
    const T lin = k.alpha * lF;
    const T llp = k.c1 * lin;
    const T llm = k.c2 * lin;
    // tested on the bounds, not on what the clamps gave: those compares would wait
    // for the clamps (short FP32 lines 7 % slower, the 16^3 half kick 70 us for 65)
    const bool p_lo = dp < -r, p_hi = dp > h, m_lo = dm < -h, m_hi = dm > r;
    const bool p_mid = !(p_lo || p_hi), m_mid = !(m_lo || m_hi);
    T own = lgi + lin;
    own = fma_(llp, p_mid ? T(-1) : T(2), own);
    own = fma_(llm, m_mid ? T(1) : T(-2), own);
    own = own + carry;
    // the factor that a bound switches is lam's, not the constant: a cell without
    // its bound adds nothing, also where lam is infinite or not a number
    lfinf = fma_(p_lo ? llp : T(0), T(-2), lfinf);
    lfinf = fma_(m_hi ? llm : T(0), T(2), lfinf);
    // the two sums are kept up cell by cell: left to the compiler, both chains
    // move behind the loop, and every cell's operands live until then (24 FP32
    // cells: 168 registers and spills, 0.83 ms for the half kick's pass)
    if constexpr (ALPHA) asm volatile("" : "+v"(lfinf), "+v"(lalpha));
    const T back = m_mid ? -llm : T(0);
    if (i > 0) l[i > 0 ? i - 1 : 0] = pending + back;
    else wrap_back = back;
    pending = own;
    carry = p_mid ? llp : T(0);
    dm = dp;
  }
  l[N - 1] = pending + (periodic ? wrap_back : T(0));
  if (periodic) l[0] = l[0] + carry;
}

}  // namespace
}  // namespace vp
