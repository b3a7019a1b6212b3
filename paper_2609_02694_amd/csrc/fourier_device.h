// Device building blocks of the Fourier kernels (internal).
#pragma once
#include "kernels.h"

namespace rbe {

// sin and cos of 2 pi u / N, N = kTurnTable, where u = m . (N s) is the phase
// of mode m at fractional coordinate s in N-ths of a turn (either factor may
// carry the N, a power of two: the scaling is exact). j = rint(u), taken by
// adding 1.5 2^52 (|u| is far below 2^51, and the sum's low bits are j mod N),
// and f = u - j are exact, so whole turns leave no rounding. The sine and
// cosine of theta = 2 pi f / N in [-pi/N, pi/N] are Taylor polynomials in f of
// degrees 5 and 6 (truncation below 1e-17 for N = 256), combined with the
// table's (sin, cos) of 2 pi j / N by the angle-addition formulas. tab is the
// table in LDS. Bound by FP64 issue (a fused multiply-add 4.6 cycles a wave):
// 19 FP64 operations a term with the dot product and two sums. As 22, with a
// conversion and the reduction to one turn first, 2M ions and 100 modes took 245
// (sums) and 177 us (gather); now 228 and 154.
constexpr int kTurnTable = kTurnTableEntries;
__device__ inline double phase_dot(double mx, double my, double mz, double sx, double sy, double sz) {
  return fma(mx, sx, fma(my, sy, mz * sz));
}
__device__ inline void sincos_phase_f64(double u, const double2 *tab, double *sn, double *cs) {
  constexpr double w = 6.283185307179586 / kTurnTable, w2 = w * w;
  const double big = u + 6755399441055744.0;  // 1.5 2^52
  const double f = u - (big - 6755399441055744.0);
  const double f2 = f * f;
  const double s = f * fma(f2, fma(f2, w * w2 * w2 / 120.0, -w * w2 / 6.0), w);
  const double c = fma(f2, fma(f2, fma(f2, -w2 * w2 * w2 / 720.0, w2 * w2 / 24.0), -0.5 * w2), 1.0);
  const double2 e = tab[__double2loint(big) & (kTurnTable - 1)];  // (sin, cos) of 2 pi j / N
  *sn = fma(e.x, c, e.y * s);
  *cs = fma(e.y, c, -(e.x * s));
}

// Phase of mode m at fractional coordinate s as an FP32 argument of the
// hardware sin/cos, which take turns: the dot product in FP64 with fused
// multiply-adds; any representative of m . s mod 1 serves, so the reduction is the
// fractional part in [0, 1) (one instruction), then rounded to FP32 (at most
// 2^-25 turns off).
__device__ inline float turn_f32(double mx, double my, double mz, double sx, double sy, double sz) {
  const double t = fma(mx, sx, fma(my, sy, mz * sz));
  return (float)__builtin_amdgcn_fract(t);
}

// Kahan-compensated FP32 sum of products: sum += a b, with the product
// fused into the compensation step (one rounding instead of two).
__device__ inline void kahan_fma(float &sum, float &comp, float a, float b) {
#pragma clang fp contract(off)
  const float y = fmaf(a, b, -comp);
  const float t = sum + y;
  comp = (t - sum) - y;
  sum = t;
}

// FP32 copies of a mode's gather coefficients.
__device__ inline void gather_floats(GatherMode &gm) {
  gm.af = (float)gm.a;
  gm.bf = (float)gm.b;
  gm.mxf = (float)gm.mx;
  gm.myf = (float)gm.my;
  gm.mzf = (float)gm.mz;
  gm.pad = 0.f;
}

// Kahan-compensated FP32 sum.
__device__ inline void kahan_add(float &sum, float &comp, float v) {
#pragma clang fp contract(off)
  const float y = v - comp;
  const float t = sum + y;
  comp = (t - sum) - y;
  sum = t;
}

}  // namespace rbe
