// GELU (exact erf form) and its derivative for the forward epilogues of the bf16 kernels.  Plain C++ beside the two hardware
// approximations that are passed in, so that its error can be measured on the host.
#pragma once
#include <cmath>

#ifdef __HIPCC__
#define HBP_HD __host__ __device__ inline __attribute__((always_inline))
#else
#define HBP_HD inline
#endif

namespace hbp {

// z = a Phi(a) and its derivative Phi(a) + a phi(a), with phi the normal density; exp2 and rcp to one unit in the last place.
//   |a| < 5/4   Phi = 1/2 + a P(a^2): the odd part of Phi as a polynomial, so that its error shrinks with a
//   beyond      Phi(-u) = phi(u) m(u), u >= 0: m, the Mills ratio, is a polynomial in t = 1 / (1 + p u) without a constant term (the
//               form of Hastings' approximations), fitted on 5/4 <= u <= 14.5: the left tail keeps its relative accuracy,
//               which 1 + erf loses to cancellation
// P, m and p are least-squares fits, reweighted until the largest error was 2.2e-9 (P, relative to Phi) and 4.2e-8 (m, relative).
// One exponential serves phi and the tail.  About 34 vector operations per element, where erff and an exponential of its own
// are above 50: the epilogue of a 256 x 256 tile is bound by them.  Largest error on the device, this form / 1 + erff: z relative,
// for -1 < a < 0 2.0e-7 / 2.7e-7, for 0 < a < 1 1.2e-7 / 1.4e-7; the derivative, absolute, 1.4e-7 / 1.6e-7; smaller in every band in
// between.  (m alone, from 0 on, is worse around 0: Phi there carries the whole error of the exponential, the reciprocal and m,
// up to 7.7e-7 of z and 4.2e-7 of the derivative.)
template <typename Exp2, typename Rcp>
HBP_HD void gelu_pair(float a, float& z, float& dz, Exp2 exp2, Rcp rcp) {
  const float s = a * a, u = fabsf(a);
  const float f = 0.39894228040143267794f * exp2(s * -0.72134752044448170368f);
  const float t = rcp(fmaf(0.4072047472000122f, u, 1.0f));
  float m = 0.1842590868473053f;
  m = fmaf(m, t, -0.4753357768058777f);
  m = fmaf(m, t, 0.23867550492286682f);
  m = fmaf(m, t, 0.14314711093902588f);
  m = fmaf(m, t, 0.3503996431827545f);
  m = fmaf(m, t, 0.40620383620262146f);
  m = fmaf(m, t, 0.4072434604167938f);
  const float q = f * (m * t);
  float p = -6.652437150478363e-06f;
  p = fmaf(p, s, 0.0001103618778870441f);
  p = fmaf(p, s, -0.0011827675625681877f);
  p = fmaf(p, s, 0.009971545077860355f);
  p = fmaf(p, s, -0.06649000197649002f);
  p = fmaf(p, s, 0.3989422619342804f);
  const float tail = a > 0.f ? 1.0f - q : q;
  const float phi = u < 1.25f ? fmaf(a, p, 0.5f) : tail;
  dz = fmaf(a, f, phi);
  z = a * phi;
}

}  // namespace hbp
