// fv_start.h -- binary32 start of the implied-volatility iteration.
//
// The four-region guess and the iteration's first step only have to bring
// the root near (the guess lands ~1e-2 from it, the step ~1e-6; the step
// that decides the root is in binary64, fv_lbr.h), so both run in binary32:
// the hardware reciprocals, square roots, 2^x and log2 x are single
// instructions there where binary64 refines or expands each one, and a
// polynomial step takes its constant as a 32-bit literal where binary64
// first moves it into a register pair.  Per quote of the wide workload the
// binary64 guess and first step took 640 vector and 270 scalar
// instructions; these take about 260 and 40.
//
// Binary32 cannot hold b itself deep in a wing, so everything is scaled by
// the bound b_max = e^{x/2}: bh = b/b_max in (0, 1) and
//   b'/b_max = e^{-g^2/2}/sqrt(2 pi),  g = h + t
// (h = x/s, t = s/2; h t = x/2 cancels in the exponent), with ratios to b'
// in place of values and logarithms in place of the values that leave the
// range.  Domain (scaled_domain, fv_lbr.h): |x| zero or in [2^-60, 128], bh
// above 2^-960, 1 - bh above 2^-40; a quote outside it, or whose iteration
// does not settle, takes the binary64 path.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fv_coeffs.h"

namespace fv {
namespace s32 {

constexpr float kInvSqrt2 = 0.70710678118654752f;
constexpr float kSqrt2 = 1.41421356237309505f;
constexpr float kInvSqrt3 = 0.57735026918962576f;
constexpr float kInvSqrt2Pi = 0.39894228040143268f;
constexpr float kSqrt2Pi = 2.50662827463100050f;
constexpr float kSqrtPi = 1.77245385090551603f;
constexpr float kSqrtPiOver2 = 1.25331413731550025f;
constexpr float kTwoOverSqrtPi = 1.12837916709551257f;
constexpr float kLnSqrt2Pi = 0.91893853320467274f;
constexpr float kLog2Sqrt2Pi = 1.32574806473616065f;
constexpr float kLog2E = 1.44269504088896341f;
constexpr float kLn2 = 0.69314718055994531f;
constexpr float kCl = 1.20919957615614523f;  // 2 pi/(3 sqrt3)

__host__ __device__ inline float rcp(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rcpf(x);
#else
  return 1.0f / x;
#endif
}
__host__ __device__ inline float sqrt(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_sqrtf(x);
#else
  return sqrtf(x);
#endif
}
__host__ __device__ inline float exp2(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_exp2f(x);
#else
  return exp2f(x);
#endif
}
__host__ __device__ inline float log2(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_logf(x);
#else
  return log2f(x);
#endif
}
__host__ __device__ inline float exp(float x) { return exp2(x * kLog2E); }
__host__ __device__ inline float log(float x) { return log2(x) * kLn2; }
// sqrt(2 pi) e^x and e^-x/sqrt(2 pi), the factor in the exponent
__host__ __device__ inline float exp_sqrt2pi(float x) { return exp2(fmaf(x, kLog2E, kLog2Sqrt2Pi)); }
__host__ __device__ inline float exp_over_sqrt2pi(float x) {
  return exp2(fmaf(-x, kLog2E, -kLog2Sqrt2Pi));
}
// ln of a positive normal binary64 number of any exponent
__host__ __device__ inline float log_of(double v) {
  int e;
  const float m = (float)frexp(v, &e);
  return (log2(m) + (float)e) * kLn2;
}

__host__ __device__ inline float log_of(float v) { return log(v); }

constexpr float kZ0 = (float)coef::kErfcxZ0;
// erfcx(z), z >= -1/2, by the guess's fit (6e-4)
constexpr int kSDeg = (int)(sizeof(coef::kErfcxS) / sizeof(double)) - 1;
constexpr int kTDeg = (int)(sizeof(coef::kErfcxT) / sizeof(double)) - 1;
constexpr int kFDeg = (int)(sizeof(coef::kErfcxF32) / sizeof(double)) - 1;

__host__ __device__ inline float erfcx(float z) {
  constexpr float kB = (float)coef::kErfcxSB;
  const float R = rcp(z + kB);
  const float y = fmaf(-2.0f * (kB - kZ0), R, 1.0f);
  float p = (float)coef::kErfcxS[kSDeg];
#pragma unroll
  for (int i = kSDeg - 1; i >= 0; --i) p = fmaf(p, y, (float)coef::kErfcxS[i]);
  return p * R;
}

// The normalised Black function at s, as ratios to b' (fv_math.h has the
// two forms), by the erfcx fit of degree 4 for the guess (6e-4, its derivative
// 1e-2: far within the few percent the guess is off; the caller knows the
// form), of degree 9 for the binary32 steps (4e-7, 7e-6: they land as near),
// or of degree 13 for the binary32 solver's own residual (6e-10).
//
// Everything is in hq = |h|/sqrt2 and tq = t/sqrt2, in which the erfcx
// arguments are q1 = hq - tq = -g/sqrt2 and q2 = hq + tq, and with them
//   g^2/2 = q1^2,  s b''/b' = h^2 - t^2 = 2 q1 q2.
// The fits' coefficients carry the factor sqrt(pi/2).
struct Eval {
  float is, hq, tq;  // 1/s, |h|/sqrt2, s/(2 sqrt2)
  float g2;          // g^2/2: b'/b_max = e^{-g2}/sqrt(2 pi)
  float H;           // s b''/b'
  float rho;         // b/b' in the difference form, (b_max - b)/b' in the complement form
  bool comp;
};

enum Fit : int { kFitGuess, kFitStep, kFitSolve };

template <Fit FIT>
__host__ __device__ inline Eval eval(float ax, float s, bool comp = false) {
  constexpr int kDeg = FIT == kFitGuess ? kSDeg : (FIT == kFitStep ? kTDeg : kFDeg);
  constexpr const double* kC =
      FIT == kFitGuess ? coef::kErfcxS : (FIT == kFitStep ? coef::kErfcxT : coef::kErfcxF32);
  constexpr float kB = (float)(FIT == kFitGuess ? coef::kErfcxSB
                                                : (FIT == kFitStep ? coef::kErfcxTB
                                                                   : coef::kErfcxF32B));
  constexpr auto c = [](int i) { return (float)(1.25331413731550025 * kC[i]); };
  Eval e;
  e.is = rcp(s);
  e.hq = ax * kInvSqrt2 * e.is;
  const float s2 = s * kInvSqrt2;  // 2 tq
  e.tq = 0.5f * s2;
  const float q1 = e.hq - e.tq, q2 = e.hq + e.tq;
  e.g2 = q1 * q1;
  e.H = (q1 + q1) * q2;
  e.comp = FIT == kFitGuess ? comp : q1 < -0.5f;
  const float z1 = e.comp ? -q1 : q1;
  const float a1 = z1 + kB, a2 = q2 + kB;
  constexpr float k2BZ = 2.0f * (kB - kZ0), kShift = kB - 2.0f * kZ0;
  // The solver's own residual has a reciprocal each and y = (z - B + 2 Z0) R,
  // as the binary64 evaluation: p(y) is steep near the money, and the steps'
  // shorter forms left 1.5 times the error of the general solver's there
  // (free: 10M quotes 99.3 us with either).
  float R12, R1, R2, y1, y2;
  if (FIT == kFitSolve) {
    R1 = rcp(a1);
    R2 = rcp(a2);
    R12 = R1 * R2;
    y1 = (z1 - kShift) * R1;
    y2 = (q2 - kShift) * R2;
  } else {
    R12 = rcp(a1 * a2);
    R1 = R12 * a2;
    R2 = R12 * a1;
    y1 = fmaf(-k2BZ, R1, 1.0f);
    y2 = fmaf(-k2BZ, R2, 1.0f);
  }
  float D = c(kDeg), B = fmaf(D, y2, c(kDeg - 1));
#pragma unroll
  for (int i = kDeg - 2; i >= 0; --i) {
    D = fmaf(D, y1, B);
    B = fmaf(B, y2, c(i));
  }
  const float diff = s2 * R12 * fmaf(-k2BZ * R1, D, B);
  const float A = fmaf(y1 - y2, D, B);
  const float sum = fmaf(A, R1, B * R2);
  e.rho = e.comp ? sum : diff;
  return e;
}

// What the start needs of a quote.  `lower`: beta below b(s_c), the value at
// the inflection point s_c = sqrt(2|x|); v = bh there and 1 - bh above, the
// scaled distance from the bound on beta's side, and lv = ln v.
struct Target {
  float ax;      // |x|
  float bh, ch;  // beta/b_max and 1 - beta/b_max (flushed to 0 below the binary32 range)
  float v, lv;
  bool lower, wing;  // the guess's region: R1 lower wing, R2, R3, R4 upper wing
};

__host__ __device__ inline uint32_t region_of(const Target& q) {
  return q.lower ? (q.wing ? 0u : 1u) : (q.wing ? 3u : 2u);
}

// The four-region initial guess (fv_lbr.h, lbr_initial_guess, states the
// regions, the maps and the rational cubic), in scaled form and in the
// distance v from the bound on beta's side, which makes the two halves
// mirror images: the tangent point s_o lies below s_c with the difference
// form's value b/b_max = v_o, or above it with the complement form's
// 1 - b/b_max = v_o; every cubic is fitted at its right end; and the maps,
// divided by their slope at v = 0, start with f/v = 1:
//   interior, v in [v_o, v_c]:  s from s_o to s_c, slopes -+b_max/b', no
//     curvature at s_c;
//   R1, v in [0, v_o]:  f = f_l, ln f = ln v - |x|/2 + ln(f/v),
//     f' = (2 pi/3) h^2 P^2 e^{t^2/2},  f/v_o = 3.03 |x| P^3 e^{t^2/2} b'/b,
//     v_o f'' = (b/(s b')) f' (2 phi(0) z/P - 2 h^2/3 - 2 + s^2/4),
//     z = |h|/sqrt3;
//   R4, v in [0, v_o]:  f = f_u, ln f = ln v - |x|/2 - ln 2 + ln(f/v),
//     f' = e^{h^2/2},  f/v_o = 2 sqrt(2 pi) P e^{h^2/2} b'/(b_max - b),
//     v_o f'' = ((b_max - b)/(s b')) f' h^2,  z = t,
// with P = Phi(-z) e^{z^2/2} = erfcx(z/sqrt2)/2 and everything at s_o.
// Returns s0 and completes q.  bh and ch come in the caller's precision V (a
// binary64 bh may be below the binary32 range; only its logarithm is read
// there).
template <class V>
__host__ __device__ inline float initial_guess(V bh, V ch, Target& q) {
  const float a = sqrt(q.ax);
  const float sc = kSqrt2 * a;
  // The lower tangent point s_l = sqrt2 a - sqrt(pi/2) (1 - erfcx(a)) and
  // 1 - erfcx(a) itself are differences that cancel near the money; both
  // come from tail(a) = (2 a/sqrt(pi) - 1 + erfcx(a))/a^2, fitted to 1e-5.
  constexpr float kB = (float)coef::kTailB;
  const float Rt = rcp(a + kB);
  const float yt = fmaf(-2.0f * kB, Rt, 1.0f);
  constexpr int kDeg = (int)(sizeof(coef::kTail) / sizeof(double)) - 1;
  float tail = (float)coef::kTail[kDeg];
#pragma unroll
  for (int i = kDeg - 1; i >= 0; --i) tail = fmaf(tail, yt, (float)coef::kTail[i]);
  tail *= Rt;
  const float om = a * fmaf(-a, tail, kTwoOverSqrtPi);  // 1 - erfcx(a)
  const float bc = 0.5f * om, cc = fmaf(-0.5f, om, 1.0f);  // bh(s_c); b'(s_c) = b_max/sqrt(2 pi)
  q.lower = q.bh < bc;
  q.v = q.lower ? q.bh : q.ch;
  q.lv = log_of(q.lower ? bh : ch);
  const float vc = q.lower ? bc : cc;
  const float so = q.lower ? kSqrtPiOver2 * q.ax * tail : fmaf(cc, kSqrt2Pi, sc);
  const Eval e = eval<kFitGuess>(q.ax, so, !q.lower);
  const float bp = exp_over_sqrt2pi(e.g2);  // b'(s_o)/b_max
  const float vo = e.rho * bp;
  q.wing = q.v < vo;
  // end data of the rational cubic: Yl, Yr its values, Dl, Dr its slopes
  // times the interval, C half its right second derivative times the
  // interval's square (in a wing all divided by v_o times the slope at 0)
  float Yl, Yr, Dl, Dr, C, D, x0;
  if (q.wing) {
    const float hq2 = e.hq * e.hq, tq2 = e.tq * e.tq;
    const float zq = q.lower ? e.hq * kInvSqrt3 : e.tq;  // z/sqrt2
    const float P = erfcx(zq);                           // twice the P above
    float M = exp(q.lower ? tq2 : hq2);
    M = q.lower ? M * P * P : M;
    Yr = M * P * rcp(e.rho) * (q.lower ? (0.125f * kCl * kSqrt2Pi) * q.ax : kSqrt2Pi);
    Dr = q.lower ? 1.04719755119659775f * hq2 * M : M;
    const float k = fmaf(-4.0f / 3.0f, hq2, (4.0f * kSqrt2 * kInvSqrt2Pi) * zq * rcp(P)) +
                    fmaf(2.0f, tq2, -2.0f);
    C = e.rho * e.is * Dr * (q.lower ? 0.5f * k : hq2);
    Yl = 0.0f;
    Dl = 1.0f;
    D = vo;
    x0 = 0.0f;
  } else {
    D = vc - vo;
    x0 = vo;
    Yl = so;
    Yr = sc;
    const float sd = q.lower ? D : -D;
    Dl = sd * rcp(bp);
    Dr = sd * kSqrt2Pi;
    C = 0.0f;
  }
  // The control parameter reproduces the second derivative at the right end.
  // Held at 0 or more the denominator stays away from zero; the lower bounds
  // that would keep the cubic monotone and convex never bind in a region
  // (the guess is the same to four digits with and without them).
  const float r = fminf(fmaxf((C + Dr - Dl) * rcp(Dr - (Yr - Yl)), 0.0f), 1e6f);
  // the position in the interval, measured from the end whose s is the
  // smaller: near the money the two ends are many decades apart
  const bool left = q.wing || q.lower;
  const float from = left ? q.v - x0 : q.bh - bc;
  const float near = fminf(fmaxf(from * rcp(D), 0.0f), 1.0f);
  const float far = 1.0f - near;
  const float tau = left ? near : far, w = left ? far : near, tw = near * far;
  const float den = fmaf(r - 3.0f, tw, 1.0f);
  const float A = fmaf(Yr, tau * tau, fmaf(fmaf(r, Yr, -Dr), tw, fmaf(r, Yl, Dl) * (w * w)));
  if (!q.wing) return fmaf(tau, A, Yl * w * w * w) * rcp(den);
  // invert the map from ln p: R1 p = Phi(-z) = (f/cl)^{1/3}, s = |x|/(sqrt3 z);
  // R4 p = Phi(-z) = f, s = 2 z
  const float lf = fmaf(log2(fmaxf(A, 1e-30f) * rcp(den * (q.lower ? kCl * q.ax : 2.0f))), kLn2,
                        fmaf(-0.5f, q.ax, q.lv));
  const float lnp = q.lower ? lf * (1.0f / 3.0f) : lf;
  const float rr = sqrt(-2.0f * fminf(lnp, -0.69314719f));
  const float pn = fmaf(rr, fmaf(rr, fmaf(rr, (float)coef::kPhiInvGP[3], (float)coef::kPhiInvGP[2]),
                                 (float)coef::kPhiInvGP[1]),
                        (float)coef::kPhiInvGP[0]);
  const float pd = fmaf(rr, fmaf(rr, fmaf(rr, (float)coef::kPhiInvGQ[3], (float)coef::kPhiInvGQ[2]),
                                 (float)coef::kPhiInvGQ[1]),
                        (float)coef::kPhiInvGQ[0]);
  const float zn = ((float)coef::kPhiInvGR0 - rr) * pn;  // z = zn/pd
  return q.lower ? q.ax * kInvSqrt3 * pd * rcp(zn) : 2.0f * zn * rcp(pd);
}

// The steps' objectives, each in the logarithm of the distance from its
// bound or in b itself (fv_lbr.h):
//   R1 1/ln b, R4 ln(1 - b/b_max), else b.
// In a wing an iterate near the root has that wing's form; one that does
// not gives a step that the binary64 iteration finds too large.
// n = -g/(s g') of the objective g, E2 and E3 its s g''/g' and s^2 g'''/g'.
// Every quantity is dimensionless, so nothing overflows for small s.
//
// One Householder(3) step, as ds/s.
__host__ __device__ inline float householder3(const Target& q, const Eval& e) {
  const float H = e.H;                                                // s b''/b'
  const float H3 = fmaf(-8.0f * e.hq, e.hq, fmaf(H, H, H));  // s^2 b'''/b' = H^2 - 3 h^2 - t^2
  float n, E2, E3;
  if (!q.wing) {
    const float W = exp_sqrt2pi(e.g2);  // b_max/b'
    n = (e.comp ? fmaf(-q.ch, W, e.rho) : fmaf(q.bh, W, -e.rho)) * e.is;
    E2 = H;
    E3 = H3;
  } else {
    const float rs = e.rho * e.is;
    const float w = q.lower ? -rcp(rs) : rcp(rs);   // -s b'/b or s b'/(b_max - b)
    const float lb = fmaf(log2(e.rho), kLn2, -kLnSqrt2Pi - e.g2);  // ln(b/b_max) or ln(1 - b/b_max)
    const float u = lb - q.lv;
    const float iL = q.lower ? rcp(fmaf(-0.5f, q.ax, lb)) : 0.0f;  // 1/ln b
    const float k = q.lower ? -1.0f - u * rcp(fmaf(-0.5f, q.ax, q.lv)) : 1.0f;  // -+ln b/ln beta
    n = u * rs * k;
    const float wi = w * iL;
    E2 = fmaf(2.0f, wi, H + w);
    E3 = fmaf(6.0f * wi, H + w + wi, fmaf(w, fmaf(2.0f, w, 3.0f * H), H3));
  }
  const float d = n * fmaf(0.5f * E2, n, 1.0f) * rcp(fmaf(n, fmaf(E3 * (1.0f / 6.0f), n, E2), 1.0f));
  return fmaxf(d, -0.5f);
}

// One Halley step, as ds/s (in R1 on ln b).
__host__ __device__ inline float halley(const Target& q, const Eval& e) {
  const float H = e.H;
  float n, E2;
  if (!q.wing) {
    const float W = exp_sqrt2pi(e.g2);
    n = (e.comp ? fmaf(-q.ch, W, e.rho) : fmaf(q.bh, W, -e.rho)) * e.is;
    E2 = H;
  } else {
    const float rs = e.rho * e.is;
    const float w = rcp(rs);
    const float u = fmaf(log2(e.rho), kLn2, -kLnSqrt2Pi - e.g2) - q.lv;
    n = q.lower ? -u * rs : u * rs;
    E2 = q.lower ? H - w : H + w;
  }
  return fmaxf(n * rcp(fmaf(0.5f * E2, n, 1.0f)), -0.5f);
}

}  // namespace s32
}  // namespace fv
