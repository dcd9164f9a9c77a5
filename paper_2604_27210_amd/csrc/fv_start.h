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
// instructions; these take about 240 and 60.
//
// Binary32 cannot hold b itself deep in a wing, so everything is scaled by
// the bound b_max = e^{x/2}: bh = b/b_max in (0, 1) and
//   b'/b_max = e^{-g^2/2}/sqrt(2 pi),  g = h + t
// (h = x/s, t = s/2; h t = x/2 cancels in the exponent), with ratios to b'
// in place of values and logarithms in place of the values that leave the
// range.  Domain (start_in_domain): |x| zero or in [2^-60, 128], bh above
// 2^-1000; a quote outside it, or whose iteration does not settle, takes the
// binary64 path.
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
__host__ __device__ inline float exp(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_exp2f(x * kLog2E);
#else
  return exp2f(x * kLog2E);
#endif
}
__host__ __device__ inline float log(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_logf(x) * kLn2;
#else
  return log2f(x) * kLn2;
#endif
}
// ln of a positive normal binary64 number of any exponent
__host__ __device__ inline float log_of_double(double v) {
  int e;
  const float m = (float)frexp(v, &e);
#if defined(__HIP_DEVICE_COMPILE__)
  return (__builtin_amdgcn_logf(m) + (float)e) * kLn2;
#else
  return (log2f(m) + (float)e) * kLn2;
#endif
}

constexpr float kZ0 = (float)coef::kErfcxZ0;
constexpr int kGDeg = (int)(sizeof(coef::kErfcxG) / sizeof(double)) - 1;
constexpr int kLoDeg = (int)(sizeof(coef::kErfcxLo) / sizeof(double)) - 1;

// erfcx(z), z >= -1/2, by the initial guess's fit (4e-6)
__host__ __device__ inline float erfcx(float z) {
  constexpr float kB = (float)coef::kErfcxGB;
  const float R = rcp(z + kB);
  const float y = fmaf(-2.0f * (kB - kZ0), R, 1.0f);
  float p = (float)coef::kErfcxG[kGDeg];
#pragma unroll
  for (int i = kGDeg - 1; i >= 0; --i) p = fmaf(p, y, (float)coef::kErfcxG[i]);
  return p * R;
}

// The normalised Black function at s, as ratios to b' (fv_math.h has the
// two forms): GUESS picks the degree-7 fit of erfcx, else the degree-12 one.
struct Eval {
  float is, h2;  // 1/s, h^2
  float g2;      // g^2/2: b'/b_max = e^{-g2}/sqrt(2 pi)
  float rho;     // b/b' in the difference form, (b_max - b)/b' in the complement form
  bool comp;
};

template <bool GUESS>
__host__ __device__ inline Eval eval(float ax, float s) {
  constexpr int kDeg = GUESS ? kGDeg : kLoDeg;
  constexpr const double* kC = GUESS ? coef::kErfcxG : coef::kErfcxLo;
  constexpr float kB = (float)(GUESS ? coef::kErfcxGB : coef::kErfcxLoB);
  Eval e;
  e.is = rcp(s);
  const float h = -ax * e.is, t = 0.5f * s;
  const float g = h + t;
  e.h2 = h * h;
  e.g2 = 0.5f * g * g;
  const float q1 = -g * kInvSqrt2, q2 = (t - h) * kInvSqrt2;
  e.comp = q1 < -kZ0;
  const float z1 = e.comp ? -q1 : q1;
  const float a1 = z1 + kB, a2 = q2 + kB;
  const float R12 = rcp(a1 * a2);
  const float R1 = R12 * a2, R2 = R12 * a1;
  constexpr float k2BZ = 2.0f * (kB - kZ0);
  const float y1 = fmaf(-k2BZ, R1, 1.0f), y2 = fmaf(-k2BZ, R2, 1.0f);
  float B = (float)kC[kDeg], D = 0.0f;
#pragma unroll
  for (int i = kDeg - 1; i >= 0; --i) {
    D = fmaf(D, y1, B);
    B = fmaf(B, y2, (float)kC[i]);
  }
  const float diff = kSqrtPi * t * R12 * fmaf(-k2BZ * R1, D, B);
  const float A = fmaf(y1 - y2, D, B);
  const float sum = kSqrtPiOver2 * fmaf(A, R1, B * R2);
  e.rho = e.comp ? sum : diff;
  return e;
}

// What the start needs of a quote.
struct Target {
  float ax;   // |x|
  float bh;   // beta/b_max (flushed to 0 below the binary32 range)
  float ch;   // 1 - beta/b_max
  float lbh;  // ln(beta/b_max)
};

enum Region : int { kR1 = 0, kR2 = 1, kR3 = 2, kR4 = 3 };

struct Guess {
  float s;
  int region;
  bool comp_o;  // evaluation form at the boundary point (diagnostics)
};

// The four-region initial guess (fv_lbr.h, lbr_initial_guess, states the
// regions, the maps and the rational cubic) in scaled form.  With
// P(z) = Phi(z) e^{z^2/2} = erfcx(-z/sqrt2)/2 the maps' values and slopes at
// the boundary point are free of exponentials that leave the range:
//   R1, everything divided by D = bh_l:  f/D = cl P^3 e^{t^2/2} sqrt(2 pi)/rho,
//       f'_beta = (2 pi/3) h^2 P^2 e^{t^2/2}  (z = h/sqrt3),
//       D f''_beta = (rho/s) f'_beta (2 phi(0) |z|/P - 2 h^2/3 - 2 + s^2/4),
//       and the cubic gives f/beta, so ln f = ln beta + ln(f/beta);
//   R4, divided by f_u = Phi(-t):  D f'_beta = -(c/b')/(2 sqrt(2 pi) P)  (z = -t),
//       at b_max that times e^{-h^2/2},
//       D^2 f''_beta = -D f'_beta (c/b') h^2/s.
__host__ __device__ inline Guess initial_guess(const Target& q) {
  Guess out;
  const float a = sqrt(q.ax);
  const float sc = kSqrt2 * a;
  float om = 1.0f - erfcx(a);  // 1 - erfcx(sqrt|x|)
  float sl = sc - kSqrtPiOver2 * om;
  if (a < 0.03f) {  // both differences cancel near the money: series in a
    constexpr float c3 = 0.752252778063675f, c5 = 0.300901111225470f, c7 = 0.0859717460644200f;
    const float tail =
        fmaf(-a, fmaf(-a, fmaf(-a, fmaf(-a, fmaf(-a, c7, 1.0f / 6.0f), c5), 0.5f), c3), 1.0f);
    om = a * fmaf(-a, tail, kTwoOverSqrtPi);
    sl = kSqrtPiOver2 * q.ax * tail;
  }
  const float bc = 0.5f * om;  // bh(s_c); b'(s_c) = b_max/sqrt(2 pi)
  const bool lower = q.bh < bc;
  const float so = lower ? sl : fmaf(1.0f - bc, kSqrt2Pi, sc);
  const Eval e = eval<true>(q.ax, so);
  out.comp_o = e.comp;
  const float ibo = kSqrt2Pi * exp(e.g2);  // b_max/b'(s_o)
  const float ro = e.rho * rcp(ibo);       // bh(s_o), or 1 - bh(s_o)
  const float bo = e.comp ? 1.0f - ro : ro;
  const float t = 0.5f * so;
  const bool wing = lower ? q.bh < bo : q.bh > bo;
  out.region = lower ? (wing ? kR1 : kR2) : (wing ? kR4 : kR3);
  // the rational cubic's end data: values Yl, Yr, slopes Dl, Dr times the
  // interval and C half the second derivative times its square
  float Yl, Yr, Dl, Dr, C, D, xl;
  float Pz = 0.0f;
  if (wing) {
    const float z = lower ? sqrt(e.h2) * kInvSqrt3 : t;  // |z|
    Pz = 0.5f * erfcx(z * kInvSqrt2);
    if (lower) {
      const float et = exp(0.5f * t * t);
      const float P2 = Pz * Pz * et;
      D = bo;
      xl = 0.0f;
      Yl = 0.0f;
      Yr = (kCl * kSqrt2Pi) * q.ax * P2 * Pz * rcp(e.rho);
      Dl = 1.0f;
      Dr = (2.0f * 1.04719755119659775f) * e.h2 * P2;
      C = 0.5f * e.rho * e.is * Dr *
          (fmaf(-2.0f / 3.0f, e.h2, (2.0f * kInvSqrt2Pi) * z * rcp(Pz)) + fmaf(t, t, -2.0f));
    } else {
      const float cr = e.comp ? e.rho : (1.0f - bo) * ibo;  // c/b'
      D = 1.0f - bo;
      xl = bo;
      Yl = 1.0f;
      Yr = 0.0f;
      Dl = -0.5f * kInvSqrt2Pi * cr * rcp(Pz);
      Dr = Dl * exp(-0.5f * e.h2);
      C = -0.5f * Dl * cr * e.h2 * e.is;
    }
  } else {
    D = lower ? bc - bo : bo - bc;
    xl = lower ? bo : bc;
    Yl = lower ? so : sc;
    Yr = lower ? sc : so;
    const float dc = D * kSqrt2Pi, dd = D * ibo;
    Dl = lower ? dd : dc;
    Dr = lower ? dc : dd;
    C = 0.0f;
  }
  const float S = Yr - Yl;
  const float gl = S - Dl, gr = Dr - S;
  // control parameter: reproduces the second derivative at the inner end,
  // held above the monotone and the convex or concave minimum
  float r = (C + Dr - Dl) * rcp(lower ? gr : gl);
  float rmin = -1.0f + 1e-6f;
  if (Dl * S >= 0.0f && Dr * S >= 0.0f && S != 0.0f) rmin = fmaxf(rmin, (Dl + Dr) * rcp(S));
  if (gl * gr >= 0.0f) {
    const float gap = fminf(fabsf(gl), fabsf(gr));
    rmin = fmaxf(rmin, fabsf(Dr - Dl) * rcp(fmaxf(gap, 1e-30f)));
  }
  r = fminf(fmaxf(r, rmin), 1e6f);  // fmaxf drops a NaN
  const float tau = fminf(fmaxf((q.bh - xl) * rcp(D), 0.0f), 1.0f);
  const float w = 1.0f - tau;
  const float den = fmaf((r - 3.0f) * tau, w, 1.0f);
  const float A = fmaf(Yr * tau, tau, fmaf(fmaf(r, Yr, -Dr) * tau, w, fmaf(r, Yl, Dl) * w * w));
  const float num = fmaf(tau, A, Yl * w * w * w);
  if (!wing) {
    out.s = num * rcp(den);
    return out;
  }
  // invert the map from ln p: R1 p = Phi(z) = (f/cl)^{1/3}, s = |x|/(sqrt3 |z|);
  // R4 p = f, s = 2 |z|
  const float lq = log(fmaxf(lower ? A : num * Pz, 1e-30f) * rcp(lower ? den * (kCl * q.ax) : den));
  const float lnp = lower ? (q.lbh - 0.5f * q.ax + lq) * (1.0f / 3.0f) : fmaf(-0.5f * t, t, lq);
  const float rr = sqrt(-2.0f * fminf(lnp, -0.69314719f));
  const float pn = fmaf(rr, fmaf(rr, fmaf(rr, (float)coef::kPhiInvGP[3], (float)coef::kPhiInvGP[2]),
                                 (float)coef::kPhiInvGP[1]),
                        (float)coef::kPhiInvGP[0]);
  const float pd = fmaf(rr, fmaf(rr, fmaf(rr, (float)coef::kPhiInvGQ[3], (float)coef::kPhiInvGQ[2]),
                                 (float)coef::kPhiInvGQ[1]),
                        (float)coef::kPhiInvGQ[0]);
  const float zi = ((float)coef::kPhiInvGR0 - rr) * pn;  // |z| pd
  out.s = lower ? q.ax * kInvSqrt3 * pd * rcp(zi) : 2.0f * zi * rcp(pd);
  return out;
}

// One Householder(3) step on the region's objective (fv_lbr.h,
// householder3_step_t), as ds/s: every quantity is made dimensionless by
// powers of s, so nothing overflows for small s.
__host__ __device__ inline float householder3(const Target& q, int region, const Eval& e, float s) {
  const float s2 = 0.25f * s * s;
  const float H = e.h2 - s2;                       // s b''/b'
  const float H3 = fmaf(H, H, -3.0f * e.h2 - s2);  // s^2 b'''/b'
  float n, E2, E3;
  if (region == kR2 || region == kR3) {
    const float W = kSqrt2Pi * exp(e.g2);  // b_max/b'
    n = (e.comp ? fmaf(-q.ch, W, e.rho) : fmaf(q.bh, W, -e.rho)) * e.is;
    E2 = H;
    E3 = H3;
  } else {
    const bool lo = region == kR1;
    // b/b' or (b_max - b)/b', whichever the objective takes
    float rho = e.rho;
    if (lo == e.comp) rho = kSqrt2Pi * exp(e.g2) - e.rho;
    const float rs = rho * e.is;
    const float w = rcp(rs);  // s b'/b or s b'/(b_max - b)
    const float lb = log(rho) - e.g2 - kLnSqrt2Pi;  // ln bh or ln(1 - bh)
    if (lo) {
      const float u = lb - q.lbh;  // ln(b/beta)
      const float L = lb - 0.5f * q.ax;
      const float iL = rcp(L);
      n = -(L * rcp(q.lbh - 0.5f * q.ax)) * u * rs;
      E2 = H - w * fmaf(2.0f, iL, 1.0f);
      E3 = H3 - 3.0f * w * H + 2.0f * w * w - 6.0f * w * (H - w) * iL + 6.0f * w * w * iL * iL;
    } else {
      n = -(log(q.ch) - lb) * rs;
      E2 = H + w;
      E3 = H3 + 3.0f * w * H + 2.0f * w * w;
    }
  }
  const float d = n * fmaf(0.5f * E2, n, 1.0f) * rcp(fmaf(n, fmaf(E3 * (1.0f / 6.0f), n, E2), 1.0f));
  return fmaxf(d, -0.5f);
}

// One Halley step as ds/s: on ln b - ln beta in the difference form, on the
// direct residual in the complement form.
__host__ __device__ inline float halley(const Target& q, const Eval& e, float s) {
  const float H = e.h2 - 0.25f * s * s;  // s b''/b'
  float n, E2;
  if (e.comp) {
    n = fmaf(-q.ch, kSqrt2Pi * exp(e.g2), e.rho) * e.is;
    E2 = H;
  } else {
    const float rs = e.rho * e.is;
    n = (q.lbh - (log(e.rho) - e.g2 - kLnSqrt2Pi)) * rs;
    E2 = H - rcp(rs);
  }
  return fmaxf(n * rcp(fmaf(0.5f * E2, n, 1.0f)), -0.5f);
}

}  // namespace s32
}  // namespace fv
