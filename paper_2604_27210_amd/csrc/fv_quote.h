// fv_quote.h -- per-quote pre-processing, post-processing, Greeks and the
// implied-volatility adjoint, shared by every kernel.
//
// Pre-processing (the paper's section 4: flags normalised, inputs validated;
// section 2.4: a Black-76 price is the discounted mid and the same r both
// discounts and inverts):
//   F  = forward:  Black-76 input, S e^{rT} (Black-Scholes),
//                  S e^{(r-q)T} (Black-Scholes-Merton);   D = e^{-rT};
//   Pu = price / D  (undiscounted),
//   I  = max(theta (F - K), 0),  M = F (call) or K (put);
//   Pu <  I  -> BELOW_INTRINSIC,  Pu == I -> AT_INTRINSIC (sigma = 0),
//   Pu >= M  -> ABOVE_MAX;  non-finite or non-positive F/S, K, T -> INVALID.
// Solvable quotes are reduced to an out-of-the-money call by put-call
// parity (Pu -= I, theta -> -theta when in the money) and normalised:
//   x = theta ln(F/K) <= 0,  beta = Pu / sqrt(F K),  s = sigma sqrt(T).
#pragma once

#include "fv_lbr.h"

namespace fv {

enum Model : int { kBlack76 = 0, kBlackScholes = 1, kBlackScholesMerton = 2 };
enum QuoteStatus : uint8_t {
  kQOk = 0,
  kQAtIntrinsic = 1,
  kQBelowIntrinsic = 2,
  kQAboveMax = 3,
  kQInvalid = 4,
  kQNotConverged = 5,
};

struct Reduced {
  double F, D;
  double isqrtT;   // 1/sqrt(T): sigma = s isqrtT
  double x, beta;  // normalised out-of-the-money call: x <= 0, 0 < beta < e^{x/2}
  double bmax;     // e^{x/2} = min(F, K)/sqrt(F K)
  double lnb;      // ln beta, to full relative precision also where beta is below
                   // the normal range (or underflowed) for an out-of-the-money quote
  uint8_t status;
};

// Finite test by classification (v_cmp_class), never by arithmetic: with
// contraction on, v - v == 0 for a product v = a b compiles to
// fma(a, b, -v) == 0, the product's rounding error, which is rarely 0.
__host__ __device__ inline bool finite_d(double v) { return __builtin_isfinite(v); }

// sqrt(T) for finite T > 0 as T / sqrt(T) from the refined reciprocal
// square root, with T scaled by 2^200 first when it is so small that
// v_rsq_f64 could see a denormal
__host__ __device__ inline double sqrt_pos(double T) {
  const bool tiny = T < 1e-290;
  const double Ts = tiny ? T * 0x1p+200 : T;
  return Ts * rsqrt(Ts) * (tiny ? 0x1p-100 : 1.0);
}

// 1/sqrt(T) for finite T > 0, with the same scaling of tiny T
__host__ __device__ inline double rsqrt_pos(double T) {
  const bool tiny = T < 1e-290;
  const double Ts = tiny ? T * 0x1p+200 : T;
  return rsqrt(Ts) * (tiny ? 0x1p+100 : 1.0);
}

// e^{a b} with the rounding error of the exponent carried into the result:
// a b = p + e exactly (p = fl(a b), e = fma(a, b, -p)) and e^{p + e} =
// e^p (1 + e) to first order (|e| <= 2^-53 |p|).  Over long maturities r T
// reaches tens, where dropping e would put tens of ulps into the forward or
// the discount factor, errors that the inputs' own conditioning does not
// cover (the exact sensitivity to r cancels between forward and discount).
// IN: the caller knows |a b| <= 700 (fexp_in).
template <bool IN = false>
__host__ __device__ inline double fexp_prod(double a, double b) {
  const double p = a * b;
  const double e = fma(a, b, -p);
  const double E = IN ? fexp_in(p) : fexp(p);
  return fma(E, e, E);
}

// e^{(r - q) T}, carrying the rounding of r - q as well (Knuth's two-sum:
// r - q = c + ce exactly)
template <bool IN = false>
__host__ __device__ inline double fexp_carry(double r, double q, double T) {
  const double c = r - q;
  const double bb = c - r;
  const double ce = (r - (c - bb)) + (-q - bb);
  const double p = c * T;
  const double e = fma(c, T, -p) + ce * T;
  const double E = IN ? fexp_in(p) : fexp(p);
  return fma(E, e, E);
}

// a - b with both operands rounded first (never contracted into an fma)
__host__ __device__ inline double minus(double a, double b) {
#pragma clang fp contract(off)
  return a - b;
}

// F / fs
template <bool IN = false>
__host__ __device__ inline double growth_of(int model, double T, double r, double q) {
  if (model == kBlack76) return 1.0;
  return model == kBlackScholesMerton ? fexp_carry<IN>(r, q, T) : fexp_prod<IN>(r, T);
}

__host__ __device__ inline double forward_of(int model, double fs, double T, double r,
                                             double q) {
  return model == kBlack76 ? fs : fs * growth_of(model, T, r, q);
}

// ln(F/K) for positive K and F >= 0: a forward that underflowed has none
// (log_ratio would make a finite number of its significand)
__host__ __device__ inline double log_moneyness(double F, double K) {
  return F == 0.0 ? -__builtin_inf() : log_ratio(F, K);
}

__host__ __device__ __attribute__((always_inline)) inline Reduced reduce_quote(int model, double price, double fs, double K,
                                                double T, double r, double q, int theta) {
  // One exit: every lane computes every field and the status is decided at
  // the end, in the order of the checks below (invalid input first).  The
  // fields of a quote whose status is not OK are meaningless and no caller
  // reads them; early returns would instead make every path set defaults.
  Reduced o;
  // S/F and K must be normal numbers (the refined hardware reciprocals
  // below need normal operands); so must the forward
  const bool ok_in = finite_d(price) && finite_d(fs) && finite_d(K) && finite_d(T) &&
                     finite_d(r) && finite_d(q) && fs >= kDblMin && K >= kDblMin && T > 0.0 &&
                     (theta == 1 || theta == -1);
  const double F = forward_of(model, fs, T, r, q);
  const bool ok_f = F >= kDblMin && finite_d(F);
  const double D = fexp_prod(-r, T);
  const double Pu = price * fexp_prod(r, T);
  const double dth = (double)theta;
  const double I = fmax(dth * (F - K), 0.0);  // intrinsic value (the sign flip is exact)
  const double M = theta > 0 ? F : K;
  o.F = F;
  o.D = D;
  o.isqrtT = rsqrt_pos(T);
  // in the money: parity to out of the money
  const double th = I > 0.0 ? -dth : dth;
  o.x = th * log_moneyness(F, K);
  // 1/sqrt(F K) as two factors: F K itself leaves the binary64 range once F
  // and K are beyond about 1e+-154, while the normalised quantities do not
  // (and scaling price, F and K by an even power of two scales both factors
  // exactly, so the result is bitwise homogeneous of degree 0)
  const double isq = rsqrt(F) * rsqrt(K);
  o.beta = (Pu - I) * isq;
  o.bmax = fmin(F, K) * isq;
  if (o.beta < 0x1p-1000 && I == 0.0) {
    // out of the money with a price too small for beta to keep full precision
    // in binary64: ln beta = ln P + r T - ln(F K)/2 from the price itself
    o.lnb = flog(price) + r * T - 0.5 * (flog(F) + flog(K));
  } else {
    o.lnb = flog(o.beta);
  }
  // the normalised price can round onto its bound even when Pu < M
  uint8_t st = o.beta < o.bmax ? kQOk : kQAboveMax;
  if (Pu >= M) st = kQAboveMax;
  if (Pu == I) st = kQAtIntrinsic;
  if (Pu < I) st = kQBelowIntrinsic;
  if (!(ok_in && ok_f)) st = kQInvalid;
  o.status = st;
  return o;
}

// What the scaled solvers (fv_lbr.h) need of a quote.  The status comes from
// the comparisons of reduce_quote on the same quantities (F - K is rounded
// here and may be contracted there, so a quote within an ulp of its intrinsic
// value can fall on either side); `general` marks a quote outside the scaled
// solvers' domain, or whose status these forms cannot decide: it goes through
// reduce_quote, which decides it whole, and the general solver.
// Against reduce_quote this drops ln beta (a logarithm) and 1/sqrt(F K)
// (two reciprocal square roots): bh = beta/b_max = (Pu - I)/min(F, K).
struct ScaledQuote {
  double F, D;
  double isqrtT;
  double x, bh, ch;  // ln(F/K) <= 0, beta/b_max and 1 - beta/b_max
  uint8_t status;
  bool general;
};

__host__ __device__ inline bool positive_normal(double v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_class(v, 0x100);
#else
  return v >= kDblMin && finite_d(v);
#endif
}

__host__ __device__ inline ScaledQuote scaled_quote(int model, double price, double fs, double K,
                                                    double T, double r, double q, int theta) {
  ScaledQuote o;
  const double rT = r * T;
  const double cT = model == kBlackScholesMerton ? minus(r, q) * T : rT;
  // The plain forms below need T normal and both exponents in range.  A
  // quote outside (an infinite or NaN rate among them) goes to the general
  // path whole, so T, r and q need no test of their own.
  const bool plain = all(T >= 1e-290, fabs(rT) <= 700.0, fabs(cT) <= 700.0);
  const double gr = growth_of<true>(model, T, r, q);
  const double F = fs * gr;
  const double cap = fexp_prod<true>(r, T);  // 1/D
  const double Pu = price * cap;
  const double dth = (double)theta;
  const double I = fmax(dth * minus(F, K), 0.0);
  const double M = theta > 0 ? F : K;
  o.F = F;
  o.D = fexp_prod<true>(-r, T);
  o.isqrtT = rsqrt(T);
  int eF;
  o.x = -fabs(log_ratio(F, K, &eF));
  // the time value from the rounded forward and the unrounded price: in the
  // money it is a small difference of large numbers, and what its operands'
  // roundings leave of it is the quote's implied volatility
  const double m = F < K ? F : K;
  const double tv = fma(price, cap, -I), im = rcp(m);
  o.bh = tv * im;
  o.ch = (m - tv) * im;
  uint8_t st = kQOk;
  if (Pu >= M) st = kQAboveMax;
  if (Pu == I) st = kQAtIntrinsic;
  if (Pu < I) st = kQBelowIntrinsic;
  const bool valid = all(finite_d(price), positive_normal(fs), positive_normal(K),
                         positive_normal(F), ((theta + 1) & ~2) == 0);
  st = valid ? st : (uint8_t)kQInvalid;
  o.status = st;
  // m below 2^1001, where rcp keeps its precision (its lower end holds to the
  // smallest normal number)
  o.general = !all(plain, st != kQOk || all(scaled_domain(o.x, o.bh, o.ch), eF <= 1000));
  return o;
}

// The general implied volatility of one quote: reduce_quote and lbr_solve.
// Replaces what scaled_quote made of F and D.
__host__ __device__ __attribute__((always_inline)) inline void lbr_general(
    int model, double price, double fs, double K, double T, double r, double q, int theta,
    double* sigma, uint8_t* status, ScaledQuote* sq, uint32_t* trace = nullptr) {
  const Reduced rd = reduce_quote(model, price, fs, K, T, r, q, theta);
  sq->F = rd.F;  // an extreme exponent or maturity made nothing of scaled_quote's
  sq->D = rd.D;
  sq->isqrtT = rd.isqrtT;
  uint8_t st = rd.status;
  double sg = st == kQAtIntrinsic ? 0.0 : __builtin_nan("");
  if (st == kQOk) {
    const LbrResult res = lbr_solve(rd.x, rd.beta, rd.bmax, rd.lnb, kLbrMinSteps, kLbrMaxSteps,
                                    kLbrStepTol, trace);
    sg = res.s * rd.isqrtT;
    if (!res.converged) st = kQNotConverged;
  }
  *sigma = sg;
  *status = st;
}

// Accurate Phi(a) for either sign of a.
__host__ __device__ inline double norm_cdf_signed(double a) { return norm_cdf(a); }

// Raw per-unit Greeks at sigma (paper section 3: get_all_greeks returns all
// five from one d1/d2 evaluation):
//   delta = dP/dS (dP/dF for Black-76), gamma = d2P/dS2, vega = dP/dsigma,
//   theta = -dP/dT per year, rho = dP/dr (Black-76: at fixed F).
// `price` is the option price at sigma (input or recomputed by the caller).
struct Greeks {
  double delta, gamma, vega, theta, rho;
};

// Terms every closed form below shares, computed once: s = sigma sqrt(T),
// d1 = ln(F/K)/s + s/2, d2 = d1 - s, Phi(theta d1), Phi(theta d2), phi(d1)
// and the discounted forward D F (= S e^{-qT} for Black-Scholes(-Merton)).
struct BsTerms {
  double sqT, s, d1, d2, N1, N2, n1, DF;
};

__host__ __device__ inline BsTerms bs_terms(double F, double K, double D, double sigma, double T,
                                            int theta) {
  BsTerms c;
  c.sqT = sqrt_pos(T);
  c.s = sigma * c.sqT;
  c.d1 = log_moneyness(F, K) / c.s + 0.5 * c.s;
  c.d2 = c.d1 - c.s;
  c.N1 = norm_cdf(theta * c.d1);
  c.N2 = norm_cdf(theta * c.d2);
  c.n1 = norm_pdf(c.d1);
  c.DF = D * F;
  return c;
}

__host__ __device__ inline Greeks greeks_from(const BsTerms& c, int model, double fs, double K,
                                              double T, double r, double q, double sigma,
                                              int theta, double F, double D, double price) {
  Greeks g;
  g.vega = c.DF * c.n1 * c.sqT;
  const double decay = 0.5 * sigma * c.DF * c.n1 / c.sqT;  // -dP/dT from the time value
  if (model == kBlack76) {
    g.delta = theta * D * c.N1;
    g.gamma = D * c.n1 / (F * c.s);
    g.theta = r * price - decay;
    g.rho = -T * price;
  } else {
    const double qy = (model == kBlackScholesMerton) ? q : 0.0;
    const double Dq = c.DF / fs;  // e^{-qT}
    g.delta = theta * Dq * c.N1;
    g.gamma = Dq * c.n1 / (fs * c.s);
    g.theta = -decay - theta * r * K * D * c.N2 + theta * qy * c.DF * c.N1;
    g.rho = theta * K * T * D * c.N2;
  }
  return g;
}

__host__ __device__ __attribute__((always_inline)) inline Greeks greeks_at(int model, double fs, double K, double T, double r,
                                            double q, double sigma, int theta, double F,
                                            double D, double price) {
  return greeks_from(bs_terms(F, K, D, sigma, T, theta), model, fs, K, T, r, q, sigma, theta, F,
                     D, price);
}

// Partial derivatives of the price at fixed sigma:
//   d/dfs = delta, d/dK = -theta D Phi(theta d2), d/dT = -(Greek theta),
//   d/dr = rho, d/dq = -theta T D F Phi(theta d1) (Black-Scholes-Merton
//   only), d/dsigma = vega.
struct PricePartials {
  double dfs, dK, dT, dr, dq, dsigma;
};

__host__ __device__ __attribute__((always_inline)) inline PricePartials price_partials(int model, double fs, double K,
                                                        double T, double r, double q,
                                                        double sigma, int theta, double F,
                                                        double D, double price) {
  PricePartials o;
  const BsTerms c = bs_terms(F, K, D, sigma, T, theta);
  const Greeks g = greeks_from(c, model, fs, K, T, r, q, sigma, theta, F, D, price);
  o.dfs = g.delta;
  o.dK = -theta * D * c.N2;
  o.dT = -g.theta;
  o.dr = g.rho;
  o.dq = (model == kBlackScholesMerton) ? -theta * T * c.DF * c.N1 : 0.0;
  o.dsigma = g.vega;
  return o;
}

// ------------------------------------------------- closed forms, scaled
// Price, Greeks and partials at a volatility from ONE evaluation of the
// normalised Black function (scaled_eval) and one exponential E =
// e^{-g^2/2}, g = h + t, for the out-of-the-money side (x <= 0, m = min(F, K)):
//   m b/b_max                     its undiscounted price,
//   m U1 and m U2                 its two terms (F Phi and K Phi of d1 and d2
//                                 in some order), U2 = E erfcx(q2)/2 and
//                                 U1 = U2 + b/b_max without cancellation (and
//                                 1 - U1 in the complement form, where the
//                                 in-the-money side needs it),
//   m E/sqrt(2 pi) = F phi(d1) = K phi(d2),
// and the in-the-money side by parity.  The general forms above and below
// evaluate two normal tails, a density and (for the Greeks) a price, with an
// exponential each, four roots and four divisions.
struct ScaledTerms {
  double P;       // undiscounted price
  double FN, KN;  // F Phi(theta d1), K Phi(theta d2)
  double V;       // F phi(d1)
};

// False outside the domain (the caller takes the general forms): |x| above
// 128, total volatility outside [2^-60, 64], b/b_max (or its complement) below
// 2^-1010 (which a clamped exponent does not reach), or the time value m part,
// discounted or not, below 2^-1000: it is at most four times F phi(d1), so
// that, both terms and their discounted values are normal numbers then.  The
// general forms multiply by the spot last or not at all.
__host__ __device__ __attribute__((always_inline)) inline bool scaled_terms(double F, double K,
                                                                            double D, double x,
                                                                            double s, int theta,
                                                                            ScaledTerms* o) {
  const ScaledEval e = scaled_eval(x, s);
  const double ea = -0.5 * e.g * e.g;
  const double E = fexp_in(fmax(ea, -700.0));
  const double dens = kInvSqrt2Pi * E;  // b'/b_max
  const double part = dens * e.rho;
  // (products that meet a sum are written as fmas: left to the compiler, one
  // kernel contracts them and another does not)
  const double hE = 0.5 * E;
  const double bh = e.comp ? fma(-dens, e.rho, 1.0) : part;
  const double U2 = hE * e.e2, U1 = fma(hE, e.e2, bh);
  const double V1 = e.comp ? fma(dens, e.rho, -U2) : 1.0 - U1;  // 1 - U1
  const bool low = F < K, call = theta > 0, itm = call ? F > K : low;
  const double m = low ? F : K, M = low ? K : F;
  const bool as_call = call != itm;  // the out-of-the-money counterpart's kind
  const double t1 = m * (itm ? V1 : U1), t2 = m * U2, t3 = itm ? fma(-m, U2, M) : t2;
  o->FN = as_call ? t1 : t3;
  o->KN = as_call ? t3 : t1;
  o->P = fma(m, bh, itm ? fabs(F - K) : 0.0);
  o->V = m * dens;
  return all(x >= -128.0, s >= 0x1p-60, s <= 64.0, part >= 0x1p-1010,
             fmin(D, 1.0) * (m * part) >= 0x1p-1000);
}

// A quote the scaled closed forms take: every quantity they divide by or
// square a normal number with room to spare, both exponents in range.
__host__ __device__ inline bool closed_form_domain(double fs, double K, double T, double rT,
                                                   double cT) {
  return all(fs >= 0x1p-300, fs <= 0x1p+300, K >= 0x1p-300, K <= 0x1p+300, T >= 1e-290,
             fabs(rT) <= 200.0, fabs(cT) <= 200.0);
}

// Forward, discount factor and terms of a quote at a volatility.
struct ClosedForm {
  double F, D, sqT, isqT, s;
  ScaledTerms t;
};

__host__ __device__ __attribute__((always_inline)) inline bool closed_form(
    int model, double fs, double K, double T, double r, double q, double sigma, int theta,
    ClosedForm* o) {
  const double cT = model == kBlackScholesMerton ? minus(r, q) * T : r * T;
  const bool in = closed_form_domain(fs, K, T, r * T, cT);
  o->F = fs * growth_of<true>(model, T, r, q);
  o->D = fexp_prod<true>(-r, T);
  o->isqT = rsqrt(T);
  o->sqT = T * o->isqT;
  o->s = sigma * o->sqT;
  const double x = -fabs(log_ratio(o->F, K));
  return all(scaled_terms(o->F, K, o->D, x, o->s, theta, &o->t), in, ((theta + 1) & ~2) == 0);
}

// The same for a quote the scaled path has just solved: its total volatility
// s, and F, D, x and 1/sqrt(T) from its reduction.
__host__ __device__ __attribute__((always_inline)) inline bool closed_form_at(
    int model, const ScaledQuote& sq, double s, double fs, double K, double T, double r, double q,
    int theta, ClosedForm* o) {
  const double cT = model == kBlackScholesMerton ? minus(r, q) * T : r * T;
  o->F = sq.F;
  o->D = sq.D;
  o->isqT = sq.isqrtT;
  o->sqT = T * sq.isqrtT;
  o->s = s;
  return all(scaled_terms(sq.F, K, sq.D, sq.x, s, theta, &o->t),
             closed_form_domain(fs, K, T, r * T, cT));
}

// The Greeks and the partials of price_partials from those terms; `price` is
// the discounted price (Black-76 theta and rho read it).
__host__ __device__ inline Greeks greeks_of(const ClosedForm& c, int model, double fs, double T,
                                            double r, double q, double sigma, int theta,
                                          double price) {
  Greeks g;
  const double ifs = rcp(fs), dth = (double)theta;
  const double V = c.D * c.t.V;  // D F phi(d1)
  const double decay = 0.5 * sigma * V * c.isqT;
  const double dFN = dth * c.D * c.t.FN;
  g.vega = V * c.sqT;
  g.delta = dFN * ifs;
  g.gamma = V * ifs * (ifs * rcp(c.s));  // V/S^2 itself may leave the normal range
  if (model == kBlack76) {
    g.theta = fma(r, price, -decay);
    g.rho = -T * price;
  } else {
    const double dKN = dth * c.D * c.t.KN;
    g.theta = fma(-r, dKN, -decay);
    if (model == kBlackScholesMerton) g.theta = fma(q, dFN, g.theta);
    g.rho = T * dKN;
  }
  return g;
}

__host__ __device__ inline PricePartials partials_of(const ClosedForm& c, int model, double fs,
                                                     double K, double T, double r, double q,
                                                     double sigma, int theta, double price) {
  PricePartials o;
  const Greeks g = greeks_of(c, model, fs, T, r, q, sigma, theta, price);
  const double dth = (double)theta;
  o.dfs = g.delta;
  o.dK = -dth * c.D * c.t.KN * rcp(K);
  o.dT = -g.theta;
  o.dr = g.rho;
  o.dq = model == kBlackScholesMerton ? -dth * T * c.D * c.t.FN : 0.0;
  o.dsigma = g.vega;
  return o;
}

// Implicit-function adjoint of the implied volatility (the paper's section 3,
// "Differentiable IV"): with vega = dP/dsigma,
//   dsigma/dP = 1/vega,   dsigma/dX = -(dP/dX at fixed sigma)/vega,
// X in (S or F, K, T, r, q).  Returns the six partials.
struct IvGrad {
  double dP, dfs, dK, dT, dr, dq;
};

__host__ __device__ inline IvGrad implicit_gradient(const PricePartials& pp) {
  IvGrad o;
  const double iv = 1.0 / pp.dsigma;
  o.dP = iv;
  o.dfs = -pp.dfs * iv;
  o.dK = -pp.dK * iv;
  o.dT = -pp.dT * iv;
  o.dr = -pp.dr * iv;
  o.dq = -pp.dq * iv;
  return o;
}

__host__ __device__ __attribute__((always_inline)) inline IvGrad iv_gradient(int model, double fs, double K, double T,
                                              double r, double q, double sigma, int theta,
                                              double price) {
  const double F = forward_of(model, fs, T, r, q);
  const double D = fexp_prod(-r, T);
  return implicit_gradient(price_partials(model, fs, K, T, r, q, sigma, theta, F, D, price));
}

// Price at sigma from the normalised Black function (accurate in the wings):
// price = D sqrt(F K) b(x, s, theta), with b of a put or an in-the-money
// option obtained from the out-of-the-money call by parity.
__host__ __device__ __attribute__((always_inline)) inline double price_at(double F, double K, double D, double sigma,
                                           double sqrtT, int theta) {
  const double lx = log_moneyness(F, K);
  // out-of-the-money side: x_otm <= 0
  const bool itm = theta * lx > 0.0;
  const double x = -fabs(lx);
  const double bmax = fexp(0.5 * x);
  const NBlack nb = normalised_black(x, sigma * sqrtT, bmax);
  const double sq = sqrt(F) * sqrt(K);  // F K may leave the binary64 range
  double p = D * sq * nb.b;
  if (itm) p += D * (theta > 0 ? (F - K) : (K - F));
  return p;
}

}  // namespace fv
