// fv_calib.hip -- calibration of per-maturity SVI smiles on ragged Black-76
// chains through the differentiable implied volatility (the paper's use
// case of IV "inside differentiable pipelines for calibration", section 1,
// with the autograd-friendly IV of section 3).
//
// Model per maturity, raw parameters theta = (a, b~, rho~, m, s~):
//   b = softplus(b~), rho = tanh(rho~), s = softplus(s~),
//   w(k) = a + b (rho (k - m) + sqrt((k - m)^2 + s^2)),   k = ln(K/F),
//   sigma_SVI = sqrt(w / T).
// Loss over the N quotes: L = (1/N) sum (IV(P_B76(sigma_SVI)) - IV_target)^2.
// One step = three launches, all graph-capturable (no allocation, no host
// synchronisation, no memset), with a workspace the caller provides:
//   1. per maturity: the natural parameters into a table (the
//      softplus/tanh transforms run once per maturity, not once per quote);
//   2. flat over the quotes, one wave per 64 consecutive quotes: SVI ->
//      Black-76 price -> LBR implied volatility -> residual -> adjoint
//      (dIV/dP = 1/vega(IV), dP/dsigma = vega(sigma), dsigma/dw =
//      1/(2 sigma T)), then the sums over the wave's lanes, segmented by
//      maturity where it holds more than one; each (wave, maturity) run
//      stores its five sums at index wave + maturity (unique: along the
//      quotes both indices only grow, and each run changes at least one), so
//      no atomics are needed and results are bitwise reproducible; each
//      workgroup stores its sum of squared errors; the first thread also advances the
//      step counter and forms Adam's bias corrections;
//   3. eight lanes per maturity: the sums of its runs -> gradient -> Adam
//      update; one workgroup more sums the squared errors to the loss, in a
//      fixed order.
// The price is handed to the solver in the normalised coordinates it
// reduces every quote to: the Black-76 price of the model is
// D sqrt(F K) (b(x, s) + intrinsic), and the solver's reduction (undiscount,
// subtract the intrinsic value, divide by min(F, K)) takes it back to
// b(x, s)/b_max exactly in exact arithmetic, so the kernel passes that of the
// out-of-the-money side to the LBR solve without the round trip.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <atomic>
#include <mutex>
#include <string>

#include "../../include/fastvol.h"
#include "fv_csr.h"
#include "fv_host.h"
#include "fv_quote.h"

namespace {

constexpr int kCalibBlock = 256;
constexpr double kWMin = 1e-10;  // total variance floor: quotes below it are skipped

// Per-maturity record of the natural parameters (k_svi_prep), read by
// k_svi_grad and k_svi_adam.
enum NatField : int {
  kNatA, kNatMu,
  kNatIsqT,   // 1/sqrt(T)
  kNatB, kNatRho, kNatS,
  kNatSigB,   // softplus'(b~) = sigmoid(b~)
  kNatSigS,   // softplus'(s~) = sigmoid(s~)
  kNatCount
};
// Per (wave, maturity) run: the five sums of the adjoint.
enum SumField : int {
  kSumG,       // sum g_w,               g_w = dL/dw of a quote
  kSumGRt,     // sum g_w sqrt((k - m)^2 + s^2)
  kSumGDk,     // sum g_w (k - m)
  kSumGDkIrt,  // sum g_w (k - m) / sqrt((k - m)^2 + s^2)
  kSumGIrt,    // sum g_w / sqrt((k - m)^2 + s^2)
  kSumCount
};
constexpr int kRecord = 6;  // doubles of workspace per run: its sums, and one for block_e2
// Control block at the start of the workspace: Adam's bias corrections of
// the step.
enum CtlField : int { kCtlC1, kCtlC2, kCtlCount };

struct KSvi {
  int64_t n_chains, n_mat, n;
  const int64_t* chain_mat_off;
  const int64_t* mat_quote_off;
  const double *F, *r, *T, *K;
  const int8_t* flag;
  const double* iv_target;
};

__device__ __forceinline__ double softplus(double z) { return z > 30.0 ? z : log1p(exp(z)); }

// The transforms from one exponential each, e = e^{-|z|} (e^{-2|z|} for
// tanh):  softplus = max(z, 0) + ln(1 + e) with ln(1 + e) from the atanh form
// of 1 + e or, above sqrt2, of (1 + e)/2; sigmoid = 1/(1 + e) or e/(1 + e);
// tanh = (1 - e)/(1 + e), near 0 through e^{2z} - 1 without cancellation.
struct Soft {
  double value, slope;
};
__device__ __forceinline__ Soft softplus_of(double z) {
  const double e = fv::fexp(-fabs(z));
  const bool up = e > 0.41421356237309504880;
  const double l = fv::log_of(fv::fdiv(up ? e - 1.0 : e, up ? e + 3.0 : e + 2.0), up ? 1 : 0);
  const double i = fv::rcp(1.0 + e);
  return Soft{fmax(z, 0.0) + l, z < 0.0 ? e * i : i};
}
__device__ __forceinline__ double tanh_of(double z) {
  const double e = fv::fexp(-2.0 * fabs(z));
  double t = fv::fdiv(1.0 - e, 1.0 + e);
  const double r = 2.0 * fabs(z);
  if (r < 0.34) {
    double p = fv::coef::kExpQ[fv::kExpDeg];
#pragma unroll
    for (int i = fv::kExpDeg - 1; i >= 0; --i) p = fma(p, r, fv::coef::kExpQ[i]);
    const double m = fma(r * r, fma(r, p, 0.5), r);  // e^r - 1
    t = fv::fdiv(m, 2.0 + m);
  }
  return copysign(t, z);
}

constexpr int kWavesPerBlock = kCalibBlock / 64;
int64_t n_waves_of(int64_t n) { return (n + 63) / 64; }

// workspace layout (doubles): control block, per-maturity records, the runs'
// sums, then each gradient workgroup's sum of squared errors (there are at
// least as many runs as waves, so a double a run holds them).  ceil(n_mat / 4) more are
// part of the documented size and not used.
int64_t workspace_doubles(int64_t n_mat, int64_t n) {
  return kCtlCount + kNatCount * n_mat + (n_mat + 3) / 4 + kRecord * (n_waves_of(n) + n_mat);
}

struct Workspace {
  double* ctl;
  double* nat;
  double* part;
  double* e2;
};

Workspace carve(double* ws, int64_t n_mat, int64_t n) {
  Workspace w;
  w.ctl = ws;
  w.nat = ws + kCtlCount;
  w.part = w.nat + kNatCount * n_mat;
  w.e2 = w.part + kSumCount * (n_waves_of(n) + n_mat);
  return w;
}

// sqrt((k - m)^2 + s^2) and its reciprocal: the refined hardware reciprocal
// square root where the radicand is a normal number, the library square
// root otherwise (s underflowed to 0 at k = m)
__device__ __forceinline__ void svi_root(double u, double& rt, double& irt) {
  if (u >= 2.2250738585072014e-308) {
    irt = fv::rsqrt(u);
    rt = u * irt;
  } else {
    rt = sqrt(u);
    irt = 1.0 / rt;
  }
}

// One wave per workgroup: 7,243 maturities are 114 waves, one to a compute
// unit, and one chain of transforms long (3.2-4.8 us; 4.1-4.9 in workgroups of
// 256 with the library's log1p, exp and tanh).
constexpr int kPrepBlock = 64;
__global__ __launch_bounds__(kPrepBlock) void k_svi_prep(int64_t n_mat,
                                                         const double* __restrict__ T,
                                                         const double* __restrict__ theta,
                                                         double* __restrict__ nat) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= n_mat) return;
  const double* th = theta + 5 * m;
  const Soft b = softplus_of(th[1]), s = softplus_of(th[4]);
  double* o = nat + kNatCount * m;
  o[kNatA] = th[0];
  o[kNatMu] = th[3];
  o[kNatIsqT] = fv::rsqrt(T[m]);
  o[kNatB] = b.value;
  o[kNatRho] = tanh_of(th[2]);
  o[kNatS] = s.value;
  o[kNatSigB] = b.slope;
  o[kNatSigS] = s.slope;
}

// ------------------------------------------------------------ lane sums
// A lane's neighbour by a cross-lane move of the vector ALU (DPP), both words.
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi =
      (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kHalfMirror = 0x141;
constexpr int kRowRor = 0x120;  // + distance

// The sum over the 16 lanes of each row, in every lane of it.
__device__ __forceinline__ double row_sum(double v) {
  v += dpp<kRowRor + 8>(v);
  v += dpp<kRowRor + 4>(v);
  v += dpp<kRowRor + 2>(v);
  return v + dpp<kRowRor + 1>(v);
}
// The sum over the 8 lanes of each half row, in every lane of it.
__device__ __forceinline__ double half_row_sum(double v) {
  v += dpp<kQuadXor1>(v);
  v += dpp<kQuadXor2>(v);
  return v + dpp<kHalfMirror>(v);
}
// Halves the values in flight: a's sum over the two halves of the wave (of
// each pair of rows) in the lower one, b's in the upper.
__device__ __forceinline__ double fold32(double a, double b) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
  const auto hi =
      __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
         __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double fold16(double a, double b) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
  const auto hi =
      __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
         __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}

// One wave of the gradient: its runs' sums to `part`; returns its sum of
// squared errors, in lane 32.
__device__ __forceinline__ double grad_wave(const KSvi& c, int64_t wave,
                                            const double* __restrict__ nat,
                                            double* __restrict__ part) {
  const int lane = (int)__lane_id();
  const int64_t w0 = wave * 64;
  if (w0 >= c.n) return 0.0;  // wave-uniform
  fv::ChainCursor cur;
  cur.init(c.mat_quote_off, c.n_mat, c.chain_mat_off, c.n_chains, w0);
  const int64_t i = w0 + lane;
  int64_t m0, cc0;
  int key, cc;
  cur.slice(w0, min(w0 + 63, c.n - 1), m0, key, cc0, cc);
  const int64_t m = m0 + key;
  const double* rec = nat + kNatCount * m0 + (unsigned)(kNatCount * key);
  const double sa = rec[kNatA], sb = rec[kNatB], srho = rec[kNatRho], smu = rec[kNatMu],
               ss = rec[kNatS], isqT = rec[kNatIsqT];
  double v[kSumCount], e2 = 0.0;
#pragma unroll
  for (int j = 0; j < kSumCount; ++j) v[j] = 0.0;
  if (i < c.n) {
    const double tgt = (c.iv_target + w0)[(unsigned)lane], K = (c.K + w0)[(unsigned)lane];
    const double F = (c.F + cc0)[(unsigned)cc];
    double lfk = fv::log_ratio(F, K);  // ln(F/K) = -k
    // (its significands make a finite number of anything: a quote with no
    // logarithm, such as a padding strike of 0, stays NaN and is skipped)
    if (__builtin_expect(!fv::all(fv::positive_normal(F), fv::positive_normal(K)), 0))
      lfk = fv::flog(F * fv::rcp(K));
    const double dk = -lfk - smu;
    double rt, irt;
    svi_root(fma(dk, dk, ss * ss), rt, irt);
    const double w = fma(sb, fma(srho, dk, rt), sa);
    if (w > kWMin && fv::finite_d(tgt)) {
      const double iw = fv::rsqrt(w);
      const double s1 = w * iw;  // sigma sqrt(T)
      // out-of-the-money side: x = -|ln(F/K)| <= 0, beta = b(x, s1)
      const double x = -fabs(lfk);
      // IV(P(sigma)) through the LBR solver; where the model price is not
      // solvable in binary64 (b rounded onto 0 or onto its bound b_max) the
      // composite takes its exact value sigma and unit slope
      double s2 = s1;
      bool solved = false;
      if (x >= -128.0 && s1 > 1e-20 && s1 < 1e3) {
        double bh, ch;
        fv::scaled_value(x, s1, &bh, &ch);
        solved = fv::scaled_domain(x, bh, ch) && fv::lbr_solve_scaled(x, bh, ch, &s2);
      }
      if (__builtin_expect(!solved, 0)) {
        const double bmax = fv::fexp(0.5 * x);
        const fv::NBlack nb = fv::normalised_black(x, s1, bmax);
        solved = nb.b > 0.0 && nb.b < bmax;
        if (solved) {
          // ln beta from the evaluator's logarithmic parts (accurate also
          // where b is below the normal range)
          const double ln_beta = nb.lnbp + fv::flog(nb.ratio);
          s2 = fv::lbr_solve(x, nb.b, bmax, ln_beta, fv::kLbrMinSteps, fv::kLbrMaxSteps,
                             fv::kLbrStepTol).s;
        }
      }
      double ratio = 1.0;
      if (solved) {
        // vega(v) = D F phi(d1(v)) sqrt(T); only vega(sigma)/vega(iv) enters:
        // with s = v sqrt(T) and d1 = ln(F/K)/s + s/2,
        //   ln(vega(s1)/vega(s2)) = -(d1(s1)^2 - d1(s2)^2)/2
        //                         = -(s1^2 - s2^2)(1/4 - L^2)/2,  L = ln(F/K)/(s1 s2),
        // which vanishes up to rounding (IV(P(sigma)) = sigma)
        const double ds = s1 - s2;
        const double L = lfk * (fabs(ds) < 1e-9 * s1 ? iw * iw : fv::rcp(s1 * s2));
        const double dl = -0.5 * ds * (s1 + s2) * fma(-L, L, 0.25);
        ratio = fabs(dl) < 1e-8 ? 1.0 + dl : fv::fexp(dl);
      }
      const double e = s2 * isqT - tgt;
      // dL/dw = (2 e/N) ratio / (2 sigma T), with 1/N applied per maturity sum
      const double g_w = e * ratio * (iw * isqT);
      v[kSumG] = g_w;
      v[kSumGRt] = g_w * rt;
      v[kSumGDk] = g_w * dk;
      v[kSumGDkIrt] = g_w * dk * irt;
      v[kSumGIrt] = g_w * irt;
      e2 = e * e;
    }
  }
  if (__builtin_amdgcn_readlane(key, 63) == 0) {
    // One maturity, the rule: all six sums at once, halving the values in
    // flight with each of the first two folds (lanes by halves, then rows),
    // 11 folds and row steps in the vector ALU where the segmented form below
    // takes 36 through LDS.
    const double w01 = fold16(fold32(v[0], v[3]), fold32(v[1], v[4]));
    const double w2 = fold32(v[2], e2);
    const double y = row_sum(w01), z = row_sum(fold16(w2, w2));
    // rows 0 .. 3 hold sums 0, 1, 3, 4; the lower half 2, the upper e2 (lane 32
    // is read)
    if ((lane & 15) == 0) {
      const int row = lane >> 4;
      double* o = part + kSumCount * (wave + m);
      o[row + (row >> 1)] = y;
      if (row == 0) o[2] = z;
    }
    return z;
  }
  // Segmented suffix sums over the lanes keyed by maturity: the maturity is
  // non-decreasing along the lanes, so equal keys at distance `off` enclose
  // a run of equal keys and each lane ends with the sum from itself to the
  // end of its run.  Lanes past the last quote carry zeros and the last
  // quote's maturity.
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int nk = __shfl_down(key, off);
    const bool add = lane + off < 64 && nk == key;
#pragma unroll
    for (int j = 0; j < kSumCount; ++j) {
      const double o = __shfl_down(v[j], off);
      if (add) v[j] += o;
    }
  }
  const int pk = __shfl_up(key, 1);
  if ((lane == 0 || pk != key) && i < c.n) {
    double* o = part + kSumCount * (wave + m);
#pragma unroll
    for (int j = 0; j < kSumCount; ++j) o[j] = v[j];
  }
  return row_sum(fold16(fold32(e2, e2), fold32(e2, e2)));
}

// Bound by the vector ALU (805 instructions per 64 quotes, an eighth of them
// the location and a tenth the sums; 1,347 with the solve in binary64 and the
// sums through LDS): 2.1M quotes in 7,529 maturities 47 us (88 with those).  At least 7 waves per SIMD: free, it takes 74
// registers, two too many, and ten steps take 530 us for 517 (below 0.5M
// quotes, where waves are few, the floor costs 1%).  Two slices per wave, as
// in the ragged solve, were 1 to 15% slower.
__global__ __launch_bounds__(kCalibBlock) __attribute__((amdgpu_waves_per_eu(7))) void k_svi_grad(
    KSvi c, const double* __restrict__ nat, double* __restrict__ ctl, double* __restrict__ part,
    double* __restrict__ block_e2, int64_t* __restrict__ step, double b1, double b2) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    // the step's counter and bias corrections; nothing else in this launch
    // reads them, k_svi_adam runs after it on the stream
    const int64_t t = *step + 1;
    *step = t;
    ctl[kCtlC1] = 1.0 - pow(b1, (double)t);
    ctl[kCtlC2] = 1.0 - pow(b2, (double)t);
  }
  // the wave's number as a scalar, so that the location runs on the scalar
  // unit
  const int wib = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const double e2 = grad_wave(c, (int64_t)blockIdx.x * kWavesPerBlock + wib, nat, part);
  // one squared-error sum per workgroup: the loss is summed by one workgroup,
  // which a sum per wave kept 2.5 us longer than the update beside it
  __shared__ double wave_e2[kWavesPerBlock];
  if (__lane_id() == 32) wave_e2[wib] = e2;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = wave_e2[0];
    for (int j = 1; j < kWavesPerBlock; ++j) t += wave_e2[j];
    block_e2[blockIdx.x] = t;
  }
}

// Adam with the counter and bias corrections k_svi_grad set, eight lanes per
// maturity (5.3 runs each on the 500-chain problem): lane l sums the runs l,
// l + 8, ... in order, a fixed butterfly over the eight completes the five
// sums, and lane j < 5 updates parameter j.  One workgroup more, the first,
// sums the workgroups' squared errors to the loss in a fixed order meanwhile.
// Launch latency and a chain of dependent loads bound it: 7,243 maturities
// 4.9 us, loss included (9.9 and 4.6 us with a wave per maturity and a launch
// for the loss).
constexpr int kAdamBlock = 1024;
constexpr int kAdamPerBlock = kAdamBlock / 8;
__global__ __launch_bounds__(kAdamBlock) void k_svi_adam(
    int64_t n_mat, int64_t n, const int64_t* __restrict__ mat_quote_off,
    const double* __restrict__ nat, const double* __restrict__ part, double* __restrict__ theta,
    double* __restrict__ am, double* __restrict__ av, double* __restrict__ grad,
    const double* __restrict__ ctl, const double* __restrict__ block_e2, int64_t blocks,
    const int64_t* __restrict__ step, double* __restrict__ loss, int64_t loss_len, double lr,
    double b1, double b2, double eps) {
  if (blockIdx.x == 0) {
    if (loss_len == 0) return;
    __shared__ double red[kAdamBlock / 64];
    double a = 0.0;
#pragma unroll 8
    for (int64_t w = threadIdx.x; w < blocks; w += kAdamBlock) a += block_e2[w];
    a = row_sum(fold16(fold32(a, a), fold32(a, a)));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) {
      // (in pairs: the sixteen sums one after the other: mean error 1.2e-16 for 1.0e-16)
#pragma unroll
      for (int h = kAdamBlock / 128; h > 0; h >>= 1)
#pragma unroll
        for (int j = 0; j < h; ++j) red[j] += red[j + h];
      const double t = red[0];
      const int64_t k = *step;
      if (k >= 1 && k <= loss_len) loss[k - 1] = t * (1.0 / (double)n);
    }
    return;
  }
  const int64_t m = (int64_t)(blockIdx.x - 1) * kAdamPerBlock + (threadIdx.x >> 3);
  const int sub = (int)(threadIdx.x & 7);
  double S[kSumCount];
#pragma unroll
  for (int j = 0; j < kSumCount; ++j) S[j] = 0.0;
  // everything the update reads that does not hang on the offsets, ahead of
  // the runs: two loads deep instead of four
  const int64_t mc = m < n_mat ? m : n_mat - 1;
  const int64_t k = 5 * mc + (sub < 5 ? sub : 4);
  const double* q = nat + kNatCount * mc;
  const double b = q[kNatB], rho = q[kNatRho], sg = q[kNatS], sig_b = q[kNatSigB],
               sig_s = q[kNatSigS];
  const double am0 = am[k], av0 = av[k], th0 = theta[k], c1 = ctl[kCtlC1], c2 = ctl[kCtlC2];
  const int64_t q0 = mat_quote_off[mc], q1 = mat_quote_off[mc + 1];
  const bool empty = q1 <= q0;  // an empty maturity has no runs and no record
  if (!empty) {
    for (int64_t w = (q0 >> 6) + sub; w <= (q1 - 1) >> 6; w += 8) {
      const double* o = part + kSumCount * (w + mc);
#pragma unroll
      for (int j = 0; j < kSumCount; ++j) S[j] += o[j];
    }
  }
#pragma unroll
  for (int j = 0; j < kSumCount; ++j) S[j] = half_row_sum(S[j]);
  if (m >= n_mat || sub >= 5) return;
  double g = 0.0;
  if (!empty) {
    // dL/dtheta = (1/N) sum g_w dw/dtheta with
    //   dw/da = 1, dw/db~ = (rho dk + rt) sigmoid(b~), dw/drho~ = b dk (1 - rho^2),
    //   dw/dm = -b (rho + dk/rt), dw/ds~ = b (s/rt) sigmoid(s~)
    switch (sub) {
      case 0: g = S[kSumG]; break;
      case 1: g = fma(rho, S[kSumGDk], S[kSumGRt]) * sig_b; break;
      case 2: g = b * (1.0 - rho * rho) * S[kSumGDk]; break;
      case 3: g = -b * fma(rho, S[kSumG], S[kSumGDkIrt]); break;
      default: g = b * sg * sig_s * S[kSumGIrt]; break;
    }
    g *= 1.0 / (double)n;
  }
  grad[k] = g;
  const double mo = b1 * am0 + (1.0 - b1) * g;
  const double vo = b2 * av0 + (1.0 - b2) * g * g;
  am[k] = mo;
  av[k] = vo;
  theta[k] = th0 - lr * (mo / c1) / (sqrt(vo / c2) + eps);
}

__global__ void k_svi_vols(KSvi c, const double* __restrict__ theta, double* __restrict__ out) {
  const int64_t m = blockIdx.x;
  const double T = c.T[m];
  int64_t lo = 0, hi = c.n_chains;  // chain of maturity m: largest lo with off[lo] <= m
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (c.chain_mat_off[mid] <= m) lo = mid; else hi = mid;
  }
  const double F = c.F[lo];
  const double* th = theta + 5 * m;
  const double a = th[0], b = softplus(th[1]), rho = tanh(th[2]), mu = th[3], s = softplus(th[4]);
  for (int64_t i = c.mat_quote_off[m] + threadIdx.x; i < c.mat_quote_off[m + 1];
       i += blockDim.x) {
    const double dk = log(c.K[i] / F) - mu;
    const double w = a + b * (rho * dk + sqrt(dk * dk + s * s));
    out[i] = w > 0.0 ? sqrt(w / T) : __builtin_nan("");
  }
}

int check_problem(const fv_svi_problem* p) {
  if (!p) return fvh::fail(FV_E_INVALID_ARG, "problem pointer is NULL");
  const fv_chains& c = p->chains;
  if (c.n_chains <= 0 || c.n_maturities <= 0 || c.n_quotes <= 0)
    return fvh::fail(FV_E_INVALID_ARG, "empty or negative chain sizes");
  if (c.n_maturities > 0x7fffffff || c.n_quotes > ((int64_t)1 << 46))
    return fvh::fail(FV_E_INVALID_ARG, "too many maturities or quotes");
  if (!c.chain_mat_off || !c.mat_quote_off || !c.F || !c.r || !c.T || !c.K || !c.flag)
    return fvh::fail(FV_E_INVALID_ARG, "NULL chain array");
  return FV_OK;
}

KSvi to_k(const fv_svi_problem* p) {
  KSvi k;
  const fv_chains& c = p->chains;
  k.n_chains = c.n_chains;
  k.n_mat = c.n_maturities;
  k.n = c.n_quotes;
  k.chain_mat_off = c.chain_mat_off;
  k.mat_quote_off = c.mat_quote_off;
  k.F = c.F;
  k.r = c.r;
  k.T = c.T;
  k.K = c.K;
  k.flag = c.flag;
  k.iv_target = p->iv_target;
  return k;
}

// The three launches of one step, with the workspace `ws` (at least
// workspace_doubles(n_mat, n) doubles, checked by the callers).
int launch_step(const fv_svi_problem* p, double* theta, double* adam_m, double* adam_v,
                int64_t* step, double* grad, double* ws, double* loss, int64_t loss_len,
                void* stream) {
  if (!p->iv_target || !theta || !adam_m || !adam_v || !step || !grad)
    return fvh::fail(FV_E_INVALID_ARG, "NULL parameter, state or gradient array");
  if (loss_len < 0) return fvh::fail(FV_E_INVALID_ARG, "loss_len < 0");
  if (!(p->lr > 0.0) || !(p->beta1 >= 0.0 && p->beta1 < 1.0) ||
      !(p->beta2 >= 0.0 && p->beta2 < 1.0) || !(p->eps > 0.0))
    return fvh::fail(FV_E_INVALID_ARG, "Adam hyper-parameters out of range");
  const KSvi k = to_k(p);
  hipStream_t s = (hipStream_t)stream;
  const Workspace w = carve(ws, k.n_mat, k.n);
  const int64_t blocks = (n_waves_of(k.n) + kWavesPerBlock - 1) / kWavesPerBlock;
  const int64_t nb = (k.n_mat + kAdamPerBlock - 1) / kAdamPerBlock + 1;
  k_svi_prep<<<dim3((unsigned)((k.n_mat + kPrepBlock - 1) / kPrepBlock)), dim3(kPrepBlock), 0,
               s>>>(k.n_mat, k.T, theta, w.nat);
  k_svi_grad<<<dim3((unsigned)blocks), dim3(kCalibBlock), 0, s>>>(
      k, w.nat, w.ctl, w.part, w.e2, step, p->beta1, p->beta2);
  k_svi_adam<<<dim3((unsigned)nb), dim3(kAdamBlock), 0, s>>>(
      k.n_mat, k.n, k.mat_quote_off, w.nat, w.part, theta, adam_m, adam_v, grad, w.ctl, w.e2,
      blocks, step, loss, loss ? loss_len : 0, p->lr, p->beta1, p->beta2, p->eps);
  return fvh::launched("fv_svi_adam_step");
}

// Workspace of the allocation-free step: one array per GPU, part of the
// library's code object (each device that loads the library holds its own
// copy until the process ends).  Host code never passes `scratch` itself to
// a kernel (on the host the name is only a stand-in): it takes the device
// address from hipGetSymbolAddress, once per device, with that device
// current.
constexpr int64_t kScratchDoubles = (int64_t)1 << 20;  // 8 MiB
constexpr int kMaxDevices = 64;
static __device__ __align__(256) double scratch[kScratchDoubles];

std::mutex g_scratch_mu;
std::atomic<double*> g_scratch_ptr[kMaxDevices];

// Device address of the current device's `scratch` into *out; FV_OK or an
// FV_E_* code with its text set.
int scratch_of_current_device(double** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fvh::fail(FV_E_HIP, std::string("hipGetDevice: ") + hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices)
    return fvh::fail(FV_E_UNSUPPORTED, "device ordinal beyond the 64 the library tracks");
  double* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!ptr) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    ptr = g_scratch_ptr[dev].load(std::memory_order_relaxed);
    if (!ptr) {
      void* p = nullptr;
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !p)
        return fvh::fail(FV_E_HIP, std::string("hipGetSymbolAddress(scratch): ") +
                                       (e != hipSuccess ? hipGetErrorString(e) : "NULL address"));
      ptr = static_cast<double*>(p);
      g_scratch_ptr[dev].store(ptr, std::memory_order_release);
    }
  }
  *out = ptr;
  return FV_OK;
}

}  // namespace

extern "C" {

int64_t fv_svi_workspace_size(const fv_svi_problem* p) {
  const int rc = check_problem(p);
  if (rc) return rc;
  return workspace_doubles(p->chains.n_maturities, p->chains.n_quotes);
}

int fv_svi_adam_step(const fv_svi_problem* p, double* theta, double* adam_m, double* adam_v,
                     int64_t* step, double* grad, double* workspace, int64_t workspace_len,
                     double* loss, int64_t loss_len, void* stream) {
  int rc = check_problem(p);
  if (rc) return rc;
  if (!workspace) return fvh::fail(FV_E_INVALID_ARG, "workspace is NULL");
  if (workspace_len < workspace_doubles(p->chains.n_maturities, p->chains.n_quotes))
    return fvh::fail(FV_E_INVALID_ARG, "workspace smaller than fv_svi_workspace_size()");
  return launch_step(p, theta, adam_m, adam_v, step, grad, workspace, loss, loss_len, stream);
}

int fv_svi_adam_step_noalloc(const fv_svi_problem* p, double* theta, double* adam_m,
                             double* adam_v, int64_t* step, double* grad, double* loss,
                             int64_t loss_len, void* stream) {
  int rc = check_problem(p);
  if (rc) return rc;
  const int64_t need = workspace_doubles(p->chains.n_maturities, p->chains.n_quotes);
  if (need > kScratchDoubles)
    return fvh::fail(FV_E_INVALID_ARG,
                     "problem needs " + std::to_string(need) +
                         " doubles of workspace; the allocation-free step holds at most " +
                         std::to_string(kScratchDoubles) + " (8 MiB): use fv_svi_adam_step");
  double* ws = nullptr;
  rc = scratch_of_current_device(&ws);
  if (rc) return rc;
  return launch_step(p, theta, adam_m, adam_v, step, grad, ws, loss, loss_len, stream);
}

int fv_svi_vols(const fv_svi_problem* p, const double* theta, double* sigma_out, void* stream) {
  int rc = check_problem(p);
  if (rc) return rc;
  if (!theta || !sigma_out) return fvh::fail(FV_E_INVALID_ARG, "NULL theta or output");
  const KSvi k = to_k(p);
  k_svi_vols<<<dim3((unsigned)k.n_mat), dim3(kCalibBlock), 0, (hipStream_t)stream>>>(k, theta,
                                                                                    sigma_out);
  return fvh::launched("fv_svi_vols");
}

}  // extern "C"
