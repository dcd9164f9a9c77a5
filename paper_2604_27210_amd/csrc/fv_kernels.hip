// fv_kernels.hip -- gfx950 kernels and the C ABI declared in include/fastvol.h.
//
// Every kernel is a single pass over struct-of-arrays inputs: each lane loads
// its quote once (consecutive lanes read consecutive quotes, so every load of
// a wave is one contiguous segment), keeps the whole solve in registers and
// stores once.  One quote per thread; a wave of the ragged kernel takes one
// or two consecutive 64-quote slices.  Divergent regions (solver branches, a
// further step, quotes outside the scaled forms' domain) are plain per-lane
// control flow: the hardware skips a side whose exec mask is empty, so a wave
// pays only for the branches its own lanes take.  The Halley kernels compact
// the lanes that need more (bisection, the general solve) with wave ballots
// into an LDS queue and work the packed queue off afterwards.
#include <hip/hip_runtime.h>

#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <string>
#include <vector>

#include "../../include/fastvol.h"
#include "fv_f32.h"
#include "fv_host.h"
#include "fv_csr.h"
#include "fv_quote.h"

// Error state shared by every entry point of the library (fv_host.h).
namespace fvh {
thread_local std::string g_last_error;
int fail(int code, const std::string& msg) {
  g_last_error = msg;
  return code;
}
int launched(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FV_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
  return FV_OK;
}
}  // namespace fvh

namespace {

using fv::Greeks;
using fv::IvGrad;
using fv::LbrResult;
using fv::Reduced;

// ------------------------------------------------------------- arguments
struct KQuotes {
  int64_t n;
  fv_arg price, fs, K, T, r, q;
  const int8_t* flag;
  int8_t flag_value;
  int hsteps;  // Halley steps before the bisection fallback (fv_set_halley_steps)
};

// A field's value for quote i: its array entry, or its broadcast value.
// ARR = true is the specialisation for calls whose per-quote fields are all
// arrays (checked on the host): the pointer-or-value choice per field and
// its condition, which the solver kernels otherwise keep across the whole
// solve, disappear.
template <bool ARR = false>
__device__ __forceinline__ double ld(const fv_arg& a, int64_t i) {
  return ARR ? a.ptr[i] : (a.ptr ? a.ptr[i] : a.value);
}
// The same for quote b + t, b uniform over the workgroup and t below 2^16:
// the base moves by scalar instructions and every field shares one 32-bit
// lane offset, where a 64-bit index costs a vector add per field.
template <bool ARR>
__device__ __forceinline__ double ld(const fv_arg& a, int64_t b, unsigned t) {
  return ARR ? (a.ptr + b)[t] : (a.ptr ? (a.ptr + b)[t] : a.value);
}
template <bool ARR>
__device__ __forceinline__ int ldflag(const KQuotes& q, int64_t b, unsigned t) {
  return ARR ? (int)(q.flag + b)[t] : (q.flag ? (int)(q.flag + b)[t] : (int)q.flag_value);
}
template <bool ARR = false>
__device__ __forceinline__ int ldflag(const KQuotes& q, int64_t i) {
  return ARR ? (int)q.flag[i] : (q.flag ? (int)q.flag[i] : (int)q.flag_value);
}

// The kernel's argument block (its one parameter, an A), read again where it
// is asked for: pointers that are needed once, at the end or on a rare path,
// do not take up scalar registers until then (there the polynomials'
// constants fill them, and what does not fit is moved to vector registers
// and back, two instructions a value).
template <class A>
__device__ __forceinline__ const A* late_args() {
  uint32_t zero;
  asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
  return (const A*)((const __attribute__((address_space(4))) char*)
                        __builtin_amdgcn_kernarg_segment_ptr() + zero);
}

// A pointer read that way, as one to global memory (the compiler knows that of
// parameters only, and would take the slower flat accesses).
template <class V>
__device__ __forceinline__ __attribute__((address_space(1))) V* global_ptr(V* p) {
  return (__attribute__((address_space(1))) V*)p;
}

struct GreekOut {
  double* p[5];
  int any;
};
// Entry b + t (split as for ld) of each output row that is wanted.
template <int N>
__device__ __forceinline__ void store_rows(double* const* rows, int64_t b, unsigned t,
                                           const double (&v)[N]) {
#pragma unroll
  for (int j = 0; j < N; ++j)
    if (double* p = rows[j]) (global_ptr(p) + b)[t] = v[j];
}
__device__ __forceinline__ void store_greeks(const GreekOut& g, int64_t b, unsigned t,
                                             const Greeks& gr) {
  store_rows<5>(g.p, b, t, {gr.delta, gr.gamma, gr.vega, gr.theta, gr.rho});
}
__device__ __forceinline__ Greeks no_greeks() {
  const double nan = __builtin_nan("");
  return Greeks{nan, nan, nan, nan, nan};
}

// Largest workgroup the kernels are compiled for (8 waves).
constexpr int kMaxBlock = 512;
// Minimum resident waves per SIMD the solver kernels are register-allocated
// for.  LBR takes 56 VGPRs (8 waves) at a floor of 4, Halley 70 (7 waves) at
// 6; floors of 4 to 8 are within 1% for both (3M quotes, Halley: 54.3, 54.3,
// 54.1 and 54.5 us at 4, 6, 7 and 8 on one card).  The fused-Greeks variants
// take 80 to 84 at a floor of 2, which is as fast as one of 6 or 7 (26.1 us).
#ifndef FV_LBR_WAVES_PER_EU
#define FV_LBR_WAVES_PER_EU 4
#endif
#ifndef FV_HALLEY_WAVES_PER_EU
#define FV_HALLEY_WAVES_PER_EU 6
#endif
#define FV_WAVES_LBR(GREEKS) ((GREEKS) ? 2 : FV_LBR_WAVES_PER_EU)
#define FV_WAVES_HALLEY(GREEKS) ((GREEKS) ? 2 : FV_HALLEY_WAVES_PER_EU)
// The ragged kernel: 8 waves per SIMD (64 VGPRs; free, it takes 66 and 72).
// 8.4M quotes, LBR 135 us against 137 at a floor of 6, Halley 145 against 149.
#ifndef FV_CHAINS_WAVES_PER_EU
#define FV_CHAINS_WAVES_PER_EU 8
#endif

constexpr int kHalleySteps = 8;  // the paper's count; the default of fv_set_halley_steps
constexpr int kMaxHalleySteps = 64;
constexpr double kBisectTol = 1e-13;

// A value the compiler cannot follow: what is loaded or computed from it is
// loaded or computed again, not kept in registers from an earlier use.
template <class V>
__device__ __forceinline__ V opaque(V i) {
  asm volatile("" : "+v"(i));
  return i;
}

// The closed-form kernels below (price, Greeks, adjoints) are bound by
// memory: one evaluation and three exponentials a quote (266 to 363 vector
// instructions, 340 to 500 with the general forms) against 57 to 113 bytes.
// 5M BSM prices: 57 to 60 us (70 before; 55 at the 5.2 TB/s of a copy), 2M
// Black-76 Greeks 29 to 37 us (45; 31), the adjoint of 1M BSM quotes 20 to 22
// us (27; 22, part of it served from cache).  One quote per thread, every field
// on a scalar base.  Quotes outside the scaled forms' domain take the general
// ones, read again from memory.

// Inputs of a quote at a volatility.
struct SigmaQuote {
  double fs, K, T, r, q, sigma;
  int th;
};
// Arguments of the closed-form kernels: `up` is the upstream gradient of the
// adjoints.
struct FormArgs {
  KQuotes q;
  fv_arg sigma;
  const double* up;
  double* out[6];
};

template <int MODEL>
__device__ __forceinline__ SigmaQuote load_quote(const FormArgs& a, int64_t b, unsigned t) {
  SigmaQuote v;
  v.fs = ld<false>(a.q.fs, b, t);
  v.K = ld<false>(a.q.K, b, t);
  v.T = ld<false>(a.q.T, b, t);
  v.r = ld<false>(a.q.r, b, t);
  v.q = MODEL == fv::kBlackScholesMerton ? ld<false>(a.q.q, b, t) : 0.0;
  v.sigma = ld<false>(a.sigma, b, t);
  v.th = ldflag<false>(a.q, b, t);
  return v;
}

// The pricing domain (sigma may be zero for a price).
__device__ __forceinline__ bool price_domain(const SigmaQuote& v) {
  return fv::finite_d(v.fs) && fv::finite_d(v.K) && fv::finite_d(v.T) && fv::finite_d(v.r) &&
         fv::finite_d(v.q) && fv::finite_d(v.sigma) && v.fs > 0.0 && v.K > 0.0 && v.T > 0.0 &&
         v.sigma >= 0.0 && (v.th == 1 || v.th == -1);
}

template <int MODEL>
__device__ __forceinline__ SigmaQuote load_late(int64_t i) {
  const FormArgs* a = late_args<FormArgs>();
  i = opaque(i);
  SigmaQuote v;
  v.fs = ld(a->q.fs, i);
  v.K = ld(a->q.K, i);
  v.T = ld(a->q.T, i);
  v.r = ld(a->q.r, i);
  v.q = MODEL == fv::kBlackScholesMerton ? ld(a->q.q, i) : 0.0;
  v.sigma = ld(a->sigma, i);
  v.th = ldflag(a->q, i);
  return v;
}

// ------------------------------------------------------------- price
template <int MODEL>
__global__ __launch_bounds__(kMaxBlock) void k_price(FormArgs args) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x;
  const unsigned t = threadIdx.x;
  if ((int64_t)t >= args.q.n - b) return;
  const SigmaQuote v = load_quote<MODEL>(args, b, t);
  fv::ClosedForm c;
  const bool fast = fv::closed_form(MODEL, v.fs, v.K, v.T, v.r, v.q, v.sigma, v.th, &c);
  double p = c.D * c.t.P;
  if (__builtin_expect(!fast, 0)) {
    const SigmaQuote w = load_late<MODEL>(b + t);
    p = __builtin_nan("");
    if (price_domain(w)) {
      const double F = fv::forward_of(MODEL, w.fs, w.T, w.r, w.q);
      const double D = fv::fexp_prod(-w.r, w.T);
      p = fv::price_at(F, w.K, D, w.sigma, fv::sqrt_pos(w.T), w.th);
    }
  }
  (global_ptr(late_args<FormArgs>()->out[0]) + b)[t] = p;
}

// The general solve of quote i, from its inputs in memory: neither they nor
// what the scaled path derived from them stay in registers across that path
// for the sake of a rare quote.
template <int MODEL, bool ARR>
__device__ __forceinline__ void lbr_general_at(const KQuotes& q, int64_t i, double* sg, uint8_t* st,
                                               fv::ScaledQuote* sq, uint32_t* trace = nullptr) {
  i = opaque(i);
  fv::lbr_general(MODEL, ld<ARR>(q.price, i), ld<ARR>(q.fs, i), ld<ARR>(q.K, i), ld<ARR>(q.T, i),
                  ld<ARR>(q.r, i), MODEL == fv::kBlackScholesMerton ? ld<ARR>(q.q, i) : 0.0,
                  ldflag<ARR>(q, i), sg, st, sq, trace);
}

// Arguments of the implied-volatility kernels.
struct IvArgs {
  KQuotes q;
  double* sig_out;
  uint8_t* st_out;
  GreekOut g;
};

// The fused Greeks of a quote of status st at its volatility sg (s in total),
// NaN where it has none.
template <int MODEL>
__device__ __forceinline__ Greeks greeks_solved(uint8_t st, bool general,
                                                const fv::ScaledQuote& sq, double s, double sg,
                                                double P, double fs, double K, double T, double r,
                                                double qy, int th) {
  Greeks gr = no_greeks();
  bool fast = false;
  if (!general) {
    fv::ClosedForm c;
    fast = fv::closed_form_at(MODEL, sq, s, fs, K, T, r, qy, th, &c);
    gr = fv::greeks_of(c, MODEL, fs, T, r, qy, sg, th, P);
  }
  if (__builtin_expect(!fast, 0)) {
    gr = no_greeks();
    if (st == fv::kQOk)
      gr = fv::greeks_at(MODEL, opaque(fs), opaque(K), opaque(T), opaque(r), opaque(qy), sg, th,
                         sq.F, sq.D, P);
  }
  return st == fv::kQOk ? gr : no_greeks();
}

// ------------------------------------------------------------- IV: LBR
// Bound by the vector ALU's issue rate: 584 vector instructions per quote,
// every side of the guess a mixed wave takes included (1,157 with the guess
// and the first step in binary64).  10M wide-wing BSM quotes: 156 to 159 us
// (355 with those), 1M BS quotes with the five Greeks: 26 to 27 us (54).
// One quote per thread: with a loop over several the compiler keeps the
// polynomials' constants in registers across the whole solve, 110 VGPRs in
// place of 55, and the book took 220 us where it then took 190.
template <int MODEL, bool GREEKS, bool ARR>
__global__ __launch_bounds__(kMaxBlock)
__attribute__((amdgpu_waves_per_eu(FV_WAVES_LBR(GREEKS)))) void k_iv_lbr(IvArgs args) {
  const KQuotes& q = args.q;
  const int64_t b = (int64_t)blockIdx.x * blockDim.x;
  const unsigned t = threadIdx.x;
  if ((int64_t)t >= q.n - b) return;
  const double P = ld<ARR>(q.price, b, t), fs = ld<ARR>(q.fs, b, t), K = ld<ARR>(q.K, b, t),
               T = ld<ARR>(q.T, b, t), r = ld<ARR>(q.r, b, t);
  const double qy = MODEL == fv::kBlackScholesMerton ? ld<ARR>(q.q, b, t) : 0.0;
  const int th = ldflag<ARR>(q, b, t);
  fv::ScaledQuote sq = fv::scaled_quote(MODEL, P, fs, K, T, r, qy, th);
  uint8_t st = sq.status;
  double sg = st == fv::kQAtIntrinsic ? 0.0 : __builtin_nan("");
  bool general = sq.general;
  double s = 0.0;
  if (st == fv::kQOk && !general) {
    general = !fv::lbr_solve_scaled(sq.x, sq.bh, sq.ch, &s);
    sg = s * sq.isqrtT;
  }
  if (__builtin_expect(general, 0)) {
    const KQuotes& late = late_args<IvArgs>()->q;
    lbr_general_at<MODEL, ARR>(late, b + t, &sg, &st, &sq);
  }
  const auto* out = late_args<IvArgs>();
  (global_ptr(out->sig_out) + b)[t] = sg;
  if (uint8_t* st_out = out->st_out) (global_ptr(st_out) + b)[t] = st;
  if (GREEKS) {
    const Greeks gr = greeks_solved<MODEL>(st, general, sq, s, sg, P, fs, K, T, r, qy, th);
    store_greeks(out->g, b, t, gr);
  }
}

// Arguments of the diagnostic kernels.
struct TraceArgs {
  KQuotes q;
  uint32_t* out;
};

// Diagnostic twin of k_iv_lbr: the same per-quote solve, recording the path
// each quote takes (guess region, evaluation forms, number of steps).
template <int MODEL>
__global__ __launch_bounds__(kMaxBlock) void k_lbr_trace(TraceArgs args) {
  const KQuotes& q = args.q;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= q.n) return;
  const double P = ld(q.price, i), fs = ld(q.fs, i), K = ld(q.K, i), T = ld(q.T, i),
               r = ld(q.r, i);
  const double qy = MODEL == fv::kBlackScholesMerton ? ld(q.q, i) : 0.0;
  fv::ScaledQuote sq = fv::scaled_quote(MODEL, P, fs, K, T, r, qy, ldflag(q, i));
  uint32_t code = 0xFFFFFFFFu;  // not solved (status != OK)
  bool general = sq.general;
  if (sq.status == fv::kQOk && !general) {
    double s;
    general = !fv::lbr_solve_scaled(sq.x, sq.bh, sq.ch, &s, &code);
  }
  if (general) {
    double sg;
    uint8_t st;
    code = 0xFFFFFFFFu;
    lbr_general_at<MODEL, false>(q, i, &sg, &st, &sq, &code);
  }
  args.out[i] = code;
}

// The Halley iteration of one quote: the scaled solve, or the general one for
// a quote outside its domain.  Returns the status; hs is set where it is OK,
// sq always.
template <int MODEL>
__device__ __forceinline__ uint8_t halley_quote(double P, double fs, double K, double T, double r,
                                                double qy, int th, int steps,
                                                fv::HalleyState* hs, fv::ScaledQuote* sq) {
  *sq = fv::scaled_quote(MODEL, P, fs, K, T, r, qy, th);
  uint8_t st = sq->status;
  if (__builtin_expect(sq->general, 0)) {
    const Reduced rd = fv::reduce_quote(MODEL, opaque(P), opaque(fs), opaque(K), opaque(T),
                                        opaque(r), opaque(qy), th);
    st = rd.status;
    if (st == fv::kQOk) *hs = fv::halley_solve(rd.x, rd.beta, rd.bmax, rd.lnb, steps);
    sq->F = rd.F;  // an extreme exponent or maturity made nothing of scaled_quote's
    sq->D = rd.D;
    sq->isqrtT = rd.isqrtT;
  } else if (st == fv::kQOk) {
    *hs = fv::halley_solve_scaled(sq->x, sq->bh, sq->ch, steps);
  }
  return st;
}

// Diagnostic twin of k_iv_halley: the number of Halley steps each quote
// takes, with bit 8 set when it fails the convergence check (and would go
// through the bisection fallback).
template <int MODEL>
__global__ __launch_bounds__(kMaxBlock) void k_halley_trace(TraceArgs args) {
  const KQuotes& q = args.q;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= q.n) return;
  const double P = ld(q.price, i), fs = ld(q.fs, i), K = ld(q.K, i), T = ld(q.T, i),
               r = ld(q.r, i);
  const double qy = MODEL == fv::kBlackScholesMerton ? ld(q.q, i) : 0.0;
  fv::HalleyState hs;
  fv::ScaledQuote sq;
  const uint8_t st = halley_quote<MODEL>(P, fs, K, T, r, qy, ldflag(q, i), q.hsteps, &hs, &sq);
  uint32_t code = 0xFFFFFFFFu;  // not solved (status != OK)
  if (st == fv::kQOk) code = (uint32_t)hs.steps | (hs.converged ? 0u : 0x100u);
  args.out[i] = code;
}

// ------------------------------------------------------------- IV: Halley
// LDS queue entry of a lane that failed the convergence check, with its
// bracket, or (lo = kGeneralQuote) that the scaled solve does not take.
struct Pending {
  int64_t i;
  double lo, hi;
};
constexpr double kGeneralQuote = -1.0;

// A queued quote: the general Halley solve where the scaled one did not take
// it, then bisection where the steps did not converge.  Both stand here, after
// the queue, and not beside the scaled solve, whose registers they would take:
// the constants of one binary64 evaluation fill the scalar file by themselves.
template <int MODEL>
__device__ __forceinline__ uint8_t queued_quote(double P, double fs, double K, double T, double r,
                                                double qy, int th, int steps, double lo,
                                                double hi, double* sg, Reduced* rd) {
  *rd = fv::reduce_quote(MODEL, P, fs, K, T, r, qy, th);
  uint8_t st = fv::kQOk;
  bool bisect = true;
  double s = 0.0;
  if (lo == kGeneralQuote) {
    st = rd->status;
    bisect = false;
    if (st == fv::kQOk) {
      const fv::HalleyState hs = fv::halley_solve(rd->x, rd->beta, rd->bmax, rd->lnb, steps);
      s = hs.s;
      bisect = !hs.converged;
      lo = hs.lo;
      hi = hs.hi;
    }
  }
  if (bisect) s = fv::bisection_solve(rd->x, rd->beta, rd->bmax, rd->lnb, lo, hi, kBisectTol);
  *sg = st == fv::kQOk ? s * rd->isqrtT
                       : st == fv::kQAtIntrinsic ? 0.0 : __builtin_nan("");
  return st;
}

// The scaled solve of a quote, or a queue entry for it: returns the status,
// sets `queued`.
template <int MODEL>
__device__ __forceinline__ uint8_t scaled_halley(double P, double fs, double K, double T, double r,
                                                 double qy, int th, int steps,
                                                 fv::HalleyState* hs, fv::ScaledQuote* sq,
                                                 double* sg, bool* queued) {
  *sq = fv::scaled_quote(MODEL, P, fs, K, T, r, qy, th);
  const uint8_t st = sq->status;
  *sg = st == fv::kQAtIntrinsic ? 0.0 : __builtin_nan("");
  *queued = sq->general;
  hs->lo = kGeneralQuote;
  if (st == fv::kQOk && !sq->general) {
    *hs = fv::halley_solve_scaled(sq->x, sq->bh, sq->ch, steps);
    *sg = hs->s * sq->isqrtT;
    *queued = !hs->converged;
  }
  return st;
}

__device__ __forceinline__ uint64_t lanemask_lt() {
  const unsigned lane = __lane_id();
  return lane ? (~0ull >> (64 - lane)) : 0ull;
}

// Bound by the vector ALU like k_iv_lbr, on the same guess; its first two
// steps are in binary32 and nearly every quote takes one binary64 step after
// them (two full steps after one at guess precision before, with both in
// binary64).  3M wide-wing BSM quotes: 51.2 us (131 before; 54.5 with the
// general solve beside the scaled one).  One quote per thread, as k_iv_lbr;
// the queue holds one entry per thread.
template <int MODEL, bool GREEKS, bool ARR>
__global__ __launch_bounds__(kMaxBlock)
__attribute__((amdgpu_waves_per_eu(FV_WAVES_HALLEY(GREEKS)))) void k_iv_halley(IvArgs args) {
  const KQuotes& q = args.q;
  extern __shared__ unsigned char smem_raw[];
  Pending* queue = reinterpret_cast<Pending*>(smem_raw);
  __shared__ int qcount;
  if (threadIdx.x == 0) qcount = 0;
  __syncthreads();

  const int64_t b = (int64_t)blockIdx.x * blockDim.x;
  const unsigned t = threadIdx.x;
  bool fail = false;
  fv::HalleyState hs;
  hs.s = 0.0;  // (what the Greeks of a quote without a volatility start from)
  hs.lo = 0.0;
  hs.hi = 0.0;
  if ((int64_t)t < q.n - b) {
    const double P = ld<ARR>(q.price, b, t), fs = ld<ARR>(q.fs, b, t), K = ld<ARR>(q.K, b, t),
                 T = ld<ARR>(q.T, b, t), r = ld<ARR>(q.r, b, t);
    const double qy = MODEL == fv::kBlackScholesMerton ? ld<ARR>(q.q, b, t) : 0.0;
    const int th = ldflag<ARR>(q, b, t);
    fv::ScaledQuote sq;
    double sg;
    const uint8_t st =
        scaled_halley<MODEL>(P, fs, K, T, r, qy, th, q.hsteps, &hs, &sq, &sg, &fail);
    if (!fail) {
      const auto* out = late_args<IvArgs>();
      (global_ptr(out->sig_out) + b)[t] = sg;
      if (uint8_t* st_out = out->st_out) (global_ptr(st_out) + b)[t] = st;
      if (GREEKS) {
        const Greeks gr =
            greeks_solved<MODEL>(st, false, sq, hs.s, sg, P, fs, K, T, r, qy, th);
        store_greeks(out->g, b, t, gr);
      }
    }
  }
  // wave-level compaction of the failing lanes into the LDS queue
  const uint64_t mask = __ballot(fail);
  if (mask) {
    int wbase = 0;
    const int cnt = __popcll(mask);
    const unsigned first = __ffsll((unsigned long long)mask) - 1;
    if (__lane_id() == first) wbase = atomicAdd(&qcount, cnt);
    wbase = __shfl(wbase, first);
    if (fail) {
      const int slot = wbase + __popcll(mask & lanemask_lt());
      queue[slot].i = b + t;
      queue[slot].lo = hs.lo;
      queue[slot].hi = hs.hi;
    }
  }
  __syncthreads();
  // The packed queue: every lane of a wave works, and no thread has more than
  // one entry (a loop would hoist its constants into 40 registers more).  An
  // empty queue, the rule, ends here.
  const int m = __builtin_amdgcn_readfirstlane(qcount);
  if (m == 0) return;
  if ((int)t < m) {
    const int64_t iq = queue[t].i;
    const auto* late = late_args<IvArgs>();
    const KQuotes& q = late->q;
    const GreekOut& g = late->g;
    const double P = ld<ARR>(q.price, iq), fs = ld<ARR>(q.fs, iq), K = ld<ARR>(q.K, iq), T = ld<ARR>(q.T, iq),
                 r = ld<ARR>(q.r, iq);
    const double qy = MODEL == fv::kBlackScholesMerton ? ld<ARR>(q.q, iq) : 0.0;
    const int th = ldflag<ARR>(q, iq);
    Reduced rd;
    double sg;
    const uint8_t st = queued_quote<MODEL>(P, fs, K, T, r, qy, th, q.hsteps, queue[t].lo,
                                           queue[t].hi, &sg, &rd);
    late->sig_out[iq] = sg;
    if (uint8_t* st_out = late->st_out) st_out[iq] = st;
    if (GREEKS)
      store_greeks(g, iq, 0,
                   st == fv::kQOk
                       ? fv::greeks_at(MODEL, fs, K, T, r, qy, sg, th, rd.F, rd.D, P)
                       : no_greeks());
  }
}

// ------------------------------------------------------------- IV: Halley, binary32
struct KQuotes32 {
  int64_t n;
  fv_arg_f32 price, fs, K, T, r, q;
  const int8_t* flag;
  int8_t flag_value;
  int hsteps;
};

// Arguments of k_iv_halley32.
struct Iv32Args {
  KQuotes32 q;
  float* sig_out;
  uint8_t* st_out;
};

__device__ __forceinline__ float ld32(const fv_arg_f32& a, int64_t i) {
  return a.ptr ? a.ptr[i] : a.value;
}
// quote b + t, split as for ld
template <bool ARR>
__device__ __forceinline__ float ld32(const fv_arg_f32& a, int64_t b, unsigned t) {
  return ARR || a.ptr ? (a.ptr + b)[t] : a.value;
}

struct Pending32 {
  int64_t i;
  float lo, hi;
};

// The binary32 twin of k_iv_halley: the same ballot + LDS compaction of the
// lanes that fail the convergence check and bisection over the packed queue,
// in float arithmetic throughout.  Bound by the vector ALU: about 470 vector
// instructions per quote (1,150 with the at-the-money start, whose lanes took
// up to 8 steps and a wave its slowest lane's).  10M wide-wing BSM quotes:
// 100 us (288 with that start).
template <int MODEL, bool ARR>
__global__ __launch_bounds__(kMaxBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_iv_halley32(
    Iv32Args args) {
  extern __shared__ unsigned char smem_raw[];
  Pending32* queue = reinterpret_cast<Pending32*>(smem_raw);
  __shared__ int qcount;
  if (threadIdx.x == 0) qcount = 0;
  __syncthreads();
  const int64_t b = (int64_t)blockIdx.x * blockDim.x;
  const unsigned t = threadIdx.x;
  bool fail = false;
  fv32::HalleyState hs;
  hs.lo = 0.0f;
  hs.hi = 0.0f;
  if ((int64_t)t < args.q.n - b) {
    const KQuotes32& q = args.q;
    const float P = ld32<ARR>(q.price, b, t), fs = ld32<ARR>(q.fs, b, t),
                K = ld32<ARR>(q.K, b, t), T = ld32<ARR>(q.T, b, t), r = ld32<ARR>(q.r, b, t);
    const float qy = MODEL == fv::kBlackScholesMerton ? ld32<ARR>(q.q, b, t) : 0.0f;
    const int th = ARR || q.flag ? (int)(q.flag + b)[t] : (int)q.flag_value;
    const fv32::ScaledQuote sq = fv32::scaled_quote(MODEL, P, fs, K, T, r, qy, th);
    uint8_t st = sq.status;
    float sg = st == fv::kQAtIntrinsic ? 0.0f : __builtin_nanf("");
    bool general = sq.general;
    if (st == fv::kQOk && !general) {
      general = !fv32::halley_solve_scaled(sq, q.hsteps, &hs);
      sg = hs.s * sq.isqrtT;
      fail = !hs.converged;
    }
    if (__builtin_expect(general, 0)) {
      const fv32::Reduced rd = fv32::reduce_quote(MODEL, opaque(P), opaque(fs), opaque(K),
                                                  opaque(T), opaque(r), opaque(qy), th);
      st = rd.status;
      sg = st == fv::kQAtIntrinsic ? 0.0f : __builtin_nanf("");
      fail = false;
      if (st == fv::kQOk) {
        hs = fv32::halley_solve(rd.x, rd.beta, rd.bmax, rd.lnb, q.hsteps);
        sg = hs.s / rd.sqrtT;
        fail = !hs.converged;
      }
    }
    if (!fail) {
      const Iv32Args* out = late_args<Iv32Args>();
      (global_ptr(out->sig_out) + b)[t] = sg;
      if (uint8_t* st_out = out->st_out) (global_ptr(st_out) + b)[t] = st;
    }
  }
  const uint64_t mask = __ballot(fail);
  if (mask) {
    int wbase = 0;
    const int cnt = __popcll(mask);
    const unsigned first = __ffsll((unsigned long long)mask) - 1;
    if (__lane_id() == first) wbase = atomicAdd(&qcount, cnt);
    wbase = __shfl(wbase, first);
    if (fail) {
      const int slot = wbase + __popcll(mask & lanemask_lt());
      queue[slot].i = b + t;
      queue[slot].lo = hs.lo;
      queue[slot].hi = hs.hi;
    }
  }
  __syncthreads();
  const int m = __builtin_amdgcn_readfirstlane(qcount);
  if (m == 0) return;
  for (int j = threadIdx.x; j < m; j += blockDim.x) {
    const Iv32Args* late = late_args<Iv32Args>();
    const KQuotes32& q = late->q;
    const int64_t i = queue[j].i;
    const float P = ld32(q.price, i), fs = ld32(q.fs, i), K = ld32(q.K, i), T = ld32(q.T, i),
                r = ld32(q.r, i);
    const float qy = MODEL == fv::kBlackScholesMerton ? ld32(q.q, i) : 0.0f;
    const int th = q.flag ? (int)q.flag[i] : (int)q.flag_value;
    const fv32::Reduced rd = fv32::reduce_quote(MODEL, P, fs, K, T, r, qy, th);
    const float s = fv32::bisection_solve(rd.x, rd.beta, rd.bmax, queue[j].lo, queue[j].hi, 2e-7f);
    late->sig_out[i] = s / rd.sqrtT;
    if (uint8_t* st_out = late->st_out) st_out[i] = fv::kQOk;
  }
}

// ------------------------------------------------------------- Greeks
template <int MODEL>
__global__ __launch_bounds__(kMaxBlock) void k_greeks(FormArgs args) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x;
  const unsigned t = threadIdx.x;
  if ((int64_t)t >= args.q.n - b) return;
  const SigmaQuote v = load_quote<MODEL>(args, b, t);
  fv::ClosedForm c;
  const bool fast = fv::closed_form(MODEL, v.fs, v.K, v.T, v.r, v.q, v.sigma, v.th, &c);
  Greeks gr = fv::greeks_of(c, MODEL, v.fs, v.T, v.r, v.q, v.sigma, v.th, c.D * c.t.P);
  if (__builtin_expect(!fast, 0)) {
    const SigmaQuote w = load_late<MODEL>(b + t);
    gr = no_greeks();
    if (price_domain(w) && w.sigma > 0.0) {
      const double F = fv::forward_of(MODEL, w.fs, w.T, w.r, w.q);
      const double D = fv::fexp_prod(-w.r, w.T);
      const double P = fv::price_at(F, w.K, D, w.sigma, fv::sqrt_pos(w.T), w.th);
      gr = fv::greeks_at(MODEL, w.fs, w.K, w.T, w.r, w.q, w.sigma, w.th, F, D, P);
    }
  }
  const FormArgs* late = late_args<FormArgs>();
  store_rows<5>(late->out, b, t, {gr.delta, gr.gamma, gr.vega, gr.theta, gr.rho});
}

// ------------------------------------------------------------- backward
template <int MODEL>
__global__ __launch_bounds__(kMaxBlock) void k_iv_backward(FormArgs args) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x;
  const unsigned t = threadIdx.x;
  if ((int64_t)t >= args.q.n - b) return;
  const SigmaQuote v = load_quote<MODEL>(args, b, t);
  const double gs = (args.up + b)[t];
  // the price enters Black-76's theta alone
  const double P = MODEL == fv::kBlack76 ? ld<false>(args.q.price, b, t) : 0.0;
  fv::ClosedForm c;
  const bool fast = fv::closed_form(MODEL, v.fs, v.K, v.T, v.r, v.q, v.sigma, v.th, &c);
  const fv::PricePartials pp =
      fv::partials_of(c, MODEL, v.fs, v.K, v.T, v.r, v.q, v.sigma, v.th, P);
  IvGrad d = fv::implicit_gradient(pp);
  bool ok = true;
  if (__builtin_expect(!fast, 0)) {
    const SigmaQuote w = load_late<MODEL>(b + t);
    ok = fv::finite_d(w.sigma) && w.sigma > 0.0 && fv::finite_d(w.fs) && fv::finite_d(w.K) &&
         fv::finite_d(w.T) && w.fs > 0.0 && w.K > 0.0 && w.T > 0.0;
    if (ok)
      d = fv::iv_gradient(MODEL, w.fs, w.K, w.T, w.r, w.q, w.sigma, w.th,
                          ld(late_args<FormArgs>()->q.price, b + t));
  }
  const double g = ok && fv::finite_d(d.dP) ? gs : 0.0;
  const FormArgs* late = late_args<FormArgs>();
  const bool z = !(ok && fv::finite_d(d.dP));
  store_rows<6>(late->out, b, t,
                {z ? 0.0 : g * d.dP, z ? 0.0 : g * d.dfs, z ? 0.0 : g * d.dK, z ? 0.0 : g * d.dT,
                 z ? 0.0 : g * d.dr, z ? 0.0 : g * d.dq});
}

// ------------------------------------------------------------- price adjoint
template <int MODEL>
__global__ __launch_bounds__(kMaxBlock) void k_price_backward(FormArgs args) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x;
  const unsigned t = threadIdx.x;
  if ((int64_t)t >= args.q.n - b) return;
  const SigmaQuote v = load_quote<MODEL>(args, b, t);
  const double g = (args.up + b)[t];
  fv::ClosedForm c;
  const bool fast = fv::closed_form(MODEL, v.fs, v.K, v.T, v.r, v.q, v.sigma, v.th, &c);
  fv::PricePartials pp =
      fv::partials_of(c, MODEL, v.fs, v.K, v.T, v.r, v.q, v.sigma, v.th, c.D * c.t.P);
  bool ok = true;
  if (__builtin_expect(!fast, 0)) {
    const SigmaQuote w = load_late<MODEL>(b + t);
    ok = price_domain(w) && w.sigma > 0.0;
    if (ok) {
      const double F = fv::forward_of(MODEL, w.fs, w.T, w.r, w.q);
      const double D = fv::fexp_prod(-w.r, w.T);
      const double P = fv::price_at(F, w.K, D, w.sigma, fv::sqrt_pos(w.T), w.th);
      pp = fv::price_partials(MODEL, w.fs, w.K, w.T, w.r, w.q, w.sigma, w.th, F, D, P);
    }
  }
  const FormArgs* late = late_args<FormArgs>();
  store_rows<6>(late->out, b, t,
                {ok ? g * pp.dfs : 0.0, ok ? g * pp.dK : 0.0, ok ? g * pp.dT : 0.0,
                 ok ? g * pp.dr : 0.0, ok ? g * pp.dq : 0.0, ok ? g * pp.dsigma : 0.0});
}

// ------------------------------------------------------------- chains
struct ChainArgs {
  int64_t n_chains, n_mat, n;
  int64_t first;  // the launch's first quote
  const int64_t* chain_mat_off;
  const int64_t* mat_quote_off;
  const double *F, *r, *T, *price, *K;
  const int8_t* flag;
  int hsteps;
  double* sigma;
  uint8_t* status;
};

// A lane that fails the Halley convergence check.
struct ChainPending {
  int64_t i;
  int32_t m, cc;  // maturity and chain of quote i
  double lo, hi;
};

// Ragged-chain kernel: one launch over the CSR offsets, one wave per SLICES
// consecutive 64-quote slices (one coalesced 512-byte load per field and
// slice).  The wave finds the maturity and chain of its first quote by two
// 64-ary searches and every lane those of its quotes from the next maturity
// and chain starts, for both slices before it solves either: only the second
// slice's maturity and chain stay live across the first solve.
// The Halley path compacts the lanes that fail its convergence check into an
// LDS queue (wave ballots, as the flat Halley kernel does; an entry per quote)
// and the workgroup bisects the packed queue afterwards.
template <int SOLVER, int SLICES>
__global__ __launch_bounds__(kMaxBlock)
__attribute__((amdgpu_waves_per_eu(FV_CHAINS_WAVES_PER_EU))) void k_iv_chains(ChainArgs c) {
  constexpr bool kHalley = SOLVER == FV_SOLVER_HALLEY;
  extern __shared__ unsigned char smem_raw[];
  ChainPending* queue = reinterpret_cast<ChainPending*>(smem_raw);
  __shared__ int qcount;
  if (kHalley) {
    if (threadIdx.x == 0) qcount = 0;
    __syncthreads();
  }
  // (the wave's number as a scalar: the location runs on the scalar unit)
  const int64_t w0 = c.first +
                     ((int64_t)blockIdx.x * (blockDim.x >> 6) +
                      __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6)) * (64 * SLICES);
  const int lane = (int)__lane_id();
  int64_t m0[SLICES] = {}, c0[SLICES] = {};
  int ml[SLICES] = {}, cl[SLICES] = {};
  const bool any = w0 < c.n;  // wave-uniform
  if (any) {
    fv::ChainCursor cur;
    cur.init(c.mat_quote_off, c.n_mat, c.chain_mat_off, c.n_chains, w0);
#pragma unroll
    for (int sl = 0; sl < SLICES; ++sl) {
      const int64_t i0 = w0 + 64 * sl;
      if (i0 < c.n) cur.slice(i0, min(i0 + 63, c.n - 1), m0[sl], ml[sl], c0[sl], cl[sl]);
    }
  }
#pragma unroll
  for (int sl = 0; sl < SLICES; ++sl) {
    const int64_t i0 = w0 + 64 * sl;
    bool fail = false;
    fv::HalleyState hs;
    hs.lo = 0.0;
    hs.hi = 0.0;
    if (any && lane < c.n - i0) {
      const double F = (c.F + c0[sl])[(unsigned)cl[sl]], r = (c.r + c0[sl])[(unsigned)cl[sl]];
      const double T = (c.T + m0[sl])[(unsigned)ml[sl]];
      const double P = (c.price + i0)[(unsigned)lane], K = (c.K + i0)[(unsigned)lane];
      const int th = (c.flag + i0)[(unsigned)lane];
      uint8_t st;
      double sg;
      if (!kHalley) {
        fv::ScaledQuote sq = fv::scaled_quote(fv::kBlack76, P, F, K, T, r, 0.0, th);
        st = sq.status;
        sg = st == fv::kQAtIntrinsic ? 0.0 : __builtin_nan("");
        bool general = sq.general;
        if (st == fv::kQOk && !general) {
          double s;
          general = !fv::lbr_solve_scaled(sq.x, sq.bh, sq.ch, &s);
          sg = s * sq.isqrtT;
        }
        if (__builtin_expect(general, 0)) {
          const ChainArgs* a = late_args<ChainArgs>();
          const int64_t io = opaque(i0 + lane), co = opaque(c0[sl] + cl[sl]),
                        mo = opaque(m0[sl] + ml[sl]);
          fv::lbr_general(fv::kBlack76, a->price[io], a->F[co], a->K[io], a->T[mo], a->r[co], 0.0,
                          a->flag[io], &sg, &st, &sq);
        }
      } else {
        fv::ScaledQuote sq;
        st = scaled_halley<fv::kBlack76>(P, F, K, T, r, 0.0, th, c.hsteps, &hs, &sq, &sg, &fail);
      }
      if (!fail) {
        const ChainArgs* a = late_args<ChainArgs>();
        (global_ptr(a->sigma) + i0)[(unsigned)lane] = sg;
        if (a->status) (global_ptr(a->status) + i0)[(unsigned)lane] = st;
      }
    }
    if (kHalley) {
      // wave-level compaction of the failing lanes into the LDS queue
      const uint64_t mask = __ballot(fail);
      if (mask) {
        int wbase = 0;
        const int cnt = __popcll(mask);
        const unsigned first = __ffsll((unsigned long long)mask) - 1;
        if (lane == (int)first) wbase = atomicAdd(&qcount, cnt);
        wbase = __shfl(wbase, first);
        if (fail) {
          const int slot = wbase + __popcll(mask & lanemask_lt());
          queue[slot].i = i0 + lane;
          queue[slot].m = (int32_t)(m0[sl] + ml[sl]);
          queue[slot].cc = (int32_t)(c0[sl] + cl[sl]);
          queue[slot].lo = hs.lo;
          queue[slot].hi = hs.hi;
        }
      }
    }
  }
  if (!kHalley) return;
  __syncthreads();
  // the packed queue: every lane of a wave works, up to SLICES entries each
  const int nq = __builtin_amdgcn_readfirstlane(qcount);
  if (nq == 0) return;
  const ChainArgs* a = late_args<ChainArgs>();
#pragma unroll
  for (int sl = 0; sl < SLICES; ++sl) {
    const int j = threadIdx.x + sl * blockDim.x;
    if (j >= nq) return;
    const int64_t iq = queue[j].i;
    const int64_t mq = queue[j].m, cq = queue[j].cc;
    Reduced rd;
    double sg;
    const uint8_t st =
        queued_quote<fv::kBlack76>(a->price[iq], a->F[cq], a->K[iq], a->T[mq], a->r[cq], 0.0,
                                   a->flag[iq], a->hsteps, queue[j].lo, queue[j].hi, &sg, &rd);
    a->sigma[iq] = sg;
    if (a->status) a->status[iq] = st;
  }
}

// ------------------------------------------------------------- normalised b
__global__ void k_normalised_black(int64_t n, const double* __restrict__ x,
                                   const double* __restrict__ s, const int8_t* __restrict__ fl,
                                   double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double xi = x[i], si = s[i];
  const int th = fl ? (int)fl[i] : 1;
  // out-of-the-money side by parity: b(x, s, th) = b(-|x|, s) + intrinsic
  const double xo = -fabs(xi);
  const double bmax = exp(0.5 * xo);
  const fv::NBlack nb = fv::normalised_black_t<0, true>(xo, si, bmax);
  double b = nb.b;
  // in the money: add the intrinsic th (e^{x/2} - e^{-x/2}) = th 2 sinh(x/2),
  // from expm1 so that small |x| keeps its relative precision
  if (th * xi > 0.0) b += th * (expm1(0.5 * xi) - expm1(-0.5 * xi));
  out[i] = b;
}

// binary32 copies of the autotuner's quotes (price, S, K, T, r, q, in that
// order, n floats each)
__global__ void k_tune_to_f32(int64_t n, const double* __restrict__ P, const double* __restrict__ S,
                              const double* __restrict__ K, const double* __restrict__ T,
                              const double* __restrict__ r, const double* __restrict__ q,
                              float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  out[i] = (float)P[i];
  out[n + i] = (float)S[i];
  out[2 * n + i] = (float)K[i];
  out[3 * n + i] = (float)T[i];
  out[4 * n + i] = (float)r[i];
  out[5 * n + i] = (float)q[i];
}

// ------------------------------------------------------------- autotune inputs
// Synthetic in-range quotes for timing candidate launch shapes: a
// counter-based generator (the splitmix64 output function of Steele, Lea &
// Flood, OOPSLA 2014) drives the same distributions as the wide-wing
// Black-Scholes-Merton workload (z~U[-6,6], sigma~logU[0.01,3],
// T~logU[1/365,5], r~U[-0.01,0.08], q~U[0,0.05], S = 100).
__device__ __forceinline__ uint64_t splitmix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__device__ __forceinline__ double unif(uint64_t key) {
  return (double)(splitmix64(key) >> 11) * 0x1.0p-53;
}

__global__ void k_tune_quotes(int64_t n, double* S, double* K, double* T, double* r,
                              double* q, double* sig, int8_t* flag) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint64_t b = (uint64_t)i * 8;
  const double z = -6.0 + 12.0 * unif(b);
  const double sg = exp(log(0.01) + unif(b + 1) * log(300.0));
  const double Ti = exp(log(1.0 / 365.0) + unif(b + 2) * log(5.0 * 365.0));
  const double ri = -0.01 + 0.09 * unif(b + 3);
  const double qi = 0.05 * unif(b + 4);
  const double F = 100.0 * exp((ri - qi) * Ti);
  S[i] = 100.0;
  K[i] = F * exp(-z * sg * sqrt(Ti));
  T[i] = Ti;
  r[i] = ri;
  q[i] = qi;
  sig[i] = sg;
  flag[i] = unif(b + 5) < 0.5 ? 1 : -1;
}

// Ragged structure for timing the chain kernel: every maturity holds
// `per_mat` quotes and every chain `mats` maturities; per-chain F = 100 and
// r, per-maturity T taken from the flat synthetic quotes.
__global__ void k_tune_chains(int64_t n_chains, int64_t n_mat, int64_t n, int mats,
                              int per_mat, const double* Tq, const double* rq, int64_t* cmo,
                              int64_t* mqo, double* F, double* r, double* T) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i <= n_chains) cmo[i] = i * mats;
  if (i <= n_mat) mqo[i] = i * per_mat;
  if (i < n_chains) {
    F[i] = 100.0;
    r[i] = rq[i * mats * per_mat];
  }
  if (i < n_mat) T[i] = Tq[i * per_mat];
  (void)n;
}

// Per-quote T and r of the ragged structure (to price its quotes).
__global__ void k_tune_expand(int64_t n, int mats, int per_mat, const double* cT,
                              const double* cr, double* Te, double* re) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  Te[i] = cT[i / per_mat];
  re[i] = cr[i / ((int64_t)per_mat * mats)];
}

// ------------------------------------------------------------- host side
int fail(int code, const std::string& msg) { return fvh::fail(code, msg); }

// A configured shape.  The workgroup size is what launches take;
// quotes_per_thread is checked, kept and given back by fv_get_launch and the
// tuning files, whose format and refusals stay as they were, and no launch
// reads it (one quote per thread was the fastest in every kernel).
struct LaunchShape {
  int block, qpt;
};
// Workgroup sizes from timing sweeps on MI355X (the wide-wing 10M-quote batch
// for the solvers); fv_autotune re-derives them for other shapes of work.
LaunchShape g_shape[FV_KERNEL_COUNT] = {
    {256, 2},  // price
    {64, 1},   // IV LBR
    {128, 4},  // IV Halley
    {256, 1},  // Greeks
    {128, 4},  // backward
    {128, 8},  // chains
    {128, 4},  // IV Halley, binary32
};

bool valid_shape(int block, int qpt) {
  return block >= 64 && block <= kMaxBlock && block % 64 == 0 && qpt >= 1 && qpt <= 16;
}

// What a shape is refused by: the Halley paths' LDS queue of the lanes that
// need more, at block x qpt entries (the launches take one per thread and
// slice).  Shapes above kMaxQueueBytes are refused.
constexpr size_t kMaxQueueBytes = 65536;

size_t queue_bytes(int kernel, int block, int qpt) {
  if (kernel == FV_KERNEL_IV_HALLEY) return sizeof(Pending) * (size_t)block * qpt;
  if (kernel == FV_KERNEL_IV_HALLEY_F32) return sizeof(Pending32) * (size_t)block * qpt;
  if (kernel == FV_KERNEL_CHAINS) return 2 * sizeof(ChainPending) * (size_t)block;  // Halley path
  return 0;
}

// Largest batch of a call.
constexpr int64_t kMaxQuotes = (int64_t)0x7fffffff * 64;

int check_quotes(int model, const fv_quotes* q) {
  if (model < FV_MODEL_BLACK76 || model > FV_MODEL_BSM)
    return fail(FV_E_INVALID_ARG, "model out of range");
  if (!q) return fail(FV_E_INVALID_ARG, "quotes pointer is NULL");
  if (q->n < 0) return fail(FV_E_INVALID_ARG, "n < 0");
  if (q->n > kMaxQuotes) return fail(FV_E_INVALID_ARG, "n above 2^31 - 1 workgroups of 64");
  if (!q->flag && q->flag_value != 1 && q->flag_value != -1)
    return fail(FV_E_INVALID_ARG, "broadcast flag_value must be +1 or -1");
  return FV_OK;
}

// Maximum Halley steps before a quote goes to the bisection fallback
// (fv_set_halley_steps); read by every launch of a Halley kernel.
std::atomic<int> g_halley_steps{kHalleySteps};

KQuotes to_k(const fv_quotes* q) {
  KQuotes k;
  k.n = q->n;
  k.price = q->price;
  k.fs = q->fs;
  k.K = q->K;
  k.T = q->T;
  k.r = q->r;
  k.q = q->q;
  k.flag = q->flag;
  k.flag_value = q->flag_value;
  k.hsteps = g_halley_steps.load(std::memory_order_relaxed);
  return k;
}

int launched(const char* what) { return fvh::launched(what); }

// A launch holds fewer than 2^32 work items: of a larger grid the count is
// taken modulo 2^32, with no error, and the quotes past it stay unwritten.
// With a quote per thread a batch may be larger, so it is launched in parts
// of at most kPart quotes, one as a rule.
constexpr int64_t kPart = (int64_t)1 << 31;

template <class A>
void advance(A& field, int64_t by) {  // fv_arg, fv_arg_f32
  if (field.ptr) field.ptr += by;
}
template <class V>
void advance(V*& p, int64_t by) {
  if (p) p += by;
}
template <class Q>
void advance_quotes(Q& q, int64_t by) {
  advance(q.price, by);
  advance(q.fs, by);
  advance(q.K, by);
  advance(q.T, by);
  advance(q.r, by);
  advance(q.q, by);
  advance(q.flag, by);
}
void advance(FormArgs& a, int64_t by) {
  advance_quotes(a.q, by);
  advance(a.sigma, by);
  advance(a.up, by);
  for (double*& p : a.out) advance(p, by);
}
void advance(IvArgs& a, int64_t by) {
  advance_quotes(a.q, by);
  advance(a.sig_out, by);
  advance(a.st_out, by);
  for (double*& p : a.g.p) advance(p, by);
}
void advance(Iv32Args& a, int64_t by) {
  advance_quotes(a.q, by);
  advance(a.sig_out, by);
  advance(a.st_out, by);
}
void advance(TraceArgs& a, int64_t by) {
  advance_quotes(a.q, by);
  advance(a.out, by);
}

// launch(args, grid) for every part of a flat batch in workgroups of `block`
// quotes.
template <class ARGS, class LAUNCH>
void in_parts(ARGS args, int block, LAUNCH launch) {
  for (int64_t left = args.q.n; left > 0; left -= kPart) {
    args.q.n = std::min(left, kPart);
    launch(args, dim3((unsigned)((args.q.n + block - 1) / block)));
    if (left > kPart) advance(args, kPart);
  }
}

int device_cus();

// Slices per wave of the ragged kernel.  One below 40 waves per SIMD (160 per
// compute unit), where the chain of a wave's location and second solve is
// what a batch waits for; above, two pay the location once.  In us, one
// against two: LBR 10.2 / 11.0 (0.5M quotes), 19.2 / 21.1 (1.0M),
// 31.5 / 32.3 (1.9M), 63.9 / 62.4 (4.2M), 133 / 128 (8.4M); Halley
// 20.7 / 21.9, 33.5 / 34.6, 68.1 / 66.5, 144 / 135 from 1.0M on.
int chain_slices(int64_t n) { return n < (int64_t)64 * 160 * device_cus() ? 1 : 2; }

int device_cus() {
  static int cache[64];  // per device ordinal; 0 = not yet queried
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (dev >= 0 && dev < 64 && cache[dev] > 0) return cache[dev];
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus <= 0)
    return 256;
  if (dev >= 0 && dev < 64) cache[dev] = cus;
  return cus;
}

// ---------------------------------------------------------- tuning table
// fv_autotune's results per (kernel family, model, size class of the batch);
// a launch takes the workgroup size of its class when there is one.
constexpr int kModels = 3;
constexpr int kBuckets = 7;
struct Tuned {
  int block, qpt;  // block == 0: not tuned
  float ms;        // the winning candidate's time when it was measured
};
Tuned g_tuned[FV_KERNEL_COUNT][kModels][kBuckets];
// while fv_autotune times a workgroup size, launches of that family take it
int g_tuning_kernel = -1;
int g_tuning_block = 0;

// Size class of a batch of n >= 1 quotes: 0 below 2^14, then one class per
// factor of 4 ([2^14, 2^16) is 1, ...), 6 from 2^24 up.
int bucket_of(int64_t n) {
  int lg = 0;
  while (lg < 62 && ((int64_t)1 << (lg + 1)) <= n) ++lg;
  if (lg < 14) return 0;
  return std::min(kBuckets - 1, (lg - 14) / 2 + 1);
}

// The workgroup size a launch of n quotes of `kernel` under `model` takes: a
// tuned entry of its size class if there is one, else the configured size, or
// one wave for a batch that would not give every CU a workgroup of that.
// Results never depend on it.
int block_for(int kernel, int model, int64_t n) {
  if (kernel == g_tuning_kernel) return g_tuning_block;
  const Tuned& t = g_tuned[kernel][model][bucket_of(n > 0 ? n : 1)];
  if (t.block) return t.block;
  const int block = g_shape[kernel].block;
  return (n + block - 1) / block < device_cus() ? 64 : block;
}

// Architecture name of the current device (hipDeviceProp_t::gcnArchName,
// e.g. "gfx950:sramecc+:xnack-"), the key a tuning file is valid for.
int device_arch(std::string* out) {
  int dev = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess)
    return fail(FV_E_HIP, "no HIP device to read the architecture of");
  *out = prop.gcnArchName;
  return FV_OK;
}

// Value of the integer field "key" inside [b, e) of a tuning file's text.
bool int_field(const std::string& t, size_t b, size_t e, const char* key, long* v) {
  const std::string k = std::string("\"") + key + "\"";
  const size_t at = t.find(k, b);
  if (at == std::string::npos || at >= e) return false;
  size_t i = at + k.size();
  while (i < e && (t[i] == ' ' || t[i] == ':')) ++i;
  char* endp = nullptr;
  const long x = strtol(t.c_str() + i, &endp, 10);
  if (endp == t.c_str() + i) return false;
  *v = x;
  return true;
}

// Reads a tuning file written by fv_tuning_save into `table` (all entries
// validated; nothing is returned on any error) and its "arch" string.
int parse_tuning(const char* path, std::string* text, std::string* arch,
                 Tuned (*table)[kModels][kBuckets]) {
  FILE* f = fopen(path, "r");
  if (!f) return fail(FV_E_INVALID_ARG, std::string("cannot read ") + path);
  char buf[4096];
  size_t got;
  text->clear();
  while ((got = fread(buf, 1, sizeof(buf), f)) > 0 && text->size() < (1u << 20))
    text->append(buf, got);
  fclose(f);
  const std::string& t = *text;
  auto bad = [&](const char* why) {
    return fail(FV_E_INVALID_ARG, std::string("tuning file ") + path + ": " + why);
  };
  if (t.find("\"format\": \"fastvol-tuning\"") == std::string::npos) return bad("not a tuning file");
  long version = 0;
  if (!int_field(t, 0, t.size(), "version", &version) || version != 1)
    return bad("unsupported version");
  const size_t a = t.find("\"arch\": \"");
  if (a == std::string::npos) return bad("no arch");
  const size_t a0 = a + 9, a1 = t.find('"', a0);
  if (a1 == std::string::npos || a1 == a0) return bad("no arch");
  *arch = t.substr(a0, a1 - a0);
  size_t pos = t.find("\"entries\"");
  if (pos == std::string::npos) return bad("no entries");
  memset(table, 0, sizeof(Tuned) * FV_KERNEL_COUNT * kModels * kBuckets);
  while ((pos = t.find('{', pos)) != std::string::npos) {
    const size_t end = t.find('}', pos);
    if (end == std::string::npos) return bad("unterminated entry");
    long k, m, b, blk, qq;
    if (!int_field(t, pos, end, "kernel", &k) || !int_field(t, pos, end, "model", &m) ||
        !int_field(t, pos, end, "bucket", &b) || !int_field(t, pos, end, "block", &blk) ||
        !int_field(t, pos, end, "qpt", &qq))
      return bad("entry without kernel, model, bucket, block or qpt");
    if (k < 0 || k >= FV_KERNEL_COUNT || m < 0 || m >= kModels || b < 0 || b >= kBuckets)
      return bad("entry out of range");
    // range-checked before the narrowing to int
    if (blk < 1 || blk > 1 << 16 || qq < 1 || qq > 1 << 16) return bad("invalid launch shape");
    if (!valid_shape((int)blk, (int)qq) || queue_bytes((int)k, (int)blk, (int)qq) > kMaxQueueBytes)
      return bad("invalid launch shape");
    float ms = 0.0f;
    const size_t mk = t.find("\"ms\"", pos);
    if (mk != std::string::npos && mk < end) {
      size_t i = mk + 4;
      while (i < end && (t[i] == ' ' || t[i] == ':')) ++i;
      ms = (float)strtod(t.c_str() + i, nullptr);
    }
    table[k][m][b] = Tuned{(int)blk, (int)qq, ms};
    pos = end + 1;
  }
  return FV_OK;
}

}  // namespace

// =================================================================== C ABI
extern "C" {

int fv_version(void) { return FV_ABI_VERSION; }

const char* fv_last_error(void) { return fvh::g_last_error.c_str(); }

int fv_set_launch(int kernel, int block, int qpt) {
  if (kernel < 0 || kernel >= FV_KERNEL_COUNT) return fail(FV_E_INVALID_ARG, "kernel id");
  if (!valid_shape(block, qpt)) return fail(FV_E_INVALID_ARG, "launch shape");
  if (queue_bytes(kernel, block, qpt) > kMaxQueueBytes)
    return fail(FV_E_INVALID_ARG, "launch shape: Halley queue above 64 KiB of LDS");
  g_shape[kernel].block = block;
  g_shape[kernel].qpt = qpt;
  // an explicit shape wins over the family's tuned entries
  memset(g_tuned[kernel], 0, sizeof(g_tuned[kernel]));
  return FV_OK;
}

int fv_set_halley_steps(int steps) {
  if (steps < 1 || steps > kMaxHalleySteps)
    return fail(FV_E_INVALID_ARG, "Halley steps outside [1, 64]");
  g_halley_steps.store(steps, std::memory_order_relaxed);
  return FV_OK;
}

int fv_get_halley_steps(void) { return g_halley_steps.load(std::memory_order_relaxed); }

int fv_get_launch(int kernel, int* block, int* qpt) {
  if (kernel < 0 || kernel >= FV_KERNEL_COUNT || !block || !qpt)
    return fail(FV_E_INVALID_ARG, "kernel id or NULL output");
  *block = g_shape[kernel].block;
  *qpt = g_shape[kernel].qpt;
  return FV_OK;
}

// Launches the kernel KERN of `model` on `args`, one quote per thread, in
// workgroups of the family's size.
#define FV_LAUNCH_FORM(KERN, FAMILY)                                                      \
  do {                                                                                    \
    const int block = block_for(FAMILY, model, q->n);                               \
    hipStream_t s = (hipStream_t)stream;                                                  \
    in_parts(args, block, [=](const auto& part, dim3 grid) {                              \
      switch (model) {                                                                    \
        case FV_MODEL_BLACK76: KERN<0><<<grid, block, 0, s>>>(part); break;               \
        case FV_MODEL_BLACK_SCHOLES: KERN<1><<<grid, block, 0, s>>>(part); break;         \
        default: KERN<2><<<grid, block, 0, s>>>(part); break;                             \
      }                                                                                   \
    });                                                                                   \
  } while (0)

int fv_price(int model, const fv_quotes* q, fv_arg sigma, double* price_out, void* stream) {
  int rc = check_quotes(model, q);
  if (rc) return rc;
  if (q->n == 0) return FV_OK;
  if (!price_out) return fail(FV_E_INVALID_ARG, "price_out is NULL");
  const FormArgs args = {to_k(q), sigma, nullptr, {price_out}};
  FV_LAUNCH_FORM(k_price, FV_KERNEL_PRICE);
  return launched("fv_price");
}

int fv_implied_vol(int model, int solver, const fv_quotes* q, double* sigma_out,
                   uint8_t* status_out, double* const* greeks_out, void* stream) {
  int rc = check_quotes(model, q);
  if (rc) return rc;
  if (solver != FV_SOLVER_LBR && solver != FV_SOLVER_HALLEY)
    return fail(FV_E_INVALID_ARG, "solver out of range");
  if (q->n == 0) return FV_OK;
  if (!sigma_out) return fail(FV_E_INVALID_ARG, "sigma_out is NULL");
  GreekOut g;
  g.any = 0;
  for (int j = 0; j < 5; ++j) {
    g.p[j] = greeks_out ? greeks_out[j] : nullptr;
    g.any |= g.p[j] != nullptr;
  }
  const IvArgs args = {to_k(q), sigma_out, status_out, g};
  hipStream_t s = (hipStream_t)stream;
  // every per-quote field an array (q only matters for Black-Scholes-Merton)
  const bool arr = q->price.ptr && q->fs.ptr && q->K.ptr && q->T.ptr && q->r.ptr && q->flag &&
                   (model != FV_MODEL_BSM || q->q.ptr);
  const int family = solver == FV_SOLVER_LBR ? FV_KERNEL_IV_LBR : FV_KERNEL_IV_HALLEY;
  const int block = block_for(family, model, q->n);
  const size_t lds = sizeof(Pending) * (size_t)block;
  in_parts(args, block, [=](const IvArgs& part, dim3 grid) {
#define FV_IV(M, G)                                                            \
  (solver == FV_SOLVER_LBR                                                     \
       ? (arr ? k_iv_lbr<M, G, true><<<grid, block, 0, s>>>(part)              \
              : k_iv_lbr<M, G, false><<<grid, block, 0, s>>>(part))            \
       : (arr ? k_iv_halley<M, G, true><<<grid, block, lds, s>>>(part)         \
              : k_iv_halley<M, G, false><<<grid, block, lds, s>>>(part)))
    switch (model * 2 + (part.g.any ? 1 : 0)) {
      case 0: FV_IV(0, false); break;
      case 1: FV_IV(0, true); break;
      case 2: FV_IV(1, false); break;
      case 3: FV_IV(1, true); break;
      case 4: FV_IV(2, false); break;
      default: FV_IV(2, true); break;
    }
#undef FV_IV
  });
  return launched(solver == FV_SOLVER_LBR ? "fv_implied_vol(LBR)" : "fv_implied_vol(Halley)");
}

int fv_implied_vol_f32(int model, const fv_quotes_f32* q, float* sigma_out,
                       uint8_t* status_out, void* stream) {
  if (model < FV_MODEL_BLACK76 || model > FV_MODEL_BSM)
    return fail(FV_E_INVALID_ARG, "model out of range");
  if (!q) return fail(FV_E_INVALID_ARG, "quotes pointer is NULL");
  if (q->n < 0) return fail(FV_E_INVALID_ARG, "n < 0");
  if (q->n > kMaxQuotes) return fail(FV_E_INVALID_ARG, "n above 2^31 - 1 workgroups of 64");
  if (!q->flag && q->flag_value != 1 && q->flag_value != -1)
    return fail(FV_E_INVALID_ARG, "broadcast flag_value must be +1 or -1");
  if (q->n == 0) return FV_OK;
  if (!sigma_out) return fail(FV_E_INVALID_ARG, "sigma_out is NULL");
  KQuotes32 k;
  k.n = q->n;
  k.price = q->price;
  k.fs = q->fs;
  k.K = q->K;
  k.T = q->T;
  k.r = q->r;
  k.q = q->q;
  k.flag = q->flag;
  k.flag_value = q->flag_value;
  k.hsteps = g_halley_steps.load(std::memory_order_relaxed);
  const int block = block_for(FV_KERNEL_IV_HALLEY_F32, model, q->n);
  const size_t lds = sizeof(Pending32) * (size_t)block;
  const Iv32Args args = {k, sigma_out, status_out};
  hipStream_t s = (hipStream_t)stream;
  const bool arr = q->price.ptr && q->fs.ptr && q->K.ptr && q->T.ptr && q->r.ptr && q->flag &&
                   (model != FV_MODEL_BSM || q->q.ptr);
  in_parts(args, block, [=](const Iv32Args& part, dim3 grid) {
#define FV_HAL32(M)                                           \
  (arr ? k_iv_halley32<M, true><<<grid, block, lds, s>>>(part) \
       : k_iv_halley32<M, false><<<grid, block, lds, s>>>(part))
    switch (model) {
      case FV_MODEL_BLACK76: FV_HAL32(0); break;
      case FV_MODEL_BLACK_SCHOLES: FV_HAL32(1); break;
      default: FV_HAL32(2); break;
    }
#undef FV_HAL32
  });
  return launched("fv_implied_vol_f32");
}

int fv_greeks(int model, const fv_quotes* q, fv_arg sigma, double* delta, double* gamma,
              double* vega, double* theta, double* rho, void* stream) {
  int rc = check_quotes(model, q);
  if (rc) return rc;
  if (q->n == 0) return FV_OK;
  if (!delta && !gamma && !vega && !theta && !rho) return FV_OK;
  const FormArgs args = {to_k(q), sigma, nullptr, {delta, gamma, vega, theta, rho}};
  FV_LAUNCH_FORM(k_greeks, FV_KERNEL_GREEKS);
  return launched("fv_greeks");
}

int fv_implied_vol_backward(int model, const fv_quotes* q, const double* sigma,
                            const double* grad_sigma, double* g_price, double* g_fs,
                            double* g_K, double* g_T, double* g_r, double* g_q, void* stream) {
  int rc = check_quotes(model, q);
  if (rc) return rc;
  if (q->n == 0) return FV_OK;
  if (!sigma || !grad_sigma) return fail(FV_E_INVALID_ARG, "sigma or grad_sigma is NULL");
  const FormArgs args = {to_k(q), fv_arg{sigma, 0.0}, grad_sigma, {g_price, g_fs, g_K, g_T, g_r, g_q}};
  FV_LAUNCH_FORM(k_iv_backward, FV_KERNEL_BACKWARD);
  return launched("fv_implied_vol_backward");
}

int fv_price_backward(int model, const fv_quotes* q, fv_arg sigma, const double* grad_price,
                      double* g_fs, double* g_K, double* g_T, double* g_r, double* g_q,
                      double* g_sigma, void* stream) {
  int rc = check_quotes(model, q);
  if (rc) return rc;
  if (q->n == 0) return FV_OK;
  if (!grad_price) return fail(FV_E_INVALID_ARG, "grad_price is NULL");
  const FormArgs args = {to_k(q), sigma, grad_price, {g_fs, g_K, g_T, g_r, g_q, g_sigma}};
  FV_LAUNCH_FORM(k_price_backward, FV_KERNEL_BACKWARD);
  return launched("fv_price_backward");
}

int fv_lbr_trace(int model, const fv_quotes* q, uint32_t* path_out, void* stream) {
  int rc = check_quotes(model, q);
  if (rc) return rc;
  if (q->n == 0) return FV_OK;
  if (!path_out) return fail(FV_E_INVALID_ARG, "path_out is NULL");
  const TraceArgs args = {to_k(q), path_out};
  FV_LAUNCH_FORM(k_lbr_trace, FV_KERNEL_IV_LBR);
  return launched("fv_lbr_trace");
}

int fv_halley_trace(int model, const fv_quotes* q, uint32_t* steps_out, void* stream) {
  int rc = check_quotes(model, q);
  if (rc) return rc;
  if (q->n == 0) return FV_OK;
  if (!steps_out) return fail(FV_E_INVALID_ARG, "steps_out is NULL");
  const TraceArgs args = {to_k(q), steps_out};
  FV_LAUNCH_FORM(k_halley_trace, FV_KERNEL_IV_LBR);
  return launched("fv_halley_trace");
}

int fv_implied_vol_chains(int solver, const fv_chains* c, double* sigma_out,
                          uint8_t* status_out, void* stream) {
  if (!c) return fail(FV_E_INVALID_ARG, "chains pointer is NULL");
  if (solver != FV_SOLVER_LBR && solver != FV_SOLVER_HALLEY)
    return fail(FV_E_INVALID_ARG, "solver out of range");
  if (c->n_chains < 0 || c->n_maturities < 0 || c->n_quotes < 0)
    return fail(FV_E_INVALID_ARG, "negative size");
  if (c->n_quotes == 0) return FV_OK;
  if (c->n_quotes > kMaxQuotes) return fail(FV_E_INVALID_ARG, "n_quotes above 2^31 - 1 workgroups of 64");
  if (c->n_maturities > 0x7fffffff || c->n_chains > 0x7fffffff)
    return fail(FV_E_INVALID_ARG, "more than 2^31 - 1 maturities or chains");
  if (c->n_chains == 0 || c->n_maturities == 0)
    return fail(FV_E_INVALID_ARG, "quotes without chains or maturities");
  if (!c->chain_mat_off || !c->mat_quote_off || !c->F || !c->r || !c->T || !c->price ||
      !c->K || !c->flag || !sigma_out)
    return fail(FV_E_INVALID_ARG, "NULL chain array");
  ChainArgs k = {c->n_chains, c->n_maturities, c->n_quotes, 0, c->chain_mat_off,
                       c->mat_quote_off, c->F, c->r, c->T, c->price, c->K, c->flag,
                       g_halley_steps.load(std::memory_order_relaxed), sigma_out, status_out};
  const int block = block_for(FV_KERNEL_CHAINS, FV_MODEL_BLACK76, k.n), slices = chain_slices(k.n);
  const int64_t per = (int64_t)slices * block;
  const size_t lds = sizeof(ChainPending) * (size_t)per;
  hipStream_t s = (hipStream_t)stream;
  for (; k.first < k.n; k.first += kPart / per * per) {  // whole waves, in order
    const int64_t part = std::min(k.n - k.first, kPart / per * per);
    const dim3 grid((unsigned)((part + per - 1) / per));
    if (solver == FV_SOLVER_LBR) {
      if (slices == 1) k_iv_chains<FV_SOLVER_LBR, 1><<<grid, block, 0, s>>>(k);
      else k_iv_chains<FV_SOLVER_LBR, 2><<<grid, block, 0, s>>>(k);
    } else {
      if (slices == 1) k_iv_chains<FV_SOLVER_HALLEY, 1><<<grid, block, lds, s>>>(k);
      else k_iv_chains<FV_SOLVER_HALLEY, 2><<<grid, block, lds, s>>>(k);
    }
  }
  return launched("fv_implied_vol_chains");
}

int fv_normalised_black(int64_t n, const double* x, const double* s, const int8_t* flag,
                        double* out, void* stream) {
  if (n < 0) return fail(FV_E_INVALID_ARG, "n < 0");
  if (n == 0) return FV_OK;
  if (!x || !s || !out) return fail(FV_E_INVALID_ARG, "NULL array");
  for (int64_t at = 0; at < n; at += kPart) {
    const int64_t part = std::min(n - at, kPart);
    k_normalised_black<<<(unsigned)((part + 255) / 256), 256, 0, (hipStream_t)stream>>>(
        part, x + at, s + at, flag ? flag + at : nullptr, out + at);
  }
  return launched("fv_normalised_black");
}

int fv_autotune(int kernel, int model, int64_t n_hint, void* stream) {
  if (kernel < 0 || kernel >= FV_KERNEL_COUNT) return fail(FV_E_INVALID_ARG, "kernel id");
  if (model < FV_MODEL_BLACK76 || model > FV_MODEL_BSM)
    return fail(FV_E_INVALID_ARG, "model out of range");
  if (n_hint < 0) return fail(FV_E_INVALID_ARG, "n_hint < 0");
  // time on a batch of the requested size class: n_hint quotes, at most
  // 2^24, rounded down to whole synthetic chains (at least one group of 8)
  const int per_mat = 256, mats = 8;
  int64_t n = std::min<int64_t>(n_hint, 1 << 24);
  n = std::max<int64_t>((n / (per_mat * mats)) * (per_mat * mats), per_mat * mats);
  // the chain kernel only runs Black-76
  const int tuned_model = kernel == FV_KERNEL_CHAINS ? FV_MODEL_BLACK76 : model;
  const int bucket = bucket_of(n_hint > 0 ? n_hint : 1);
  const int64_t n_mat = n / per_mat, n_chains = n_mat / mats;
  hipStream_t s = (hipStream_t)stream;

  // scratch for this call only
  std::vector<void*> bufs;
  auto alloc = [&](size_t bytes) -> void* {
    void* p = nullptr;
    if (hipMalloc(&p, bytes) != hipSuccess) return nullptr;
    bufs.push_back(p);
    return p;
  };
  auto release = [&]() {
    for (void* p : bufs) (void)hipFree(p);
    bufs.clear();
  };
  double *S = (double*)alloc(n * 8), *K = (double*)alloc(n * 8), *T = (double*)alloc(n * 8),
         *r = (double*)alloc(n * 8), *q = (double*)alloc(n * 8), *sig = (double*)alloc(n * 8),
         *P = (double*)alloc(n * 8), *o1 = (double*)alloc(n * 8), *o2 = (double*)alloc(n * 8);
  int8_t* flag = (int8_t*)alloc(n);
  uint8_t* st = (uint8_t*)alloc(n);
  float* f32 = kernel == FV_KERNEL_IV_HALLEY_F32 ? (float*)alloc((size_t)6 * n * 4) : nullptr;
  int64_t *cmo = (int64_t*)alloc((n_chains + 1) * 8), *mqo = (int64_t*)alloc((n_mat + 1) * 8);
  double *cF = (double*)alloc(n_chains * 8), *cr = (double*)alloc(n_chains * 8),
         *cT = (double*)alloc(n_mat * 8);
  for (void* p : bufs)
    if (!p) {
      release();
      return fail(FV_E_HIP, "fv_autotune: device allocation failed");
    }
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess) {
    release();
    return fail(FV_E_HIP, "fv_autotune: event creation failed");
  }
  if (hipEventCreate(&e1) != hipSuccess) {
    (void)hipEventDestroy(e0);
    release();
    return fail(FV_E_HIP, "fv_autotune: event creation failed");
  }
  const unsigned g256 = (unsigned)((n + 255) / 256);
  k_tune_quotes<<<g256, 256, 0, s>>>(n, S, K, T, r, q, sig, flag);
  k_tune_chains<<<(unsigned)((n_mat + 256) / 256), 256, 0, s>>>(n_chains, n_mat, n, mats, per_mat,
                                                              T, r, cmo, mqo, cF, cr, cT);

  fv_quotes qs;
  memset(&qs, 0, sizeof(qs));
  qs.n = n;
  qs.price.ptr = P;
  qs.fs.ptr = S;
  qs.K.ptr = K;
  qs.T.ptr = T;
  qs.r.ptr = r;
  qs.q.ptr = q;
  qs.flag = flag;
  fv_arg sa;
  sa.ptr = sig;
  sa.value = 0.0;
  fv_chains cs;
  memset(&cs, 0, sizeof(cs));
  cs.n_chains = n_chains;
  cs.n_maturities = n_mat;
  cs.n_quotes = n;
  cs.chain_mat_off = cmo;
  cs.mat_quote_off = mqo;
  cs.F = cF;
  cs.r = cr;
  cs.T = cT;
  cs.price = P;
  cs.K = K;
  cs.flag = flag;

  int rc = FV_OK;
  // input prices: the model's own prices of sigma (the chain kernel reads
  // Black-76 prices of the chain forwards)
  if (kernel == FV_KERNEL_CHAINS) {
    k_tune_expand<<<g256, 256, 0, s>>>(n, mats, per_mat, cT, cr, o1, o2);
    fv_quotes cq = qs;
    cq.fs.ptr = nullptr;
    cq.fs.value = 100.0;
    cq.T.ptr = o1;
    cq.r.ptr = o2;
    rc = fv_price(FV_MODEL_BLACK76, &cq, sa, P, stream);
  } else {
    rc = fv_price(model, &qs, sa, P, stream);
  }
  fv_quotes_f32 q32;
  memset(&q32, 0, sizeof(q32));
  if (f32) {
    k_tune_to_f32<<<g256, 256, 0, s>>>(n, P, S, K, T, r, q, f32);
    q32.n = n;
    q32.price.ptr = f32;
    q32.fs.ptr = f32 + n;
    q32.K.ptr = f32 + 2 * n;
    q32.T.ptr = f32 + 3 * n;
    q32.r.ptr = f32 + 4 * n;
    q32.q.ptr = f32 + 5 * n;
    q32.flag = flag;
  }

  auto run = [&]() -> int {
    switch (kernel) {
      case FV_KERNEL_PRICE: return fv_price(model, &qs, sa, o1, stream);
      case FV_KERNEL_IV_LBR: return fv_implied_vol(model, FV_SOLVER_LBR, &qs, o1, st, nullptr, stream);
      case FV_KERNEL_IV_HALLEY:
        return fv_implied_vol(model, FV_SOLVER_HALLEY, &qs, o1, st, nullptr, stream);
      case FV_KERNEL_GREEKS: return fv_greeks(model, &qs, sa, o1, o2, nullptr, nullptr, nullptr, stream);
      case FV_KERNEL_BACKWARD:
        return fv_implied_vol_backward(model, &qs, sig, sig, o1, o2, nullptr, nullptr, nullptr,
                                       nullptr, stream);
      case FV_KERNEL_IV_HALLEY_F32:
        return fv_implied_vol_f32(model, &q32, (float*)o1, st, stream);
      default: return fv_implied_vol_chains(FV_SOLVER_LBR, &cs, o1, st, stream);
    }
  };
  int best = 0;
  float best_ms = 1e30f;
  for (int b : {64, 128, 256, 512}) {
    if (rc != FV_OK) break;
    g_tuning_kernel = kernel;
    g_tuning_block = b;
    rc = run();  // warm-up
    float mn = 1e30f;
    for (int rep = 0; rep < 3 && rc == FV_OK; ++rep) {
      if (hipEventRecord(e0, s) != hipSuccess) {
        rc = fail(FV_E_HIP, "fv_autotune: event record");
        break;
      }
      rc = run();
      float ms = 0.0f;
      if (rc == FV_OK && (hipEventRecord(e1, s) != hipSuccess ||
                          hipEventSynchronize(e1) != hipSuccess ||
                          hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
        rc = fail(FV_E_HIP, "fv_autotune: event timing");
      mn = std::min(mn, ms);
    }
    if (rc == FV_OK && mn < best_ms) {
      best_ms = mn;
      best = b;
    }
  }
  g_tuning_kernel = -1;
  if (rc == FV_OK && best) g_tuned[kernel][tuned_model][bucket] = Tuned{best, 1, best_ms};
  // best-effort cleanup: an error here cannot change the result above
  (void)hipStreamSynchronize(s);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  release();
  return rc;
}

int fv_launch_shape(int kernel, int model, int64_t n, int* block, int* qpt) {
  if (kernel < 0 || kernel >= FV_KERNEL_COUNT || !block || !qpt)
    return fail(FV_E_INVALID_ARG, "kernel id or NULL output");
  if (model < FV_MODEL_BLACK76 || model > FV_MODEL_BSM)
    return fail(FV_E_INVALID_ARG, "model out of range");
  if (n < 1) return fail(FV_E_INVALID_ARG, "n < 1");
  *block = block_for(kernel, kernel == FV_KERNEL_CHAINS ? FV_MODEL_BLACK76 : model, n);
  *qpt = kernel == FV_KERNEL_CHAINS ? chain_slices(n) : 1;
  return FV_OK;
}

int fv_tuning_reset(void) {
  memset(g_tuned, 0, sizeof(g_tuned));
  return FV_OK;
}

int fv_tuning_save(const char* path) {
  if (!path) return fail(FV_E_INVALID_ARG, "path is NULL");
  std::string arch;
  const int rc = device_arch(&arch);
  if (rc) return rc;
  FILE* f = fopen(path, "w");
  if (!f) return fail(FV_E_INVALID_ARG, std::string("cannot write ") + path);
  fprintf(f, "{\"format\": \"fastvol-tuning\", \"version\": 1, \"arch\": \"%s\", \"entries\": [",
          arch.c_str());
  bool first = true;
  for (int k = 0; k < FV_KERNEL_COUNT; ++k)
    for (int m = 0; m < kModels; ++m)
      for (int b = 0; b < kBuckets; ++b) {
        const Tuned& t = g_tuned[k][m][b];
        if (!t.block) continue;
        fprintf(f, "%s\n  {\"kernel\": %d, \"model\": %d, \"bucket\": %d, \"block\": %d, "
                   "\"qpt\": %d, \"ms\": %.6g}",
                first ? "" : ",", k, m, b, t.block, t.qpt, (double)t.ms);
        first = false;
      }
  fprintf(f, "\n]}\n");
  const bool ok = !ferror(f);
  fclose(f);
  return ok ? FV_OK : fail(FV_E_INVALID_ARG, std::string("write failed: ") + path);
}

int fv_tuning_load(const char* path) {
  if (!path) return fail(FV_E_INVALID_ARG, "path is NULL");
  std::string text, arch;
  Tuned table[FV_KERNEL_COUNT][kModels][kBuckets];
  int rc = parse_tuning(path, &text, &arch, table);
  if (rc) return rc;
  std::string here;
  rc = device_arch(&here);
  if (rc) return rc;
  if (arch != here)
    return fail(FV_E_UNSUPPORTED, "tuning file is for " + arch + ", this device is " + here);
  memcpy(g_tuned, table, sizeof(g_tuned));
  return FV_OK;
}

}  // extern "C"
