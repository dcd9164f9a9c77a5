// fv_csr.h -- wave-cooperative location of quotes in CSR (offset-array)
// layouts: chain -> maturity -> quote, as the ragged-chain and calibration
// kernels read them.  Every helper here is called by all 64 lanes of a wave
// together and returns wave-uniform results, but the lanes' offsets of a slice.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fv {

constexpr int64_t kOffEnd = INT64_MAX;

__device__ __forceinline__ int64_t ld_off(const int64_t* __restrict__ off, int64_t count,
                                          int64_t idx) {
  return idx < count ? off[idx] : kOffEnd;
}

// The starts after an index, relative to a key (lane j holds off[base + 1 + j]
// - key, or kRelEnd from there on and past the last entry: a wave looks no
// further than that), consumed in order through a wave-uniform cursor.  A
// start before the key is -1: of those only the sign is read, and a batch may
// hold many times 2^31 quotes.
constexpr int kRelEnd = 0x7fffffff;
struct OffWindow {
  const int64_t* off;
  int64_t count, base, key;
  int v, j;
  __device__ __forceinline__ int load() const {
    const int64_t d = ld_off(off, count, base + 1 + __lane_id()) - key;
    return d < kRelEnd ? (d < 0 ? -1 : (int)d) : kRelEnd;
  }
  // Returns the largest m in [0, count) with off[m] <= key (off
  // non-decreasing, off[0] <= key), and leaves the window at the starts after
  // it.  A 64-ary search: each level is one load per lane at 64 evenly spaced
  // candidates and a ballot, and the last, at distance 1, is the window
  // itself: a dependent load less per search than with a window of its own,
  // and the location is a chain of those.  With the window in 32 bits, 273k
  // quotes in 60 chains (Halley) 8.8 -> 8.2 us, 8.4M in 2,000 (LBR) 130 ->
  // 125, the calibration's step on 500 chains 51.6 -> 49.1 (any count and any
  // distance, below, take 0.5 of that back).  The loads stay below `count`;
  // malformed (decreasing) offsets still shrink the range every level and give
  // an m below it.
  __device__ __forceinline__ int64_t locate(const int64_t* __restrict__ o, int64_t c, int64_t k) {
    off = o;
    count = c;
    key = k;
    const uint32_t next = (uint32_t)__lane_id() + 1;
    base = 0;
    int64_t left = count;  // m is in [base, base + left)
    // by halves down to what the candidates' 32 bits hold (the calibration
    // takes any number of chains; the shift is scalar, a 64-bit comparison
    // is not)
    while (__builtin_expect((int)(left >> 31), 0)) {
      const int64_t half = left >> 1;
      const bool le = off[base + half] <= key;
      base += le ? half : 0;
      left = le ? left - half : half;
    }
    while (left > 64) {
      const uint32_t step = (uint32_t)((left + 63) >> 6);
      const uint32_t at = next * step;
      const bool le = at < (uint32_t)left && (off + base)[at] <= key;
      const int64_t skip = (int64_t)__popcll(__ballot(le)) * step;
      base += skip;
      left = min(left - skip, (int64_t)step);
    }
    v = load();
    j = __popcll(__ballot(v <= 0));
    return base + j;
  }
  __device__ __forceinline__ int peek() {
    if (j == 64) {
      base += 64;
      j = 0;
      v = load();
    }
    return __builtin_amdgcn_readlane(v, j);
  }
  __device__ __forceinline__ void pop() { ++j; }
};

// Maturity and chain of every lane's quote as a wave walks consecutive
// 64-quote slices in increasing order (slice k covers quotes i0 .. i0 + 63,
// lane l holds quote i0 + l).  The wave finds the maturity and chain of its
// first quote by two 64-ary searches, then keeps a window of the next 64
// maturity starts and chain starts in registers: each slice reads the starts
// that fall inside it (a few wave-uniform readlanes, usually none) and every
// lane gets its maturity and chain without a search of its own.
struct ChainCursor {
  OffWindow mw, cw;
  int64_t mstart, cstart;  // maturity and chain of the current slice's first quote
  __device__ __forceinline__ void init(const int64_t* mat_quote_off, int64_t n_mat,
                                       const int64_t* chain_mat_off, int64_t n_chains,
                                       int64_t w0) {
    mstart = mw.locate(mat_quote_off, n_mat, w0);
    cstart = cw.locate(chain_mat_off, n_chains, mstart);
  }
  // The slice starting at quote i0 whose last quote is ilast.  The lane's
  // maturity and chain, as offsets from those of quote i0, which are returned
  // in m0 and c0: uniform bases and 32-bit lane offsets are what the loads
  // take, and lane comparisons of 32 bits.
  __device__ __forceinline__ void slice(int64_t i0, int64_t ilast, int64_t& m0, int& m,
                                        int64_t& c0, int& c) {
    const int lane = (int)__lane_id();
    // maturity of every lane: starts at or before i0, then those inside
    const int first = (int)(i0 - mw.key), last = (int)(ilast - mw.key);
    while (mw.peek() <= first) { ++mstart; mw.pop(); }
    m0 = mstart;
    m = 0;
    int npop = 0;
    for (int b; (b = mw.peek()) <= last; mw.pop(), ++npop) m += lane >= b - first;
    // chain of every lane, keyed by maturity
    const int mfirst = (int)(mstart - cw.key);
    while (cw.peek() <= mfirst) { ++cstart; cw.pop(); }
    c0 = cstart;
    c = 0;
    int cpop = 0;
    for (int b; (b = cw.peek()) <= mfirst + npop; cw.pop(), ++cpop) c += m >= b - mfirst;
    mstart += npop;
    cstart += cpop;
  }
};

}  // namespace fv
