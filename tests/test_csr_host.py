"""The wave's location of its quotes (fv_csr.h) on the CPU: the header is
compiled against a model of the wave, 64 fibers that meet at every cross-lane
operation, and its maturities and chains are compared with a plain search.  No
quote is needed, so the offsets can be as large as the entry points accept."""
import ctypes
import mmap
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WAVE = r'''
#pragma once
#include <stdint.h>
#include <stdlib.h>
#include <ucontext.h>
#include <algorithm>
#define __device__
#define __forceinline__ inline
using std::max;
using std::min;
static ucontext_t g_host, g_lane[64];
static int g_cur, g_done, g_phase[64];
static uint64_t g_slot[2][64];
inline int __lane_id() { return g_cur; }
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
// every lane stores a value, then reads all lanes'
inline const uint64_t* wave_exchange(uint64_t v) {
  const int me = g_cur, p = g_phase[me]++ & 1;
  g_slot[p][me] = v;
  swapcontext(&g_lane[me], &g_host);
  return g_slot[p];
}
inline uint64_t __ballot(bool b) {
  const uint64_t* s = wave_exchange(b);
  uint64_t m = 0;
  for (int j = 0; j < 64; ++j) m |= s[j] << j;
  return m;
}
inline int wave_readlane(int v, int lane) { return (int)(uint32_t)wave_exchange((uint32_t)v)[lane]; }
#define __builtin_amdgcn_readlane wave_readlane
static void (*g_body)(int);
inline void wave_main(int lane) {
  g_body(lane);
  ++g_done;
}
inline void run_wave(void (*body)(int)) {
  static char* stacks = (char*)malloc(64 * 65536);
  g_body = body;
  g_done = 0;
  for (int l = 0; l < 64; ++l) {
    g_phase[l] = 0;
    getcontext(&g_lane[l]);
    g_lane[l].uc_stack.ss_sp = stacks + l * 65536;
    g_lane[l].uc_stack.ss_size = 65536;
    g_lane[l].uc_link = &g_host;
    makecontext(&g_lane[l], (void (*)())wave_main, 1, l);
  }
  while (g_done < 64) {
    const int before = g_done;
    for (g_cur = 0; g_cur < 64; ++g_cur) swapcontext(&g_host, &g_lane[g_cur]);
    if (g_done != before && g_done != 64) abort();  // the lanes parted
  }
}
'''

SRC = r'''
#include "fv_csr.h"
static const int64_t *g_mo, *g_co;
static int64_t g_nm, g_nc, g_n, g_w0, *g_m, *g_c;
static int g_slices;
extern "C" void h_slices(const int64_t* mo, int64_t nm, const int64_t* co, int64_t nc, int64_t n,
                         int64_t w0, int slices, int64_t* m, int64_t* c) {
  g_mo = mo; g_nm = nm; g_co = co; g_nc = nc; g_n = n; g_w0 = w0; g_slices = slices; g_m = m; g_c = c;
  run_wave([](int lane) {
    fv::ChainCursor cur;
    cur.init(g_mo, g_nm, g_co, g_nc, g_w0);
    for (int s = 0; s < g_slices; ++s) {
      const int64_t i0 = g_w0 + 64 * s;
      if (i0 >= g_n) break;
      int64_t m0, c0;
      int m, c;
      cur.slice(i0, min(i0 + 63, g_n - 1), m0, m, c0, c);
      g_m[64 * s + lane] = m0 + m;
      g_c[64 * s + lane] = c0 + c;
    }
  });
}
'''


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("csr")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(WAVE)
    (d / "s.cpp").write_text(SRC)
    so = str(d / "s.so")
    subprocess.run(["g++", "-O1", "-std=gnu++17", "-shared", "-fPIC", "-I" + str(d),
                    "-I" + os.path.join(ROOT, "paper_2604_27210_amd", "csrc"), str(d / "s.cpp"), "-o", so],
                   check=True)
    return ctypes.CDLL(so)


def _p(a):
    return ctypes.c_void_p(a.ctypes.data)


def _check(host, mqo, cmo, w0, slices):
    nm, nc, n = len(mqo) - 1, len(cmo) - 1, int(mqo[-1])
    m, c = (np.full(64 * slices, -1, dtype=np.int64) for _ in range(2))
    host.h_slices(_p(mqo), ctypes.c_int64(nm), _p(cmo), ctypes.c_int64(nc), ctypes.c_int64(n),
                  ctypes.c_int64(w0), slices, _p(m), _p(c))
    i = np.arange(w0, min(w0 + 64 * slices, n))
    want = np.searchsorted(mqo[:nm], i, side="right") - 1
    assert np.array_equal(m[:len(i)], want), (w0, m[:len(i)], want)
    assert np.array_equal(c[:len(i)], np.searchsorted(cmo[:nc], want, side="right") - 1), w0


# quotes per maturity, maturities per chain (0: empty)
LAYOUTS = {
    "short": ([3, 1, 0, 70, 200], [1, 2, 0, 4], 500),
    "a start far behind": ([1, 3_000_000_000, 129, 5_000_000_000, 1], [1, 2], 5),
    "60 of 50M": ([50_000_000], [7], 60),
    "5,000 of 10M": ([10_000_000, 0, 63], [3, 0, 1], 5000),
    "the most quotes": ([(1 << 46) // 100], [10], 99),
}


@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_location_equals_a_plain_search(host, layout):
    sizes, per_chain, nm = LAYOUTS[layout]
    mqo = np.r_[0, np.cumsum(np.resize(sizes, nm))].astype(np.int64)
    cuts = np.cumsum(np.resize(per_chain, nm * len(per_chain)))
    cmo = np.r_[0, cuts[cuts < nm], nm].astype(np.int64)
    n = int(mqo[-1])
    rng = np.random.default_rng(nm)
    at = np.r_[0, n - 1, n // 2, rng.integers(0, n, 40), rng.choice(mqo, 20) - 64]
    for w0 in np.unique(np.clip(at, 0, n - 1) // 128 * 128):
        for slices in (1, 2):
            _check(host, mqo, cmo, int(w0), slices)


@pytest.mark.parametrize("chains", [(1 << 31) + 5, (1 << 32) - 10, (1 << 32) + 1000, (1 << 33) + 77])
@pytest.mark.parametrize("tail", [1, 300])
def test_chains_beyond_32_bits(host, chains, tail):
    """The calibration takes any number of chains, most of them empty here:
    all but the last `tail` start at maturity 0 (untouched pages of a mapping),
    those at one maturity each."""
    size = 8 * (chains + 1)
    buf = mmap.mmap(-1, size, flags=mmap.MAP_PRIVATE | mmap.MAP_ANONYMOUS | 0x4000)  # not reserved
    cmo = np.frombuffer(buf, dtype=np.int64)
    cmo[-tail:] = np.arange(1, tail + 1)
    mqo = np.arange(0, 65 * tail + 1, 65, dtype=np.int64)
    for w0 in range(0, int(mqo[-1]), 64 if tail == 1 else 1280):
        _check(host, mqo, cmo, w0, 1)
