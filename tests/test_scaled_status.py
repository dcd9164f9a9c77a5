"""Quotes that the scaled solves take have the status that the general
reduction gives them, on the CPU: over prices of every size, at and around the
money, at and beyond the bounds, with missing and impossible inputs."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r'''
#include <cstdint>
#include "fv_f32.h"
#include "fv_quote.h"
// `taken`: the status the kernels give without the general path, 255 where
// they ask it.
extern "C" void h_status64(int model, int64_t n, const double* P, const double* fs, const double* K,
                           const double* T, const double* r, const double* q, const int8_t* th,
                           uint8_t* taken, uint8_t* general) {
  for (int64_t i = 0; i < n; ++i) {
    const fv::ScaledQuote s = fv::scaled_quote(model, P[i], fs[i], K[i], T[i], r[i], q[i], th[i]);
    bool ask = s.general;
    double root;
    if (s.status == fv::kQOk && !ask) ask = !fv::lbr_solve_scaled(s.x, s.bh, s.ch, &root);
    taken[i] = ask ? 255 : s.status;
    general[i] = fv::reduce_quote(model, P[i], fs[i], K[i], T[i], r[i], q[i], th[i]).status;
  }
}
extern "C" void h_status32(int model, int64_t n, const double* P, const double* fs, const double* K,
                           const double* T, const double* r, const double* q, const int8_t* th,
                           uint8_t* taken, uint8_t* general) {
  for (int64_t i = 0; i < n; ++i) {
    const float v[] = {(float)P[i], (float)fs[i], (float)K[i], (float)T[i], (float)r[i], (float)q[i]};
    const fv32::ScaledQuote s =
        fv32::scaled_quote(model, v[0], v[1], v[2], v[3], v[4], v[5], th[i]);
    bool ask = s.general;
    fv32::HalleyState hs;
    if (s.status == 0 && !ask) ask = !fv32::halley_solve_scaled(s, 8, &hs);
    taken[i] = ask ? 255 : s.status;
    general[i] = fv32::reduce_quote(model, v[0], v[1], v[2], v[3], v[4], v[5], th[i]).status;
  }
}
'''


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("status")
    src, so = str(d / "s.cpp"), str(d / "s.so")
    with open(src, "w") as f:
        f.write(SRC)
    csrc = os.path.join(ROOT, "paper_2604_27210_amd", "csrc")
    subprocess.run(["g++", "-O2", "-std=gnu++17", "-ffp-contract=off", "-shared", "-fPIC",
                    "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + csrc, src, "-o", so], check=True)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("bits", [64, 32])
@pytest.mark.parametrize("model", [0, 1, 2])
def test_status_as_the_general_reduction(host, bits, model):
    rng = np.random.default_rng(10 * bits + model)
    n = 300_000
    f = np.float64 if bits == 64 else np.float32
    tiny, huge = (1e-307, 1e307) if bits == 64 else (1e-37, 1e37)
    logu = lambda lo, hi: np.exp(rng.uniform(np.log(lo), np.log(hi), n))
    pick = lambda *v: rng.choice(v, n)
    special = np.array([0.0, -0.0, np.nan, np.inf, -np.inf, -1.0, tiny / 100, tiny, huge, 1.0])
    some = lambda v: np.where(rng.random(n) < 0.01, rng.choice(special, n), v)
    with np.errstate(all="ignore"):
        fs = some(np.where(rng.random(n) < 0.8, logu(1e-3, 1e5), logu(tiny, huge)))
        T = some(np.where(rng.random(n) < 0.8, logu(1e-3, 40.0), logu(tiny, 1e4)))
        r = some(rng.uniform(-0.02, 0.1, n))
        # only Black-Scholes-Merton has a yield; the kernels pass 0 for the others
        q = some(rng.uniform(0.0, 0.06, n)) if model == 2 else np.zeros(n)
        long = rng.random(n) < 0.05
        r = np.where(long, rng.uniform(-90.0, 90.0, n) * (1 if bits == 32 else 8) / T, r)
        F = fs * np.exp((r - q) * T) if model else fs
        # at the money to the last place, or any number of standard deviations away
        K = some(F * np.where(rng.random(n) < 0.3, 1.0 + pick(-2, -1, 0, 0, 1, 2) * np.finfo(f).eps,
                              np.exp(rng.normal(0.0, 1.0, n) * logu(1e-6, 30.0))))
        fs, T, r, q, K = (v.astype(f).astype(np.float64) for v in (fs, T, r, q, K))
        th = pick(1, -1).astype(np.int8)
        th[rng.random(n) < 0.002] = 0
        intrinsic, upper = np.maximum(th * (F - K), 0.0), np.where(th > 0, F, K)
        # time values of every size up to the bound, and prices on and off both
        value = intrinsic + (upper - intrinsic) * np.where(rng.random(n) < 0.7, rng.random(n), logu(tiny, 1.0))
        value = np.where(rng.random(n) < 0.2, pick(1.0, 0.0) * (upper - intrinsic) + intrinsic, value)
        P = np.exp(-r * T) * value
        P = np.where(rng.random(n) < 0.1, P * (1.0 + pick(-2, -1, 1, 2) * np.finfo(f).eps), P)
        P = some(P).astype(f).astype(np.float64)
    cols = [np.ascontiguousarray(v, dtype=np.float64) for v in (P, fs, K, T, r, q)]
    taken, general = np.empty(n, dtype=np.uint8), np.empty(n, dtype=np.uint8)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    (host.h_status64 if bits == 64 else host.h_status32)(model, ctypes.c_int64(n), *[p(c) for c in cols], p(th),
                                                         p(taken), p(general))
    mine = taken != 255
    assert mine.mean() > 0.5 and len(np.unique(taken)) >= 5
    bad = np.where(mine & (taken != general))[0]
    assert len(bad) == 0, (len(bad), [(taken[i], general[i], P[i], fs[i], K[i], T[i], r[i], th[i]) for i in bad[:4]])
