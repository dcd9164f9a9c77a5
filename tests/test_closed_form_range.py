"""The scaled closed forms (price, Greeks, partials from one evaluation) at
spots of any size, on the CPU: the headers are compiled for the host, and
wherever the scaled forms say they hold, they agree with the general ones."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle
from _helpers import U

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r'''
#include <cstdint>
#include "fv_quote.h"
extern "C" void h_forms(int model, int64_t n, const double* fs, const double* K, const double* T,
                        const double* r, const double* q, const double* sg, const int8_t* th,
                        int8_t* fast, double* scaled, double* general) {
  for (int64_t i = 0; i < n; ++i) {
    fv::ClosedForm c;
    fast[i] = fv::closed_form(model, fs[i], K[i], T[i], r[i], q[i], sg[i], th[i], &c);
    const double F = fv::forward_of(model, fs[i], T[i], r[i], q[i]), D = fv::fexp_prod(-r[i], T[i]);
    const double P = fv::price_at(F, K[i], D, sg[i], fv::sqrt_pos(T[i]), th[i]);
    const fv::Greeks g = fv::greeks_of(c, model, fs[i], T[i], r[i], q[i], sg[i], th[i], c.D * c.t.P);
    const fv::PricePartials p =
        fv::partials_of(c, model, fs[i], K[i], T[i], r[i], q[i], sg[i], th[i], c.D * c.t.P);
    const fv::Greeks gg = fv::greeks_at(model, fs[i], K[i], T[i], r[i], q[i], sg[i], th[i], F, D, P);
    const fv::PricePartials pp =
        fv::price_partials(model, fs[i], K[i], T[i], r[i], q[i], sg[i], th[i], F, D, P);
    const double a[] = {c.D * c.t.P, g.delta, g.gamma, g.vega, g.rho, p.dK, p.dq};
    const double b[] = {P, gg.delta, gg.gamma, gg.vega, gg.rho, pp.dK, pp.dq};
    for (int j = 0; j < 7; ++j) {
      scaled[7 * i + j] = a[j];
      general[7 * i + j] = b[j];
    }
  }
}
extern "C" void h_at(double F, double K, double D, double sg, int th, double* o) {
  o[0] = fv::price_at(F, K, D, sg, 1.0, th);
  const fv::Greeks g = fv::greeks_at(1, 1e-200, K, 1.0, -2.0, 0.0, sg, th, F, D, o[0]);
  o[1] = g.delta, o[2] = g.gamma, o[3] = g.vega, o[4] = g.rho;
}
'''
NAMES = ["price", "delta", "gamma", "vega", "rho", "dK", "dq"]


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("forms")
    src, so = str(d / "s.cpp"), str(d / "s.so")
    with open(src, "w") as f:
        f.write(SRC)
    csrc = os.path.join(ROOT, "paper_2604_27210_amd", "csrc")
    subprocess.run(["g++", "-O2", "-std=gnu++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I" + csrc, src, "-o", so], check=True)
    return ctypes.CDLL(so)


def _forms(host, model, *cols, th):
    n = len(cols[0])
    cols = [np.ascontiguousarray(c, dtype=np.float64) for c in cols]
    th = np.full(n, th, dtype=np.int8)
    fast, a, b = np.zeros(n, dtype=np.int8), np.empty((n, 7)), np.empty((n, 7))
    p = lambda v: v.ctypes.data_as(ctypes.c_void_p)
    host.h_forms(model, ctypes.c_int64(n), *[p(c) for c in cols], p(th), p(fast), p(a), p(b))
    return fast.astype(bool), a, b


@pytest.mark.parametrize("model", [0, 1, 2])
@pytest.mark.parametrize("th", [1, -1])
def test_small_and_large_spots(host, model, th):
    """Out of the money down to the last binary64 densities, spots from
    2^-300 to 2^300, total volatilities from 2^-30 to 8, rates that grow or
    discount by up to e^150.  Every factor is a product of a few values within
    2 u, but the density's: its exponent -d^2/2 is rounded (u d^2/2), and d
    itself (2 u d, d^2 in the exponent again): 64 u (1 + d^2/2) covers both
    forms.  A value below the normal range has its last place instead."""
    rng = np.random.default_rng(17 + model)
    n = 60_000
    s = np.exp(rng.uniform(np.log(2.0 ** -30), np.log(8.0), n))
    h = rng.uniform(0.0, 37.5, n)
    fs = 2.0 ** rng.uniform(-300.0, 300.0, n)
    T = np.exp(rng.uniform(np.log(1e-3), np.log(50.0), n))
    r = rng.choice([0.0, 0.03, -150.0, 150.0], n) / T
    q = r * rng.choice([0.0, 1.0, 0.99], n) if model == 2 else np.zeros(n)
    F = fs * np.exp((r - q) * T) if model else fs
    K = F * np.exp(th * h * s)  # out of the money
    ok = np.isfinite(K) & (K > 1e-300) & np.isfinite(F) & (F > 1e-300)
    fs, K, T, r, q, s, h = (v[ok] for v in (fs, K, T, r, q, s, h))
    with np.errstate(all="ignore"):
        fast, a, b = _forms(host, model, fs, K, T, r, q, s / np.sqrt(T), th=th)
    assert fast.mean() > 0.2
    tol = (64 * U * (1.0 + 0.5 * (h + s) ** 2))[:, None]
    bad = fast[:, None] & ~(np.abs(a - b) <= tol * np.abs(b) + 2.0 ** -1070)
    # where the general form's own density or tail (at h + s/2) leaves the
    # normal range it is the one that is off: binary128 there
    i = np.where(bad.any(axis=1) & (h + 0.5 * s > 37.0))[0]
    if len(i):
        fl = np.full(len(i), th, dtype=np.int8)
        name = ["black76", "bs", "bsm"][model]
        c = [v[i] for v in (fs, K, T, r, q, s / np.sqrt(T))]
        P, g = oracle.price(name, *c, fl), oracle.greeks(name, *c, fl)
        v = oracle.iv_grad_at(name, *c, fl)  # -(dP/dX)/vega
        ref = np.stack([P, g["delta"], g["gamma"], g["vega"], g["rho"], -v[:, 2] * g["vega"], -v[:, 5] * g["vega"]], 1)
        bad[i] &= ~(np.abs(a[i] - ref) <= tol[i] * np.abs(ref) + 2.0 ** -1070)
    for j, name in enumerate(NAMES):
        i = np.where(bad[:, j])[0]
        assert len(i) == 0, (name, len(i), ["fs %.3g T %.3g r %.3g s %.3g h %.3g: %.17g %.17g"
                                            % (fs[k], T[k], r[k], s[k], h[k], a[k, j], b[k, j]) for k in i[:3]])


@pytest.mark.parametrize("K", [100.0, 1e-3, 1e-200])
@pytest.mark.parametrize("sigma", [0.3, 0.0])
def test_forward_that_underflows(host, K, sigma):
    """A forward of 0 has no logarithm: each value is NaN or the limit (a call
    worth nothing, a put worth the discounted strike), never another number."""
    for th, limit in ((1, [0.0, 0.0, 0.0, 0.0, 0.0]), (-1, [2.0 * K, 0.0, 0.0, 0.0, -2.0 * K])):
        o = np.empty(5)
        host.h_at(*[ctypes.c_double(v) for v in (0.0, K, 2.0, sigma)], th, o.ctypes.data_as(ctypes.c_void_p))
        assert np.all(np.isnan(o) | (o == limit)), (th, o)
