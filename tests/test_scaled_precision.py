"""What the scaled solve leaves in a root it is handed the value of, on the CPU.
The calibration prices a volatility and takes the implied one, and its
gradient sums the difference over thousands of quotes, so the systematic part
counts and not only the largest error."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from _helpers import U

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r'''
#include <cstdint>
#include "fv_f32.h"
#include "fv_quote.h"
extern "C" void h_back(int64_t n, const double* x, const double* s, double* scaled, double* general) {
  for (int64_t i = 0; i < n; ++i) {
    double bh, ch;
    fv::scaled_value(x[i], s[i], &bh, &ch);
    scaled[i] = -1.0;
    if (fv::scaled_domain(x[i], bh, ch)) fv::lbr_solve_scaled(x[i], bh, ch, &scaled[i]);
    const double bmax = fv::fexp(0.5 * x[i]);
    const fv::NBlack nb = fv::normalised_black(x[i], s[i], bmax);
    general[i] = fv::lbr_solve(x[i], nb.b, bmax, nb.lnbp + fv::flog(nb.ratio), fv::kLbrMinSteps,
                               fv::kLbrMaxSteps, fv::kLbrStepTol).s;
  }
}
extern "C" void h_ratio(int64_t n, const double* x, const double* s, double* scaled,
                        double* general) {
  for (int64_t i = 0; i < n; ++i) {
    const fv::ScaledEval e = fv::scaled_eval(x[i], s[i]);
    const fv::NBlack nb = fv::normalised_black(x[i], s[i], fv::fexp(0.5 * x[i]));
    scaled[i] = e.rho;
    general[i] = e.comp ? nb.cratio : nb.ratio;
  }
}
extern "C" void h_ratio32(int64_t n, const double* x, const double* s, double* scaled,
                          double* general) {
  for (int64_t i = 0; i < n; ++i) {
    const float xf = (float)x[i], sf = (float)s[i];
    const fv::s32::Eval e = fv::s32::eval<fv::s32::kFitSolve>(-xf, sf);
    const fv32::NBlack nb = fv32::normalised_black(xf, sf, fv32::fexp(0.5f * xf));
    scaled[i] = e.rho;
    general[i] = (double)(e.comp ? nb.c : nb.b) / nb.bp;
  }
}
extern "C" void h_plane(int64_t n, const double* x, const double* s, double* lbr, double* hal,
                        double* cond) {
  for (int64_t i = 0; i < n; ++i) {
    const double bmax = fv::fexp(0.5 * x[i]);
    const fv::NBlack nb = fv::normalised_black(x[i], s[i], bmax);
    const double bh = nb.b / bmax, ch = nb.c / bmax;
    cond[i] = fmin(nb.b, nb.c) / (s[i] * nb.bp);
    lbr[i] = hal[i] = -1.0;
    if (!fv::scaled_domain(x[i], bh, ch)) continue;
    if (!fv::lbr_solve_scaled(x[i], bh, ch, &lbr[i])) lbr[i] = -2.0;
    const fv::HalleyState hs = fv::halley_solve_scaled(x[i], bh, ch, 8);
    hal[i] = hs.converged ? hs.s : -2.0;
  }
}
'''


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("back")
    src, so = str(d / "s.cpp"), str(d / "s.so")
    with open(src, "w") as f:
        f.write(SRC)
    csrc = os.path.join(ROOT, "paper_2604_27210_amd", "csrc")
    subprocess.run(["g++", "-O2", "-std=gnu++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I" + csrc, src, "-o", so], check=True)
    return ctypes.CDLL(so)


def test_a_priced_volatility_comes_back(host):
    """Strikes and volatilities of the calibration's chains.  The mean of
    s'/s - 1 stays below a quarter of the unit roundoff (its sampling error is
    3e-16 / sqrt(n) = 5e-19), as that of the general solve does; no root is
    further off than 32 u."""
    rng = np.random.default_rng(1)
    n = 300_000
    T = np.exp(rng.uniform(np.log(1.0 / 365.0), np.log(5.0), n))
    k = rng.uniform(-1.2, 1.2, n) * np.sqrt(T)
    s = np.ascontiguousarray((rng.uniform(0.12, 0.4, n) + 0.1 * k * k - 0.05 * k) * np.sqrt(T))
    x = -np.abs(k)
    out = [np.empty(n) for _ in range(2)]
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    host.h_back(ctypes.c_int64(n), p(x), p(s), *[p(o) for o in out])
    for root in out:
        err = root / s - 1.0
        assert np.max(np.abs(err)) <= 32 * U
        assert abs(err.mean()) <= 0.25 * U, err.mean()


def test_roots_by_their_conditioning(host):
    """The whole plane that the scaled solve takes, the upper wing down to
    1 - beta/b_max = 2^-40 with it: a value within a few u of its own (b, or
    b_max - b where that is the smaller) gives its s back within 16 u times
    1 + b/(s b') (or (b_max - b)/(s b')), and every quote settles."""
    rng = np.random.default_rng(2)
    n = 400_000
    s = np.exp(rng.uniform(np.log(1e-9), np.log(15.0), n))
    g = rng.uniform(-36.0, 7.3, n)  # h + t
    x = np.minimum(s * (g - 0.5 * s), 0.0)
    x[:2000] = 0.0
    keep = x >= -128.0
    x, s = np.ascontiguousarray(x[keep]), np.ascontiguousarray(s[keep])
    lbr, hal, cond = (np.empty(len(x)) for _ in range(3))
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    host.h_plane(ctypes.c_int64(len(x)), p(x), p(s), p(lbr), p(hal), p(cond))
    inside = lbr != -1.0
    assert inside.mean() > 0.8
    assert not np.any(lbr[inside] == -2.0) and not np.any(hal[inside] == -2.0)
    err = np.abs(lbr / s - 1.0)[inside] / (U * (1.0 + cond[inside]))
    print("LBR: %.3g u of the conditioning at most" % err.max())
    assert np.all(err <= 16.0)
    assert np.all(np.abs(hal / s - 1.0)[inside] <= 1e-8)


@pytest.mark.parametrize("bits", [64, 32])
def test_evaluation_as_precise_as_the_general_one(host, bits):
    """b/b' (or its complement) near the money, where an error in it is the
    root's: rms against 40 digits no larger than the general evaluator's, which
    takes both reciprocals by themselves (25% for the sample of 1,500 and the
    two roundings that the binary64 evaluation's common reciprocal leaves)."""
    mp = pytest.importorskip("mpmath").mp
    mp.dps = 40
    rng = np.random.default_rng(3)
    n = 1500
    s = np.exp(rng.uniform(np.log(0.01), np.log(2.0), n))
    x = -rng.uniform(0.0, 0.5, n) * s
    if bits == 32:
        s, x = (v.astype(np.float32).astype(np.float64) for v in (s, x))
    out = [np.empty(n) for _ in range(2)]
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    (host.h_ratio if bits == 64 else host.h_ratio32)(ctypes.c_int64(n), p(x), p(s), *[p(o) for o in out])
    want = []
    for xi, si in zip(x, s):
        h, t = mp.mpf(float(xi)) / mp.mpf(float(si)), mp.mpf(float(si)) / 2
        q1, q2 = -(h + t) / mp.sqrt(2), (t - h) / mp.sqrt(2)
        f = lambda q: mp.exp(q * q) * mp.erfc(q)
        v = f(-q1) + f(q2) if q1 < -0.5 else f(q1) - f(q2)
        want.append(mp.sqrt(mp.pi / 2) * v)
    rms = [float(mp.sqrt(sum((mp.mpf(float(a)) / w - 1) ** 2 for a, w in zip(o, want)) / n)) for o in out]
    print("b/b': scaled %.3g, general %.3g" % tuple(rms))
    assert rms[0] <= 1.25 * rms[1]
