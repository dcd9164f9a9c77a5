"""The scaled solves (binary32 start, binary64 last steps) at the edges of
the domain that sends a quote to them, against the oracle: |ln(F/K)| at 0,
one ulp and around 128, beta/b_max around 2^-960 and 1 - 2^-40, forwards and
strikes around 2^+-1000, tiny and long maturities; on both sides of each edge
the quote takes another path and the answer has to hold.

On the CPU the same headers are compiled for the host and the scaled roots
compared with the general solver's over the plane both accept."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle
from _helpers import U, compare_iv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r'''
#include <cstdint>
#include "fv_quote.h"
extern "C" void h_scaled(int64_t n, const double* x, const double* s, double* lbr, double* hal,
                         double* gen) {
  for (int64_t i = 0; i < n; ++i) {
    const double bmax = fv::fexp(0.5 * x[i]);
    const fv::NBlack nb = fv::normalised_black(x[i], s[i], bmax);
    const double bh = nb.b / bmax, ch = nb.c / bmax;
    lbr[i] = hal[i] = gen[i] = -1.0;
    if (!fv::scaled_domain(x[i], bh, ch)) continue;
    if (!fv::lbr_solve_scaled(x[i], bh, ch, &lbr[i])) lbr[i] = -2.0;
    const fv::HalleyState hs = fv::halley_solve_scaled(x[i], bh, ch, 8);
    hal[i] = hs.converged ? hs.s : -2.0;
    gen[i] = fv::lbr_solve(x[i], nb.b, bmax, fv::flog(nb.b), 2, 4, 1e-6).s;
  }
}
'''


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("scaled")
    src, so = str(d / "s.cpp"), str(d / "s.so")
    with open(src, "w") as f:
        f.write(SRC)
    csrc = os.path.join(ROOT, "paper_2604_27210_amd", "csrc")
    subprocess.run(["g++", "-O2", "-std=gnu++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I" + csrc, src, "-o", so], check=True)
    return ctypes.CDLL(so)


def test_scaled_roots_match_the_general_solver_on_the_host(host):
    """Every (x, s) of a log-spaced plane with beta below 0.99 b_max whose
    quote the scaled path accepts.  The general solver is within 8 u of the
    root times the conditioning 1 + b/(s b'), as the parity bound has it; the
    two may be that far apart twice over, and Halley keeps its 1e-8."""
    ax = np.concatenate([[0.0], np.geomspace(2.0 ** -53, 128.0, 120)])
    h = np.concatenate([-np.geomspace(1e-3, 30.0, 60)])
    x, s = [], []
    for a in ax:
        cand = a / -h if a > 0 else np.geomspace(1e-12, 6.0, 60)
        x += [-a] * len(cand)
        s += list(cand)
    x, s = np.array(x), np.array(s)
    keep = (s > 1e-16) & (s < 20.0) & (0.5 * s + x / s < 2.3)
    x, s = np.ascontiguousarray(x[keep]), np.ascontiguousarray(s[keep])
    out = [np.empty(len(x)) for _ in range(3)]
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    host.h_scaled(ctypes.c_int64(len(x)), p(x), p(s), *[p(o) for o in out])
    lbr, hal, gen = out
    inside = gen > 0
    assert inside.mean() > 0.9
    assert not np.any(lbr[inside] == -2.0) and not np.any(hal[inside] == -2.0)
    # b/b' <= s off the upper wing; kept below 0.99 b_max, b'/b_max > 0.02
    cond = 1.0 + 50.0 / s[inside] * np.minimum(1.0, s[inside])
    assert np.all(np.abs(lbr - gen)[inside] <= 16 * U * cond * gen[inside])
    assert np.all(np.abs(hal - gen)[inside] <= 1e-8 * gen[inside])


def _edge_quotes():
    """(F, K, T, r, sigma, flag) on both sides of every edge."""
    rows = []
    for fl in (1, -1):
        for sig in (0.02, 0.3, 2.0):  # at the money and one ulp from it
            for K in (100.0, np.nextafter(100.0, 200.0), np.nextafter(100.0, 0.0)):
                rows.append((100.0, K, 0.7, 0.03, sig, fl))
        for lx in (127.9, 127.9999, 128.0001, 128.1, 200.0):  # |x| around 128
            for sig in (4.0, 9.0, 16.0):
                rows.append((1.0, np.exp(lx), 1.0, 0.0, sig, 1))
                rows.append((1.0, np.exp(-lx), 1.0, 0.0, sig, -1))
        for e in (-1005, -1001, -1000, -999, -800, 800, 998, 999, 1000, 1005):  # F, K around 2^+-1000
            rows.append((2.0 ** e, 1.25 * 2.0 ** e, 0.5, 0.02, 0.4, fl))
        for T in (1e-300, 1e-289, 1e-12, 40.0, 80.0):
            rows.append((100.0, 100.0 * np.exp(-0.3 * np.sqrt(T)), T, 0.01, 0.4, fl))
    # deep out of the money: beta/b_max around 2^-960 (h^2/2 ~ 665), and high
    # total volatility: 1 - beta/b_max around 2^-40 (s ~ 14)
    for h in np.linspace(36.0, 37.2, 25):
        rows.append((100.0, 100.0 * np.exp(h * 0.2), 1.0, 0.0, 0.2, 1))
    for s in np.linspace(13.0, 15.5, 26):
        rows.append((100.0, 120.0, 1.0, 0.0, s, 1))
        rows.append((100.0, 80.0, 1.0, 0.0, s, -1))
    return [np.array(c, dtype=np.float64) for c in zip(*rows)]


@pytest.mark.gpu
@pytest.mark.parametrize("solver", ["lbr", "halley"])
@pytest.mark.parametrize("entry", ["flat", "chains"])
def test_domain_edges_against_the_oracle(solver, entry):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_27210_amd as fv
    F, K, T, r, sig, fl = _edge_quotes()
    flag = fl.astype(np.int8)
    P = oracle.price("black76", F, K, T, r, np.zeros_like(F), sig, flag)
    keep = (P > 0) & np.isfinite(P)
    F, K, T, r, P, flag = (a[keep] for a in (F, K, T, r, P, flag))
    n = len(F)
    d = lambda a, dt=torch.float64: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dt)
    if entry == "flat":
        s, st = fv.implied_vol("black76", d(P), d(F), d(K), d(T), d(r), flag=d(flag, torch.int8),
                               solver=solver)
    else:  # every quote a chain of one maturity of one strike
        off = torch.arange(n + 1, dtype=torch.int64, device="cuda")
        s, st = fv.implied_vol_chains(off, off, d(F), d(r), d(T), d(P), d(K), d(flag, torch.int8),
                                      solver=solver)
    res = compare_iv("black76", solver, P, F, K, T, r, np.zeros(n), flag, s.cpu().numpy(),
                     st.cpu().numpy())
    print("edges %s %s: %d quotes, %d solved, max err/tol %.3g"
          % (entry, solver, n, res["n_ok"], res["max_ratio"]))
    assert len(res["status_bad"]) == 0, res["status_bad"][:5]
    assert len(res["value_bad"]) == 0, (res["value_bad"][:5], res["max_ratio"])
    assert len(res["nan_bad"]) == 0 and res["n_ok"] > 0.8 * n
