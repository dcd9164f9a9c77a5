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


@pytest.mark.gpu
@pytest.mark.parametrize("model", ["black76", "bsm"])
def test_closed_form_edges_against_the_oracle(model):
    """Price, Greeks and the price adjoint on both sides of every edge of the
    scaled closed forms' domain: spot and strike around 2^+-300, total
    volatility around 2^-60 and 64, exponents around 200, a density around
    e^-690, F = K and one ulp from it, maturities from 1e-300 up; calls and
    puts.  Each value within 64 u times the conditioning that binary64
    arguments give a density or tail probability at d (greek_terms), the
    price as the Greeks."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_27210_amd as fv
    from _helpers import GREEK_NAMES, greek_terms, greeks_bad
    rows = []
    for e in (-301, -300, -299, 299, 300, 301):
        rows.append((2.0 ** e, 1.1 * 2.0 ** e, 0.5, 0.02, 0.01, 0.4))
    for s in (2.0 ** -61, 2.0 ** -60, 2.0 ** -59, 2.0 ** -30, 40.0, 63.9, 64.1):
        rows.append((100.0, 100.0, 1.0, 0.0, 0.0, s))
    for rT in (190.0, 199.9, 200.1, 260.0):
        rows.append((100.0, 100.0, 50.0, rT / 50.0, rT / 50.0, 0.3))
        rows.append((100.0, 100.0, 50.0, -rT / 50.0, -rT / 50.0, 0.3))
    for h in np.linspace(36.5, 37.6, 23):
        rows.append((100.0, 100.0 * np.exp(h * 0.25), 1.0, 0.0, 0.0, 0.25))
        rows.append((100.0, 100.0 * np.exp(-h * 0.25), 1.0, 0.0, 0.0, 0.25))
    for K in (100.0, np.nextafter(100.0, 200.0), np.nextafter(100.0, 0.0), 60.0, 170.0):
        for sg in (1e-3, 0.2, 2.0, 12.0):
            rows.append((100.0, K, 0.7, 0.0, 0.0, sg))
    for T in (1e-300, 1e-291, 1e-289, 1e-12, 60.0):
        rows.append((100.0, 100.0 * np.exp(0.4 * np.sqrt(T)), T, 0.03, 0.01, 0.5))
    cols = [np.array(c, dtype=np.float64) for c in zip(*rows)]
    cols = [np.concatenate([c, c]) for c in cols]
    S, K, T, r, q, sg = cols
    n = len(S)
    flag = np.where(np.arange(n) < n // 2, 1, -1).astype(np.int8)
    if model == "black76":
        q = np.zeros(n)
    d = lambda a, dt=torch.float64: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dt)
    kw = dict(flag=d(flag, torch.int8), q=d(q) if model == "bsm" else None)
    p = fv.price(model, d(S), d(K), d(T), d(r), d(sg), **kw).cpu().numpy()
    ref = oracle.price(model, S, K, T, r, q, sg, flag)
    # binary128 itself has no digits of F Phi(d1) - K Phi(d2) left at a total
    # volatility below 1e-30; at the money the price is m s/sqrt(2 pi) (1 +
    # O(s^2)) there
    tiny = (sg * np.sqrt(T) < 1e-30) & (S == K)
    ref = np.where(tiny, S * sg * np.sqrt(T) / np.sqrt(2.0 * np.pi), ref)
    kappa, _ = greek_terms(model, S, K, T, r, q, sg, flag, ref)
    bad = np.where(~(np.abs(p - ref) <= 64 * U * kappa * np.abs(ref) + 1e-300))[0]
    assert len(bad) == 0, [(S[i], K[i], T[i], sg[i], p[i], ref[i]) for i in bad[:4]]
    g = {k: v.cpu().numpy()
         for k, v in fv.greeks(model, d(S), d(K), d(T), d(r), d(sg), **kw).items()}
    bad, worst = greeks_bad(model, S, K, T, r, q, sg, flag, g, P=ref)
    print("closed-form edges %s: %d quotes, max err/tol %.3g" % (model, n, worst))
    for name in GREEK_NAMES:
        assert len(bad[name]) == 0, (name, [(S[i], K[i], T[i], sg[i]) for i in bad[name][:4]])
    a = {k: v.cpu().numpy()
         for k, v in fv.price_backward(model, d(S), d(K), d(T), d(r), d(sg), d(np.ones(n)),
                                       **kw).items()}
    for mine, theirs, sign in (("fs", "delta", 1.0), ("T", "theta", -1.0), ("r", "rho", 1.0),
                               ("sigma", "vega", 1.0)):
        assert np.array_equal(a[mine], sign * g[theirs]), mine


@pytest.mark.gpu
@pytest.mark.parametrize("broadcast", [False, True])
def test_binary32_domain_edges(broadcast):
    """The binary32 solver on both sides of the edges that send a quote to its
    general path: beta around 2^-100, 1 - beta/b_max around 2^-20 (s ~ 9.5),
    maturities around 2^-100, r T around 80, F and K one ulp apart, F and K
    far from 1; with arrays and with broadcast r and q.  The binary32
    contract, as test_gpu_f32 has it."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_27210_amd as fv
    from test_gpu_f32 import compare_f32
    f32 = np.float32
    rows = []  # F, K, T, sigma (r = 0)
    for h in np.linspace(10.8, 11.6, 17):
        rows.append((100.0, 100.0 * np.exp(0.25 * h), 1.0, 0.25))
    for s in np.linspace(8.5, 10.5, 17):
        rows += [(100.0, 130.0, 1.0, s), (100.0, 70.0, 1.0, s)]
    for T in (2.0 ** -101, 2.0 ** -100, 2.0 ** -99, 1e-12):
        rows.append((100.0, 100.0 * np.exp(0.5 * np.sqrt(T)), T, 0.5))
    for K in (f32(100.0), np.nextafter(f32(100.0), f32(200.0)), np.nextafter(f32(100.0), f32(0.0))):
        rows += [(100.0, float(K), 0.5, sg) for sg in (0.01, 0.3, 2.0)]
    for e in (-99.0, -60.0, 60.0, 99.0, 101.0):
        rows.append((2.0 ** e, 1.2 * 2.0 ** e, 0.5, 0.4))
    F, K, T, sg = (np.array(c).astype(f32).astype(np.float64) for c in zip(*rows))
    r = np.zeros(len(F))
    if not broadcast:  # long exponents: the forward grows as the strike does
        rT = np.array([70.0, 79.9, 80.1, 85.0])
        F, T = np.concatenate([F, np.full(4, 1e-20)]), np.concatenate([T, np.full(4, 50.0)])
        r = np.concatenate([r, (rT / 50.0).astype(f32).astype(np.float64)])
        K = np.concatenate([K, (1e-20 * np.exp(r[-4:] * 50.0)).astype(f32).astype(np.float64)])
        sg = np.concatenate([sg, np.full(4, f32(0.3), dtype=np.float64)])
    n = len(F)
    flag = np.where(K >= F * np.exp(r * T), 1, -1).astype(np.int8)
    P = oracle.price("bs", F, K, T, r, np.zeros(n), sg, flag).astype(f32).astype(np.float64)
    keep = P >= np.finfo(f32).tiny
    F, K, T, r, P, flag = (a[keep] for a in (F, K, T, r, P, flag))
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=f32)).to("cuda")
    sig, st = fv.implied_vol_f32("bs", d(P), d(F), d(K), d(T), 0.0 if broadcast else d(r),
                                 flag=torch.from_numpy(flag).to("cuda"))
    ok, worst = compare_f32("bs", [P, F, K, T, r, np.zeros(len(F))], flag,
                            sig.cpu().numpy().astype(np.float64), st.cpu().numpy())
    print("binary32 edges: %d of %d solved, max err/tol %.3g" % (ok, len(F), worst))
    assert ok > 0.7 * len(F)


@pytest.mark.gpu
@pytest.mark.parametrize("solver", ["lbr", "halley"])
@pytest.mark.parametrize("side", [-1, 0, 77])
def test_chains_at_the_slice_rule(solver, side):
    """The ragged kernel takes one 64-quote slice per wave below 160 waves per
    compute unit and two from there: on both sides, quote by quote the flat
    solve of the same inputs (each within 1e-12 of the root)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_27210_amd as fv
    n = 64 * 160 * torch.cuda.get_device_properties(0).multi_processor_count + side
    rng = np.random.default_rng(n)
    cuts = np.unique(rng.integers(1, n, 4000))
    mqo = np.r_[0, cuts, n]
    nm = mqo.size - 1
    cmo = np.r_[0, np.unique(rng.integers(1, nm, 300)), nm]
    mat = torch.from_numpy(np.repeat(np.arange(nm), np.diff(mqo))).cuda()
    chain = torch.from_numpy(np.repeat(np.arange(cmo.size - 1), np.diff(cmo))).cuda()[mat]
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    F, r = d(rng.uniform(50, 150, cmo.size - 1)), d(rng.uniform(0, 0.05, cmo.size - 1))
    T = d(rng.uniform(0.05, 2.0, nm))
    sig = d(rng.uniform(0.1, 0.6, n))
    K = F[chain] * torch.exp(d(rng.uniform(-2, 2, n)) * sig * T[mat].sqrt())
    flag = torch.where(K < F[chain], -1, 1).to(torch.int8)
    fs, Tq, rq = F[chain].contiguous(), T[mat].contiguous(), r[chain].contiguous()
    P = fv.price("black76", fs, K, Tq, rq, sig, flag=flag)
    P[::1013] = -1.0
    want, want_st = fv.implied_vol("black76", P, fs, K, Tq, rq, flag=flag, solver=solver)
    got, got_st = fv.implied_vol_chains(d(cmo), d(mqo), F, r, T, P, K, flag, solver=solver)
    assert torch.equal(got_st, want_st)
    ok = want_st == 0
    assert ok.sum() > 0.99 * n
    tol = 2e-12 if solver == "lbr" else 2e-8
    assert ((got - want).abs()[ok] <= tol * want[ok]).all()
    assert got[~ok].isnan().all()
