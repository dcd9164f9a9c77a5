"""The wave's location of its quotes in the CSR offsets, at the counts where
its 64-ary search takes another level or its window of starts another load:
every quote of the ragged kernel has its own maturity's T and chain's F and r,
so a wrong one gives another volatility than the flat solve."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# maturities, quotes per maturity (0: empty), maturities per chain
LAYOUTS = {
    "1 of 1": (1, [1], [1]), "1 of 300": (1, [300], [1]), "63": (63, [1, 5], [1]),
    "64": (64, [3], [2, 0, 1]), "65": (65, [3], [1]), "66": (66, [2, 70], [66]),
    "4096 short": (4096, [1], [1, 2, 3]), "4097": (4097, [1, 2], [64, 1]),
    "4160": (4160, [2], [65]), "4161": (4161, [2, 1], [1]),
    "empty runs": (5000, [0] * 70 + [129], [3, 0]), "all but the last empty": (700, [0], [7]),
    "262145": (262145, [1], [1, 0, 4]),
}


@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_ragged_equals_flat(layout):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_27210_amd as fv
    nm, sizes, per_chain = LAYOUTS[layout]
    size = np.resize(sizes, nm)
    if size.sum() == 0:
        size[-1] = 200
    mqo = np.r_[0, np.cumsum(size)]
    cuts = np.cumsum(np.resize(per_chain, nm * len(per_chain)))
    cmo = np.r_[0, cuts[cuts < nm], nm]
    n, nc = int(mqo[-1]), cmo.size - 1
    rng = np.random.default_rng(nm)
    mat = np.repeat(np.arange(nm), size)
    chain = np.repeat(np.arange(nc), np.diff(cmo))[mat]
    F, r = rng.uniform(50, 150, nc), rng.uniform(0, 0.05, nc)
    T, sig = rng.uniform(0.05, 2.0, nm), rng.uniform(0.1, 0.6, n)
    d = lambda a, t=torch.float64: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", t)
    K = F[chain] * np.exp(rng.uniform(-1.5, 1.5, n) * sig * np.sqrt(T[mat]))
    flag = d(np.where(K < F[chain], -1, 1), torch.int8)
    fs, K, Tq, rq = d(F[chain]), d(K), d(T[mat]), d(r[chain])
    P = fv.price("black76", fs, K, Tq, rq, d(sig), flag=flag)
    for solver, tol in (("lbr", 2e-12), ("halley", 2e-8)):  # each within half of it of the root
        want, want_st = fv.implied_vol("black76", P, fs, K, Tq, rq, flag=flag, solver=solver)
        got, st = fv.implied_vol_chains(d(cmo, torch.int64), d(mqo, torch.int64), d(F), d(r), d(T),
                                        P, K, flag, solver=solver)
        assert torch.equal(st, want_st) and (st == 0).all()
        assert ((got - want).abs() <= tol * want).all(), solver
