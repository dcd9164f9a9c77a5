"""The calibration step at the edges of its lane sums and its update: waves
inside one maturity and across many, one to sixteen runs per maturity, empty
maturities, more maturities than one workgroup updates, parameters on both
sides of each transform's branches, against the oracle's gradient and loss."""
import numpy as np
import pytest

import oracle
from oracle import svi

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LAYOUTS = {"one": [1], "w-1": [63], "w": [64], "w+1": [65], "two": [128], "eight runs": [512],
           "nine": [513], "sixteen": [1000], "short": [1] * 70, "two blocks": [3] * 129,
           "empty ends": [0, 64, 0, 0, 63, 1, 0], "mixed": [130, 5, 0, 700, 64, 2, 200]}


def test_quotes_without_logarithm_are_skipped():
    """A strike of 0, below 0 or subnormal has no ln(K/F) (the forward's
    quotient overflows): such a quote adds nothing to gradient or loss."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27210_amd.calibrate import SviCalibrator
    K = np.array([90.0, 100.0, 110.0, 0.0, -100.0, -0.0, np.nan, 1e-310])
    target = np.full(8, 0.3)
    raw = np.array([[0.04, -2.0, 0.1, 0.0, -1.0]])
    d = lambda a, t=torch.float64: torch.as_tensor(np.ascontiguousarray(a)).to("cuda", t)
    cal = SviCalibrator(d([0, 1], torch.int64), d([0, 8], torch.int64), d([100.0]), d([0.0]),
                        d([1.0]), d(K), d(np.ones(8), torch.int8), d(target), raw)
    cal.step()
    torch.cuda.synchronize()
    k = np.log(K[:3] / 100.0)
    L, G = svi.loss_and_grad(raw, k, np.zeros(3, dtype=int), np.ones(1), target[:3])
    # the mean is over all eight quotes; every term is off by a few ulps
    assert abs(cal.loss[0].item() - L * 3 / 8) <= 2.0 ** -45 * L
    g = cal.grad.cpu().numpy()
    assert np.all(np.abs(g - G[0] * 3 / 8) <= 2.0 ** -45 * np.abs(G).max())


@pytest.mark.parametrize("max_steps", [4, 0])
@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_step_matches_oracle(layout, max_steps):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27210_amd.calibrate import SviCalibrator
    size = np.array(LAYOUTS[layout])
    nm, n = size.size, int(size.sum())
    rng = np.random.default_rng(nm * 1000 + n)
    mat = np.repeat(np.arange(nm), size)
    T = rng.uniform(0.05, 3.0, nm)
    # softplus on both sides of 0 and of its log's halving at e^-0.88, tanh on
    # both sides of its series' end at 0.17
    raw = np.stack([rng.uniform(0.01, 0.1, nm), rng.uniform(-3.0, 1.0, nm),
                    rng.choice([-1.5, -0.2, -0.16, -1e-9, 1e-9, 0.16, 0.2, 0.9], nm),
                    rng.uniform(-0.1, 0.1, nm), rng.uniform(-3.0, 1.5, nm)], 1)
    F = 100.0
    k = rng.uniform(-1.0, 1.0, n) * np.sqrt(T[mat]) * 0.3
    K = F * np.exp(k)
    k = np.log(K / F)
    target = rng.uniform(0.1, 0.5, n)
    target[rng.random(n) < 0.05] = np.nan
    d = lambda a, t=torch.float64: torch.as_tensor(np.ascontiguousarray(a)).to("cuda", t)
    cal = SviCalibrator(d([0, nm], torch.int64), d(np.r_[0, np.cumsum(size)], torch.int64),
                        d([F]), d([0.02]), d(T), d(K), d(np.where(rng.random(n) < 0.5, 1, -1),
                                                         torch.int8),
                        d(target), raw, max_steps=max_steps)
    cal.step()
    torch.cuda.synchronize()
    L, G = svi.loss_and_grad(raw, k, mat, T, target)
    # Every term of a sum is off by a few ulps of sigma in (sigma - target),
    # of the weights' factors and of the parameters; 256 u bounds their sum.
    a, b, rho, m, s = svi.natural(raw)
    sig = svi.svi_vols(raw, k, mat, T)
    ok = np.isfinite(target)
    dk = k - m[mat]
    rt = np.sqrt(dk * dk + s[mat] ** 2)
    size_of = np.where(ok, (sig + np.abs(np.nan_to_num(target))) / (sig * T[mat] * n), 0.0)
    dw = np.stack([np.ones(n), np.abs(rho[mat] * dk) + rt, b[mat] * (np.abs(dk) + 1e-3),
                   b[mat] * (np.abs(rho[mat]) + np.abs(dk) / rt), b[mat] * s[mat] / rt * s[mat]], 1)
    tol = np.stack([np.bincount(mat, size_of * dw[:, j], minlength=nm) for j in range(5)], 1)
    tol = 2.0 ** -45 * (tol + np.abs(G))
    g = cal.grad.cpu().numpy().reshape(-1, 5)
    assert np.all(np.abs(g - G) <= tol), np.max(np.abs(g - G) / np.where(tol > 0, tol, 1))
    assert np.all(g[size == 0] == 0.0)
    th = raw - 1e-2 * np.sign(g) * (np.abs(g) / (np.abs(g) + 1e-8))  # Adam's first step
    np.testing.assert_allclose(cal.theta.cpu().numpy().reshape(-1, 5), th, rtol=0, atol=1e-9)
    if max_steps:
        e = np.where(ok, sig - target, 0.0)
        tol_L = 2.0 ** -45 * (L + np.sum(np.abs(e) * (sig + 1.0)) / n)
        assert abs(cal.loss[0].item() - L) <= tol_L
