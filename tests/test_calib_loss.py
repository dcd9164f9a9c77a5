"""The loss of a calibration step over many quotes against an extended-precision
sum of the squared errors."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_loss_to_the_last_place():
    """A sum of 200,000 squares in a tree of partial sums, times 1/N: 1/N, the
    product and the last levels of the tree round by up to u/2 each (0.29 u
    rms), what lies below averages out and so do the errors of the terms (10 u
    each, 200,000 of them).  The mean of sixty stays below u."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27210_amd.calibrate import SviCalibrator
    L = np.longdouble
    d = lambda a, t=torch.float64: torch.as_tensor(np.ascontiguousarray(a)).to("cuda", t)
    nm, per = 1000, 200
    n = nm * per
    errors = []
    for seed in range(60):
        rng = np.random.default_rng(seed)
        raw = np.stack([rng.uniform(0.02, 0.05, nm), rng.uniform(-2.5, -1.0, nm), rng.uniform(-0.7, 0.0, nm),
                        rng.uniform(-0.1, 0.1, nm), rng.uniform(-2.5, -1.0, nm)], 1)
        T = rng.uniform(0.1, 3.0, nm)
        mat = np.repeat(np.arange(nm), per)
        K = 100.0 * np.exp(rng.uniform(-1.0, 1.0, n) * np.sqrt(T[mat]))
        target = rng.uniform(0.1, 0.5, n)
        a, b, rho, mu, s = (v[mat] for v in raw.astype(L).T)
        b, rho, s = np.log1p(np.exp(b)), np.tanh(rho), np.log1p(np.exp(s))
        dk = np.log(K.astype(L) / L(100.0)) - mu
        e = np.sqrt((a + b * (rho * dk + np.sqrt(dk * dk + s * s))) / T[mat].astype(L)) - target.astype(L)
        want = np.sum(e * e) / n
        cal = SviCalibrator(d([0, nm], torch.int64), d(np.arange(nm + 1) * per, torch.int64), d([100.0]),
                            d([0.01]), d(T), d(K), d(np.ones(n), torch.int8), d(target), raw)
        cal.step()
        torch.cuda.synchronize()
        errors.append(float(abs(L(cal.loss[0].item()) - want) / want))
    print("loss: mean error %.3g, max %.3g" % (np.mean(errors), np.max(errors)))
    assert np.mean(errors) <= 2.0 ** -53
