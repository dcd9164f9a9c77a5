"""Batches of more than 2^32 quotes, which no single launch of a quote per
thread covers: every entry point fills its outputs to the end.  The fields are
broadcast where they can be, so that a call needs little more than its output
(35 GB in binary64)."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N_LARGE = (1 << 32) + 65
FLAT = ["price", "iv_lbr", "iv_halley", "greeks", "price_backward", "iv_f32", "lbr_trace", "halley_trace",
        "normalised_black"]


@pytest.fixture(autouse=True)
def room():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.get_device_properties(0).total_memory < 200e9:
        pytest.skip("needs a card of 200 GB")
    yield
    torch.cuda.empty_cache()


def _full(out, n, value):
    """Every entry is the value (in pieces: a comparison of all of them at once
    would take as much memory again)."""
    return all(bool((out[a:min(n, a + (1 << 28))] == value).all()) for a in range(0, n, 1 << 28))


@pytest.mark.parametrize("call", FLAT)
def test_flat(call):
    from paper_2604_27210_amd import _native as N
    lib = N.load()
    p = ctypes.c_void_p
    f32 = call == "iv_f32"
    dt = torch.float32 if f32 else torch.int32 if call.endswith("trace") else torch.float64
    stream = p(torch.cuda.current_stream().cuda_stream)

    def run(n, out):
        out.fill_(-7)
        Arg, Quotes = (N.FvArgF32, N.FvQuotesF32) if f32 else (N.FvArg, N.FvQuotes)
        f = lambda v: Arg(None, v)
        q = Quotes(n, f(4.9), f(100.0), f(110.0), f(0.5), f(0.01), f(0.0), None, 1)
        ref, o = ctypes.byref(q), p(out.data_ptr())
        if call == "price":
            rc = lib.fv_price(1, ref, f(0.3), o, stream)
        elif call in ("iv_lbr", "iv_halley"):
            rc = lib.fv_implied_vol(1, 0 if call == "iv_lbr" else 1, ref, o, None, None, stream)
        elif call == "greeks":
            rc = lib.fv_greeks(1, ref, f(0.3), None, None, o, None, None, stream)
        elif call == "price_backward":  # the upstream gradient is the output before: -7 each
            rc = lib.fv_price_backward(1, ref, f(0.3), o, None, None, None, None, None, o, stream)
        elif call == "iv_f32":
            rc = lib.fv_implied_vol_f32(1, ref, o, None, stream)
        elif call == "lbr_trace":
            rc = lib.fv_lbr_trace(1, ref, o, stream)
        elif call == "halley_trace":
            rc = lib.fv_halley_trace(1, ref, o, stream)
        else:
            src = torch.full((n,), 0.4, dtype=dt, device="cuda")  # b(0.4, 0.4)
            rc = lib.fv_normalised_black(n, p(src.data_ptr()), p(src.data_ptr()), None, o, stream)
        N.check(rc, call)
        torch.cuda.synchronize()
        return out

    small = run(64, torch.empty(64, dtype=dt, device="cuda"))
    value = small[0].item()
    assert bool((small == value).all()) and value != -7
    out = run(N_LARGE, torch.empty(N_LARGE, dtype=dt, device="cuda"))
    assert _full(out, N_LARGE, value)


@pytest.mark.parametrize("solver", ["lbr", "halley"])
def test_ragged(solver):
    """Two 64-quote slices a wave: the limit is at 2^33 quotes.  Three chains of
    three maturities each, the last of one, 2^31 quotes and more between starts;
    price and strike are one array (a call worth 100 on a forward of 150)."""
    import paper_2604_27210_amd as fv
    n = (1 << 33) + 130
    quotes = torch.full((n,), 100.0, dtype=torch.float64, device="cuda")
    flag = torch.ones(n, dtype=torch.int8, device="cuda")
    mqo = torch.tensor([0, 1, 2_500_000_000, 5_000_000_001, 5_000_000_100, 8_000_000_000, (1 << 33) + 1, n],
                       dtype=torch.int64)
    cmo = torch.tensor([0, 3, 6, 7], dtype=torch.int64)
    F, r = [150.0, 160.0, 170.0], [0.0, 0.01, 0.02]
    T = [0.5, 1.0, 1.5, 2.0, 2.5, 3.0, 3.5]
    d = lambda v: torch.tensor(v, dtype=torch.float64, device="cuda")
    sigma = fv.implied_vol_chains(cmo.cuda(), mqo.cuda(), d(F), d(r), d(T), quotes, quotes, flag,
                                  solver=solver, with_status=False)
    torch.cuda.synchronize()
    for m in range(7):
        chain = int(torch.searchsorted(cmo, m, right=True)) - 1
        want = fv.implied_vol("black76", quotes[:1], F[chain], quotes[:1], T[m], r[chain], solver=solver,
                              with_status=False).item()
        lo, hi = int(mqo[m]), int(mqo[m + 1])
        piece = sigma[lo:hi]
        assert abs(piece[0].item() - want) <= (2e-12 if solver == "lbr" else 2e-8) * want
        assert _full(piece, hi - lo, piece[0].item()), m
