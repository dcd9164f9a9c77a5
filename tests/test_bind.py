"""The compiled tensor marshalling: what it refuses, with which exception
(no GPU needed), and that every form of argument it accepts reaches the
library as the same call made through ctypes structures."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2604_27210_amd as fv
from paper_2604_27210_amd import _native as N
from paper_2604_27210_amd import api

V = torch.ones(4, dtype=torch.float64)
F32 = torch.ones(4, dtype=torch.float32)
REFUSED = {
    "no tensor": (ValueError, "at least one", lambda: fv.implied_vol("bs", 1.0, 2.0, 3.0, 4.0, 0.0)),
    "host tensor": (ValueError, "must be on the GPU", lambda: fv.implied_vol("bs", V, V, V, V, V)),
    "host f32": (ValueError, "must be on the GPU", lambda: fv.implied_vol_f32("bs", F32, 1, 1, 1, 0)),
    "host chains": (ValueError, "chain_mat_off must be on the GPU",
                    lambda: fv.implied_vol_chains(*[V] * 8)),
    "not a tensor": (TypeError, "chain_mat_off must be a tensor",
                     lambda: fv.implied_vol_chains(*[1.0] * 8)),
    "matrix": (ValueError, "fs must be 1-D", lambda: fv.price("bs", V.reshape(2, 2), V, 1, 0, 1)),
    "not a number": (TypeError, None, lambda: fv.price("bs", [1.0], V, 1.0, 0.0, 1.0)),
    "no number": (ValueError, None, lambda: fv.price("bs", "x", V, 1.0, 0.0, 1.0)),
    "model": (KeyError, None, lambda: fv.greeks("heston", V, V, 1.0, 0.0, 1.0)),
    "solver": (KeyError, None, lambda: fv.implied_vol("bs", V, V, V, V, V, solver="bisect")),
}


@pytest.mark.parametrize("what", list(REFUSED))
def test_refusals(what):
    kind, text, call = REFUSED[what]
    with pytest.raises(kind, match=text):
        call()


def _quotes(n, cls, arg, price, fs, K, T, r, q, flag):
    """The call's structure through ctypes."""
    def one(v):
        if v is None:
            return arg(None, 0.0)
        if isinstance(v, torch.Tensor) and v.dim() > 0:
            return arg(v.data_ptr(), 0.0)
        return arg(None, float(v))
    if isinstance(flag, torch.Tensor):
        fp, f = flag.data_ptr(), 1
    else:
        fp, f = None, (1 if str(flag).lower()[0] == "c" else -1) if isinstance(flag, str) else int(flag)
    return cls(n, *[one(v) for v in (price, fs, K, T, r, q)], fp, f), one


FORMS = ["arrays", "scalars", "zero-dim", "no q", "put", "minus one"]


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 65, 1001])
@pytest.mark.parametrize("form", FORMS)
def test_same_call_as_ctypes(form, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lib, dev = N.load(), "cuda"
    g = torch.Generator().manual_seed(n)
    rnd = lambda lo, hi: (torch.rand(n, generator=g, dtype=torch.float64) * (hi - lo) + lo).to(dev)
    fs, K, T, r, q, sig = rnd(90, 110), rnd(80, 120), rnd(0.1, 2), rnd(0, 0.05), rnd(0, 0.03), rnd(0.1, 0.6)
    flag = torch.where(rnd(0, 1) < 0.5, 1, -1).to(torch.int8)
    if form == "scalars":
        fs, T, r, q, flag = 100, 0.5, np.float64(0.01), 0.02, "c"
    elif form == "zero-dim":
        T, r, flag = torch.tensor(0.5), torch.tensor(0.01, dtype=torch.float64, device=dev), 1.0
    elif form == "no q":
        q = None
    elif form == "put":
        flag = "Put"
    elif form == "minus one":
        flag = -1
    empty = lambda *s, dt=torch.float64: torch.empty(s, dtype=dt, device=dev)
    p = ctypes.c_void_p
    stream = torch.cuda.Stream()
    for st in (None, stream):
        raw = p((st or torch.cuda.current_stream()).cuda_stream)
        torch.cuda.synchronize()
        ref = lambda t: p(t.data_ptr())
        qs, one = _quotes(n, N.FvQuotes, N.FvArg, None, fs, K, T, r, q, flag)
        P = empty(n)
        N.check(lib.fv_price(2, ctypes.byref(qs), one(sig), ref(P), raw), "price")
        out = empty(n)
        got = [fv.price("bsm", fs, K, T, r, sig, flag=flag, q=q, stream=st)]
        assert fv.price("bsm", fs, K, T, r, sig, flag=flag, q=q, out=out, stream=st) is out
        want, rows = [P], lambda k: [empty(n) for _ in range(k)]
        got.append(out)
        want.append(P)
        G = rows(5)
        N.check(lib.fv_greeks(2, ctypes.byref(qs), one(sig), *map(ref, G), raw), "greeks")
        d = fv.greeks("bsm", fs, K, T, r, sig, flag=flag, q=q, stream=st)
        assert list(d) == list(api.GREEK_NAMES)
        got += list(d.values())
        want += G
        gs = rows(6)
        N.check(lib.fv_price_backward(2, ctypes.byref(qs), one(sig), ref(P), *map(ref, gs), raw), "pb")
        d = fv.price_backward("bsm", fs, K, T, r, sig, P, flag=flag, q=q, stream=st)
        assert list(d) == ["fs", "K", "T", "r", "q", "sigma"]
        got += list(d.values())
        want += gs
        qs, _ = _quotes(n, N.FvQuotes, N.FvArg, P, fs, K, T, r, q, flag)
        gs = rows(6)
        N.check(lib.fv_implied_vol_backward(2, ctypes.byref(qs), ref(sig), ref(P), *map(ref, gs), raw), "b")
        d = fv.implied_vol_backward("bsm", P, fs, K, T, r, sig, P, flag=flag, q=q, stream=st)
        assert list(d) == ["price", "fs", "K", "T", "r", "q"]
        got += list(d.values())
        want += gs
        for name, solver in (("lbr", 0), ("halley", 1)):
            s, t8, G = empty(n), empty(n, dt=torch.uint8), rows(5)
            arr = (p * 5)(*[x.data_ptr() for x in G])
            N.check(lib.fv_implied_vol(2, solver, ctypes.byref(qs), ref(s), ref(t8), arr, raw), "iv")
            a, b, c = fv.implied_vol("bsm", P, fs, K, T, r, flag=flag, q=q, solver=name, greeks=True,
                                     stream=st)
            e, h = fv.implied_vol("bsm", P, fs, K, T, r, flag=flag, q=q, solver=solver,
                                  with_status=False, greeks=True, stream=st)
            N.check(lib.fv_implied_vol(2, solver, ctypes.byref(qs), ref(s), ref(t8), None, raw), "iv")
            f = fv.implied_vol("bsm", P, fs, K, T, r, flag=flag, q=q, solver=name, with_status=False,
                               stream=st)
            got += [f, b, *c.values(), *h.values()]
            want += [s, t8, *G, *G]
            assert a.shape == e.shape == f.shape
            trace = empty(n, dt=torch.int32)
            fn = lib.fv_halley_trace if solver else lib.fv_lbr_trace
            N.check(fn(2, ctypes.byref(qs), ref(trace), raw), "trace")
            got.append((api.halley_trace if solver else api.lbr_trace)(
                "bsm", P, fs, K, T, r, flag=flag, q=q, stream=st))
            want.append(trace)
        to32 = lambda v: v.float() if isinstance(v, torch.Tensor) and v.dim() else v
        a32 = [to32(v) for v in (P, fs, K, T, r, q)]
        torch.cuda.synchronize()
        qs, _ = _quotes(n, N.FvQuotesF32, N.FvArgF32, *a32, flag)
        s, t8 = empty(n, dt=torch.float32), empty(n, dt=torch.uint8)
        N.check(lib.fv_implied_vol_f32(2, ctypes.byref(qs), ref(s), ref(t8), raw), "f32")
        got += fv.implied_vol_f32("bsm", *a32[:5], flag=flag, q=a32[5], stream=st)
        want += [s, t8]
        torch.cuda.synchronize()
        for i, (x, y) in enumerate(zip(got, want)):
            assert x.dtype == y.dtype and x.shape == y.shape, i
            assert torch.equal(x.nan_to_num(-7.0) if x.is_floating_point() else x,
                               y.nan_to_num(-7.0) if y.is_floating_point() else y), i


@pytest.mark.gpu
def test_gpu_refusals():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    v, w = torch.ones(4, dtype=torch.float64, device="cuda"), torch.ones(6, dtype=torch.float64, device="cuda")
    i8 = torch.ones(4, dtype=torch.int8, device="cuda")
    for kind, text, call in [
            (TypeError, "K must be torch.float64 .got torch.float32.",
             lambda: fv.implied_vol("bs", v, v, v.float(), v, v)),
            (ValueError, "K must be contiguous", lambda: fv.implied_vol("bs", v, v, w[::2], v, v)),
            (ValueError, "length mismatch: T has 6, expected 4", lambda: fv.greeks("bs", v, v, w, v, v)),
            (TypeError, "flag tensor must be int8", lambda: fv.price("bs", v, v, v, v, v, flag=v)),
            (ValueError, "flag length", lambda: fv.price("bs", w, w, w, w, w, flag=i8)),
            (TypeError, "flag must be", lambda: fv.price("bs", v, v, v, v, v, flag=i8[0])),
            (TypeError, "grad_sigma must be a tensor",
             lambda: fv.implied_vol_backward("bs", v, v, v, v, v, v, 1.0)),
            (TypeError, "sigma must be a tensor",
             lambda: fv.implied_vol_backward("bs", v, v, v, v, v, 0.2, v)),
            (TypeError, "torch.float32", lambda: fv.implied_vol_f32("bs", v, v, v, v, v)),
            (N.FastvolError, "fv_price failed .-1.: model out of range",
             lambda: fv.price(7, v, v, v, v, v))]:
        with pytest.raises(kind, match=text):
            call()
    e = torch.empty(0, dtype=torch.float64, device="cuda")
    s, st = fv.implied_vol("bs", e, e, e, e, e)
    assert s.shape == st.shape == (0,)


@pytest.mark.gpu
def test_gpu_buffers_hold_every_quote():
    """A buffer that the kernels index by quote and that is shorter than the
    batch (or 0-dim) is refused before any launch; a longer one is read and
    written as far as the batch goes."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    v = torch.full((4,), 2.0, dtype=torch.float64, device="cuda")
    w = torch.full((6,), 2.0, dtype=torch.float64, device="cuda")
    for short in (v[:3], v[0], v[:0]):
        m = short.numel()
        for text, call in [
                ("grad_sigma has %d, expected 4" % m,
                 lambda: fv.implied_vol_backward("bs", v, v, v, v, v, v, short)),
                ("sigma has %d, expected 4" % m,
                 lambda: fv.implied_vol_backward("bs", v, v, v, v, v, short, v)),
                ("grad_price has %d, expected 4" % m,
                 lambda: fv.price_backward("bs", v, v, v, v, v, short)),
                ("out has %d, expected 4" % m, lambda: fv.price("bs", v, v, v, v, v, out=short))]:
            with pytest.raises(ValueError, match="length mismatch: " + text):
                call()
    P = fv.price("bs", v, v, v, v, v)
    out = torch.full((6,), -1.0, dtype=torch.float64, device="cuda")
    assert fv.price("bs", v, v, v, v, v, out=out) is out
    assert torch.equal(out[:4], P) and (out[4:] == -1.0).all()
    a = fv.implied_vol_backward("bs", P, v, v, v, v, v, v)
    b = fv.implied_vol_backward("bs", P, v, v, v, v, v, w)
    assert all(torch.equal(a[k], b[k]) for k in a)
    one = fv.price("bs", v[:1], v[:1], v[:1], v[:1], v[:1])
    got = fv.implied_vol_backward("bs", one, v[:1], v[:1], v[:1], v[:1], v[0], v[1])
    assert all(torch.equal(got[k], a[k][:1]) for k in a)
