"""Python surface of the library: thin marshalling over the C ABI (tensors
through csrc/fv_bind.cpp, the rest through ctypes).

Every argument that is a per-quote field may be a Python float (broadcast to
all quotes) or a contiguous float64 tensor on the GPU.  Results are float64
tensors on the same device, produced on the current torch stream.  Nothing
here computes: a missing or unloadable library raises, there is no fallback.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional

import torch

from . import _native as N


def _model(model) -> int:
    if isinstance(model, str):
        return N.MODELS[model.lower()]
    return int(model)


def _solver(solver) -> int:
    if isinstance(solver, str):
        return N.SOLVERS[solver.lower()]
    return int(solver)


# the current stream's raw handle without building a Stream object (about
# 3 us per call saved on the small-batch path)
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


def _stream_ptr(stream=None, device: Optional[int] = None) -> int:
    """Raw hipStream_t of `stream`, or of torch's current stream on `device`
    (an ordinal; the current device when None)."""
    if stream is not None:
        return int(stream.cuda_stream)
    if _raw_stream is not None:
        return _raw_stream(torch.cuda.current_device() if device is None else device)
    return int(torch.cuda.current_stream(device).cuda_stream)


def _dev_tensor(t: torch.Tensor, name: str, dtype=torch.float64) -> torch.Tensor:
    if not isinstance(t, torch.Tensor):
        raise TypeError("%s must be a tensor" % name)
    if not t.is_cuda:
        raise ValueError("%s must be on the GPU (got %s)" % (name, t.device))
    if t.dtype != dtype:
        raise TypeError("%s must be %s (got %s)" % (name, dtype, t.dtype))
    if not t.is_contiguous():
        raise ValueError("%s must be contiguous" % name)
    return t


def _ptr(t: Optional[torch.Tensor]):
    return ctypes.c_void_p(t.data_ptr()) if t is not None else None


# options of an implied-volatility call (what it returns)
_STATUS, _GREEKS, _GREEK_BLOCK = 1, 2, 4


def _flat(fn, model, solver, price, fs, K, T, r, q, sigma, grad, flag, option, stream):
    """One launch over a flat batch (csrc/fv_bind.cpp): checks the fields
    (each a number, or a contiguous float64 GPU vector, all of one length),
    allocates the outputs and calls the library's function `fn`."""
    return N.bind().flat(fn, _model(model), solver, price, fs, K, T, r, q, sigma, grad, flag,
                         option, None if stream is None else int(stream.cuda_stream))


def price(model, fs, K, T, r, sigma, flag="c", q=None, out=None, stream=None) -> torch.Tensor:
    """Model price (Black-76: discounted, on forward fs; else spot fs)."""
    return _flat(N.FN_PRICE, model, 0, None, fs, K, T, r, q, sigma, None, flag, out, stream)


GREEK_NAMES = ("delta", "gamma", "vega", "theta", "rho")


def implied_vol(model, price, fs, K, T, r, flag="c", q=None, solver="lbr", greeks=False,
                with_status=True, stream=None):
    """Implied volatility.  Returns sigma, or (sigma, status) with
    ``with_status``; with ``greeks=True`` a dict of the five Greeks at the
    solved sigma is appended (rows of one [5, n] tensor)."""
    return _flat(N.FN_IV, model, _solver(solver), price, fs, K, T, r, q, None, None, flag,
                 (_STATUS if with_status else 0) | (_GREEKS if greeks else 0), stream)


def implied_vol_f32(model, price, fs, K, T, r, flag="c", q=None, with_status=True, stream=None):
    """Implied volatility in binary32 arithmetic (Halley path): per-quote
    fields are Python floats or contiguous float32 GPU tensors; returns a
    float32 sigma (and the uint8 status with ``with_status``)."""
    return N.bind().flat_f32(_model(model), price, fs, K, T, r, q, flag, 1 if with_status else 0,
                             None if stream is None else int(stream.cuda_stream))


def greeks(model, fs, K, T, r, sigma, flag="c", q=None, stream=None) -> dict:
    """delta, gamma, vega, theta (= -dP/dT), rho as raw per-unit derivatives."""
    return _flat(N.FN_GREEKS, model, 0, None, fs, K, T, r, q, sigma, None, flag, None, stream)


def implied_vol_backward(model, price, fs, K, T, r, sigma, grad_sigma, flag="c", q=None,
                         stream=None) -> dict:
    """dL/d(price, fs, K, T, r, q) from dL/dsigma (implicit-function adjoint)."""
    return _flat(N.FN_IV_BACKWARD, model, 0, price, fs, K, T, r, q, sigma, grad_sigma, flag, None,
                 stream)


def price_backward(model, fs, K, T, r, sigma, grad_price, flag="c", q=None, stream=None) -> dict:
    """dL/d(fs, K, T, r, q, sigma) from dL/dprice (adjoint of ``price``)."""
    return _flat(N.FN_PRICE_BACKWARD, model, 0, None, fs, K, T, r, q, sigma, grad_price, flag,
                 None, stream)


def implied_vol_chains(chain_mat_off, mat_quote_off, F, r, T, price, K, flag, solver="lbr",
                       with_status=True, stream=None):
    """Implied volatility of ragged Black-76 chains (CSR offsets, int64)."""
    return N.bind().chains(_solver(solver), chain_mat_off, mat_quote_off, F, r, T, price, K, flag,
                           1 if with_status else 0,
                           None if stream is None else int(stream.cuda_stream))


def normalised_black(x, s, flag=None, stream=None) -> torch.Tensor:
    _dev_tensor(x, "x")
    _dev_tensor(s, "s")
    if flag is not None:
        _dev_tensor(flag, "flag", torch.int8)
    if x.numel() != s.numel():
        raise ValueError("x and s lengths differ")
    out = torch.empty_like(x)
    N.check(N.load().fv_normalised_black(x.numel(), _ptr(x), _ptr(s), _ptr(flag), _ptr(out),
                                         ctypes.c_void_p(_stream_ptr(stream, out.get_device()))),
            "fv_normalised_black")
    return out


def lbr_trace(model, price, fs, K, T, r, flag="c", q=None, stream=None) -> torch.Tensor:
    """Per-quote path code of the LBR solver (see fv_lbr_trace)."""
    return _flat(N.FN_LBR_TRACE, model, 0, price, fs, K, T, r, q, None, None, flag, None, stream)


def halley_trace(model, price, fs, K, T, r, flag="c", q=None, stream=None) -> torch.Tensor:
    """Per-quote Halley step count and fallback bit (see fv_halley_trace)."""
    return _flat(N.FN_HALLEY_TRACE, model, 0, price, fs, K, T, r, q, None, None, flag, None, stream)


def set_halley_steps(steps: int) -> None:
    """Halley steps before the bisection fallback (fv_set_halley_steps)."""
    N.check(N.load().fv_set_halley_steps(int(steps)), "fv_set_halley_steps")


def get_halley_steps() -> int:
    return int(N.load().fv_get_halley_steps())


def set_launch(kernel, block: int, quotes_per_thread: int) -> None:
    k = N.KERNELS[kernel] if isinstance(kernel, str) else int(kernel)
    N.check(N.load().fv_set_launch(k, int(block), int(quotes_per_thread)), "fv_set_launch")


def get_launch(kernel):
    k = N.KERNELS[kernel] if isinstance(kernel, str) else int(kernel)
    b, q = ctypes.c_int(), ctypes.c_int()
    N.check(N.load().fv_get_launch(k, ctypes.byref(b), ctypes.byref(q)), "fv_get_launch")
    return b.value, q.value


def autotune(kernel, model="bsm", n_hint: int = 1 << 22, stream=None):
    """Time the workgroup sizes of one kernel family on `n_hint` synthetic
    quotes and keep the fastest for that model and size class; returns the
    shape a launch then has."""
    k = N.KERNELS[kernel] if isinstance(kernel, str) else int(kernel)
    N.check(N.load().fv_autotune(k, _model(model), int(n_hint),
                                 ctypes.c_void_p(_stream_ptr(stream))), "fv_autotune")
    return launch_shape(k, model, max(1, int(n_hint)))


# one batch size per size class of the tuning table (2^12 .. 2^24)
TUNING_SIZES = (1 << 12, 1 << 15, 1 << 17, 1 << 19, 1 << 21, 1 << 23, 1 << 24)


def autotune_all(kernels=None, models=("bsm",), sizes=TUNING_SIZES, stream=None) -> dict:
    """fv_autotune over kernel families x models x sizes; returns
    {(kernel, model, size): (block, quotes_per_thread)}."""
    kernels = kernels or [k for k in N.KERNELS]
    out = {}
    for kern in kernels:
        for model in (("black76",) if kern == "chains" else models):
            for n in sizes:
                out[(kern, model, n)] = autotune(kern, model, n, stream)
    return out


def launch_shape(kernel, model, n: int):
    """(block, quotes per thread) a launch of n quotes would use."""
    k = N.KERNELS[kernel] if isinstance(kernel, str) else int(kernel)
    b, q = ctypes.c_int(), ctypes.c_int()
    N.check(N.load().fv_launch_shape(k, _model(model), int(n), ctypes.byref(b), ctypes.byref(q)),
            "fv_launch_shape")
    return b.value, q.value


def save_tuning(path) -> None:
    N.check(N.load().fv_tuning_save(os.fsencode(path)), "fv_tuning_save")


def load_tuning(path) -> None:
    N.check(N.load().fv_tuning_load(os.fsencode(path)), "fv_tuning_load")


def reset_tuning() -> None:
    N.check(N.load().fv_tuning_reset(), "fv_tuning_reset")


def version() -> int:
    return int(N.load().fv_version())
