"""Differentiable fault-tolerant FFT layer.

``fft(x)`` is the forward DFT of each row of a complex CUDA tensor,
y_j = sum_n x_n w_N^{jn} (TurboFFT Section II), computed by the library's
HIP kernels with the two-sided checksum.  Its backward pass applies the
adjoint of that linear map, F^H = conj(W)^T, which is the unscaled inverse DFT:
for a real loss, PyTorch's complex gradient (d/dRe + i d/dIm) of x is
F^H applied to the gradient of y.  The backward transform runs through the
same kernels with its own two-sided checksum (a plan created with the
unscaled-inverse flag), so a fault in either direction is detected and
corrected.
"""
from __future__ import annotations

import threading

import torch

from . import Plan

# shape -> {stream handle: (forward plan, adjoint plan)}.  A plan must not run on
# two streams at once (it owns its workspace, tickets and report), so every
# stream has its own.
_PLANS: dict = {}
_LAST: dict = {}  # shape -> {"forward" | "backward": the plan that last executed}
_LOCK = threading.Lock()  # the backward passes run on autograd's threads


def _key(n: int, batch: int, dtype, device) -> tuple:
    return (n, batch, str(dtype), str(device))


def _plans(n: int, batch: int, dtype, device, stream=None) -> tuple[Plan, Plan]:
    st = (stream if stream is not None else torch.cuda.current_stream(device)).cuda_stream
    with _LOCK:
        pairs = _PLANS.setdefault(_key(n, batch, dtype, device), {})
        if st not in pairs:
            with torch.cuda.device(device):
                if pairs and torch.cuda.is_current_stream_capturing():
                    # nothing can be allocated while a graph is captured: the
                    # graph takes over the pair of the warm-up, and that stream
                    # gets a new one when it next needs it
                    pairs[st] = pairs.pop(next(reversed(pairs)))
                else:
                    pairs[st] = (Plan(n, batch, dtype), Plan(n, batch, dtype, inverse_unscaled=True))
        return pairs[st]


def clear_plan_cache() -> None:
    with _LOCK:
        for pairs in _PLANS.values():
            for fwd, adj in pairs.values():
                fwd.close()
                adj.close()
        _PLANS.clear()
        _LAST.clear()


class UncorrectableError(RuntimeError):
    """A flagged checksum group of the layer's transform was not corrected."""


def _verify(plan: Plan, what: str) -> None:
    counts, _ = plan.report()
    if counts["uncorrectable"] or counts["dropped"]:
        raise UncorrectableError(f"{what}: {counts}")


class _FFTFunction(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, ft_mode, check):
        n = x.shape[-1]
        batch = x.numel() // n
        st = torch.cuda.current_stream(x.device)
        fwd, _ = _plans(n, batch, x.dtype, x.device, st)
        ctx.ft_mode = ft_mode
        ctx.check = check
        xc = x.contiguous()
        y = fwd.forward(xc, ft_mode=ft_mode, stream=st).view(x.shape)
        _LAST.setdefault(_key(n, batch, x.dtype, x.device), {})["forward"] = fwd
        if check and ft_mode == "correct":
            _verify(fwd, "forward transform")
        return y

    @staticmethod
    def backward(ctx, gy):
        n = gy.shape[-1]
        st = torch.cuda.current_stream(gy.device)
        batch = gy.numel() // n
        _, adj = _plans(n, batch, gy.dtype, gy.device, st)
        gx = adj.inverse(gy.contiguous(), ft_mode=ctx.ft_mode, stream=st)
        _LAST.setdefault(_key(n, batch, gy.dtype, gy.device), {})["backward"] = adj
        if ctx.check and ctx.ft_mode == "correct":
            _verify(adj, "backward transform")
        return gx.view(gy.shape), None, None


def fft(x: torch.Tensor, ft_mode: str = "correct", check: bool = False) -> torch.Tensor:
    """Forward DFT along the last axis of a complex64/complex128 CUDA tensor,
    differentiable, fault tolerant in both directions.

    The outcome of the checks is in the plans' reports, which the layer does
    not read by default (reading one waits for the transform's stream): call
    ``last_reports()`` to see detected, corrected and uncorrectable groups.
    With ``check=True`` (CORRECT mode) every forward and backward transform
    reads its report and raises ``UncorrectableError`` when a flagged group
    could not be corrected or a record was dropped."""
    if not x.is_complex():
        raise TypeError("fft expects a complex tensor")
    return _FFTFunction.apply(x, ft_mode, check)


def last_reports():
    """Reports of the most recent forward and backward executions of each shape
    (length, batch, dtype, device)."""
    with _LOCK:
        last = {}
        for key, pairs in _PLANS.items():
            for fwd, adj in pairs.values():
                last[key] = {"forward": fwd, "backward": adj, **_LAST.get(key, {})}
    return {key: {way: plan.report() for way, plan in ways.items()} for key, ways in last.items()}
