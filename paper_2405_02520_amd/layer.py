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

class _Shape:
    """The plans of one (length, batch, dtype, device).  A plan must not run on
    two streams at once (it owns its workspace, tickets and report), so every
    stream has a pair of its own."""

    def __init__(self, n, batch, dtype, device):
        self.args = (n, batch, dtype)
        self.device = device
        self.name = (n, batch, str(dtype), str(device))
        self.pairs: dict = {}  # stream handle -> (forward plan, adjoint plan)
        self.last = [None, None]  # the plans that last executed, forward and adjoint

    def pair(self, stream) -> tuple[Plan, Plan]:
        return self.pairs.get(stream.cuda_stream) or self._new_pair(stream.cuda_stream)

    def _new_pair(self, st) -> tuple[Plan, Plan]:
        with _LOCK, torch.cuda.device(self.device):
            if st not in self.pairs:
                if self.pairs and torch.cuda.is_current_stream_capturing():
                    # nothing can be allocated while a graph is captured: the
                    # graph takes over the pair of the warm-up, and that stream
                    # gets a new one when it next needs it
                    self.pairs[st] = self.pairs.pop(next(reversed(self.pairs)))
                else:
                    self.pairs[st] = (Plan(*self.args), Plan(*self.args, inverse_unscaled=True))
            return self.pairs[st]


_SHAPES: dict = {}
_LOCK = threading.Lock()  # the backward passes run on autograd's threads


def _shape(n: int, batch: int, dtype, device) -> _Shape:
    key = (n, batch, dtype, device)
    return _SHAPES.get(key) or _SHAPES.setdefault(key, _Shape(*key))


def _plans(n: int, batch: int, dtype, device) -> tuple[Plan, Plan]:
    return _shape(n, batch, dtype, device).pair(torch.cuda.current_stream(device))


def clear_plan_cache() -> None:
    with _LOCK:
        for shape in _SHAPES.values():
            for fwd, adj in shape.pairs.values():
                fwd.close()
                adj.close()
            shape.pairs.clear()
        _SHAPES.clear()


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
        shape = _shape(n, batch, x.dtype, x.device)
        fwd = shape.last[0] = shape.pair(st)[0]
        ctx.call = (shape, st, ft_mode, check)
        xc = x.contiguous()
        y = fwd.forward(xc, ft_mode=ft_mode, stream=st).view(x.shape)
        if check and ft_mode == "correct":
            _verify(fwd, "forward transform")
        return y

    @staticmethod
    def backward(ctx, gy):
        shape, st, ft_mode, check = ctx.call
        # (autograd runs it on the forward's stream; a stream object made on its
        # thread costs 15 us)
        if torch._C._cuda_getCurrentRawStream(shape.device.index) != st.cuda_stream:
            st = torch.cuda.current_stream(shape.device)
        adj = shape.last[1] = shape.pair(st)[1]
        gx = adj.inverse(gy.contiguous(), ft_mode=ft_mode, stream=st)
        if check and ft_mode == "correct":
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
        for shape in _SHAPES.values():
            for pair in shape.pairs.values():
                last[shape.name] = [ran or plan for ran, plan in zip(shape.last, pair)]
    return {name: {"forward": fwd.report(), "backward": adj.report()} for name, (fwd, adj) in last.items()}
