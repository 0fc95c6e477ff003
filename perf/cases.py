"""The workloads whose speed is tracked, as plain cases over the public entry points.

A case is a dict of plain values.  Three kinds:

* ``plan``: one batched transform, ``Plan.forward`` or ``Plan.inverse``, of
  ``batch`` signals of ``n`` points in ``mode`` (checksum off, detect or
  correct) with checksum groups of ``group`` signals (0: the default);
* ``layer``: the differentiable layer, forward and backward through autograd;
* ``ragged``: ``count`` signals of mixed lengths 2^kmin..2^kmax in one flat
  buffer, one graph replay, as one persistent kernel or as per-class launches.

Inputs are i.i.d. U[-1, 1) in the real and imaginary part, as in the benchmark.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2405_02520_amd as tf
from paper_2405_02520_amd import layer

_TORCH = {"c64": torch.complex64, "c128": torch.complex128}
_REAL = {"c64": torch.float32, "c128": torch.float64}
_SIZE = {"c64": 8, "c128": 16}
# the most elements of one drawn case, by element type (1 GiB in, 1 GiB out)
_LOG2_ELEMS = {"c64": 27, "c128": 26}


def _plan(name, dtype, n, batch, mode="correct", inverse=False, group=0):
    return dict(name=name, kind="plan", dtype=dtype, n=n, batch=batch, mode=mode, inverse=inverse, group=group)


def listed():
    return [
        # the smallest everyday call: one group of short signals, latency bound
        _plan("c64_256_b64", "c64", 1 << 8, 64),
        # a handful of longer signals in a loop: two passes, still latency bound
        _plan("c64_16384_b5", "c64", 1 << 14, 5),
        # the fault campaign: 2000 groups of 16 signals, checked and reported only
        _plan("c64_1024_campaign", "c64", 1 << 10, 32000, mode="detect", group=16),
        # the differentiable layer at its full size, forward and backward
        dict(name="layer_4096", kind="layer", dtype="c64", n=1 << 12, batch=2048, mode="correct"),
        # the throughput sweep, one precision and one length at a time
        _plan("c64_8192", "c64", 1 << 13, 1 << 14),
        _plan("c64_2e17_inverse", "c64", 1 << 17, 1000, inverse=True),  # a batch that is no power of two
        _plan("c64_2e19_off", "c64", 1 << 19, 128, mode="off"),  # without the checksum
        _plan("c64_2e22", "c64", 1 << 22, 32),
        _plan("c128_4096", "c128", 1 << 12, 1 << 14),
        _plan("c128_2e15_inverse", "c128", 1 << 15, 2000, inverse=True),
        _plan("c128_2e20", "c128", 1 << 20, 64),
        # mixed lengths, the ragged benchmark's distribution at a quarter of its signals
        dict(name="ragged_1024", kind="ragged", dtype="c64", count=1024, kmin=6, kmax=20, layout=20240504,
             persistent=True, mode="correct", inverse=False),
    ]


def draw(rng):
    dtype = rng.choice(["c64", "c64", "c64", "c128", "c128"])
    mode = rng.choice(["correct", "correct", "correct", "correct", "detect", "off"])
    inverse = rng.random() < 0.35
    kind = rng.choice(["plan"] * 8 + ["layer", "ragged"])
    top = _LOG2_ELEMS[dtype]
    if kind == "ragged":
        kmin = rng.randint(6, 10)
        kmax = rng.randint(kmin + 2, 20)
        # a count whose expected size stays a factor of two below the largest case
        mean = sum(1 << k for k in range(kmin, kmax + 1)) / (kmax - kmin + 1)
        most = max(2.0, min(4096.0, (1 << (top - 1)) / mean))
        count = max(2, int(math.exp(rng.uniform(math.log(2.0), math.log(most)))))
        return dict(kind=kind, dtype=dtype, count=count, kmin=kmin, kmax=kmax, layout=rng.randint(1, 10 ** 9),
                    persistent=rng.random() < 0.5, mode=mode, inverse=inverse)
    k = rng.randint(6, 14) if kind == "layer" else rng.randint(4, 24)
    elems = 2.0 ** rng.uniform(max(k, 14), top - (1 if kind == "layer" else 0))
    batch = max(1, int(elems / (1 << k)))
    if kind == "layer":
        return dict(kind=kind, dtype=dtype, n=1 << k, batch=batch, mode=mode)
    return dict(kind=kind, dtype=dtype, n=1 << k, batch=batch, mode=mode, inverse=inverse, group=0)


def _lengths(case):
    k = np.random.default_rng(case["layout"]).integers(case["kmin"], case["kmax"] + 1, size=case["count"])
    return np.int64(1) << k.astype(np.int64)


def _uniform(shape, dtype, seed, device):
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    re = torch.rand(shape, generator=g, device=device, dtype=_REAL[dtype])
    im = torch.rand(shape, generator=g, device=device, dtype=_REAL[dtype])
    return torch.complex(re.mul_(2).sub_(1), im.mul_(2).sub_(1))


def _inputs(case, seed):
    if case["kind"] == "ragged":
        return [_uniform((int(_lengths(case).sum()),), case["dtype"], seed, "cuda")]
    shape = (case["batch"], case["n"])
    x = [_uniform(shape, case["dtype"], seed, "cuda")]
    if case["kind"] == "layer":  # the gradient that arrives from above
        x.append(_uniform(shape, case["dtype"], seed + 1000003, "cuda"))
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    state = dict(case=case, x=x[0])
    if case["kind"] == "plan":
        state["plan"] = tf.Plan(case["n"], case["batch"], case["dtype"], group=case["group"])
    elif case["kind"] == "layer":
        state["x"].requires_grad_(True)
        state["gy"] = x[1]
    else:
        state["plan"] = tf.Ragged(_lengths(case), dtype=case["dtype"], persistent=case["persistent"])
        state["out"] = torch.empty_like(x[0])
    return state


def run(state):
    case, x = state["case"], state["x"]
    if case["kind"] == "plan":
        plan = state["plan"]
        return (plan.inverse if case["inverse"] else plan.forward)(x, ft_mode=case["mode"])
    if case["kind"] == "layer":
        y = layer.fft(x, ft_mode=case["mode"])
        (gx,) = torch.autograd.grad(y, x, state["gy"])
        return y.detach(), gx
    return state["plan"].execute(x, state["out"], ft_mode=case["mode"], inverse=case["inverse"], use_graph=True)


def work(case):
    if case["kind"] == "ragged":
        ln = _lengths(case)
        elems = int(ln.sum())
        flops = float((5.0 * ln * np.log2(ln)).sum())
    else:
        elems = case["n"] * case["batch"]
        flops = 5.0 * elems * math.log2(case["n"])
    both = 2 if case["kind"] == "layer" else 1  # forward and backward
    return {"bytes": 2 * elems * _SIZE[case["dtype"]] * both, "flops": flops * both}


def _dft(x, inverse):
    return torch.fft.ifft(x, dim=-1) if inverse else torch.fft.fft(x, dim=-1)


def exact(case, seed):
    x = [t.cpu().to(torch.complex128) for t in _inputs(case, seed)]
    if case["kind"] == "plan":
        return _dft(x[0], case["inverse"])
    if case["kind"] == "layer":
        return _dft(x[0], False), _dft(x[1], True) * case["n"]
    ln = _lengths(case)
    off = np.concatenate([[0], np.cumsum(ln)[:-1]])
    out = torch.empty_like(x[0])
    for n in np.unique(ln):
        at = torch.from_numpy(off[ln == n])[:, None] + torch.arange(int(n))[None, :]
        out[at] = _dft(x[0][at], case["inverse"])
    return out
