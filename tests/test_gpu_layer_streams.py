"""The differentiable layer with equal shapes on two streams at once, and in a
captured graph that replays between eager calls on another stream: a one-pass
length whose groups are shared by workgroups, tile launches, and a two-pass
length (workspace)."""
import numpy as np
import pytest

import oracle
import tfft_inputs as inputs

pytestmark = pytest.mark.gpu

SHAPES = [(256, 64), (4096, 514), (1 << 14, 6), (1 << 14, 128)]


@pytest.fixture(scope="module")
def layer():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2405_02520_amd import layer as L

    yield L
    L.clear_plan_cache()


def _data(n, batch, seed):
    import torch

    x0 = inputs.uniform(seed, batch, n, np.complex64)
    x = torch.from_numpy(x0).cuda().requires_grad_(True)
    rows = sorted({0, batch // 2, batch - 1})
    return x, rows, oracle.fft(x0[rows].astype(np.complex128))


def _step(layer, x):
    import torch

    y = layer.fft(x)
    (g,) = torch.autograd.grad(y, x, y.detach())
    return y.detach(), g


def _check(x, rows, ref, y, g):
    # the adjoint applied to the transform is n x
    assert oracle.rel_l2(y[rows].cpu().numpy(), ref) <= 1e-5
    assert oracle.rel_l2(g.cpu().numpy(), x.shape[-1] * x.detach().cpu().numpy()) <= 1e-5


@pytest.mark.parametrize("n,batch", SHAPES)
def test_two_streams(layer, n, batch):
    import torch

    print(f"two streams {n} x {batch}", flush=True)
    data = [_data(n, batch, 9300 + i) for i in range(2)]
    streams = [torch.cuda.Stream() for _ in data]
    torch.cuda.synchronize()
    outs = [[], []]
    for _ in range(6):
        for i, st in enumerate(streams):
            with torch.cuda.stream(st):
                outs[i].append(_step(layer, data[i][0]))
    torch.cuda.synchronize()
    for (x, rows, ref), runs in zip(data, outs):
        for y, g in runs:
            _check(x, rows, ref, y, g)
    (rep,) = [r for k, r in layer.last_reports().items() if k[:2] == (n, batch)]
    assert rep["forward"][0]["detected"] == 0 and rep["backward"][0]["detected"] == 0


@pytest.mark.parametrize("n,batch", SHAPES)
def test_graph_replays_beside_eager_calls(layer, n, batch):
    import torch

    print(f"graph {n} x {batch}", flush=True)
    layer.clear_plan_cache()
    (xg, rows, refg), (xe, _, refe) = _data(n, batch, 9310), _data(n, batch, 9311)
    warm, other = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(warm):
        _step(layer, xg)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        yg, gg = _step(layer, xg)
    for _ in range(4):
        yg.zero_()
        gg.zero_()
        torch.cuda.synchronize()
        g.replay()
        with torch.cuda.stream(warm):
            ye, ge = _step(layer, xe)
        with torch.cuda.stream(other):
            yo, go = _step(layer, xe)
        torch.cuda.synchronize()
        _check(xg, rows, refg, yg, gg)
        _check(xe, rows, refe, ye, ge)
        _check(xe, rows, refe, yo, go)
