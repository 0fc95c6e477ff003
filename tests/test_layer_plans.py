"""Which plans the differentiable layer runs on which stream (CPU: the plans
and streams are stand-ins): a plan owns its workspace and must not run on two
streams at once."""
import contextlib
import types

import pytest
import torch


class FakePlan:
    def __init__(self, n, batch, dtype, inverse_unscaled=False):
        if FakePlan.capturing:
            raise AssertionError("a plan allocates: not under capture")
        self.adjoint, self.ran = inverse_unscaled, []

    def forward(self, x, ft_mode, stream=None):
        self.ran.append(FakePlan.at())
        return torch.fft.fft(x)

    def inverse(self, x, ft_mode, stream=None):
        self.ran.append(FakePlan.at())
        return torch.fft.ifft(x, norm="forward")

    def report(self):
        return self

    def close(self):
        pass


@pytest.fixture()
def layer(monkeypatch):
    from paper_2405_02520_amd import layer as L

    L.clear_plan_cache()
    FakePlan.capturing, FakePlan.at = False, lambda: L.at
    monkeypatch.setattr(L, "Plan", FakePlan)
    monkeypatch.setattr(torch.cuda, "device", lambda d: contextlib.nullcontext())
    monkeypatch.setattr(torch.cuda, "current_stream", lambda d=None: types.SimpleNamespace(cuda_stream=L.at))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda i: L.at, raising=False)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: FakePlan.capturing)
    monkeypatch.setattr(L, "at", 0, raising=False)
    yield L
    L.clear_plan_cache()


def _step(L):
    x = torch.randn(3, 8, dtype=torch.complex64, requires_grad=True)
    y = L.fft(x)
    (g,) = torch.autograd.grad(y, x, torch.ones_like(y))
    assert torch.allclose(g, torch.fft.ifft(torch.ones_like(y), norm="forward"))


def test_every_stream_has_its_own_plans(layer):
    pairs = []
    for st in (11, 22, 11, 22):
        layer.at = st
        _step(layer)
        pairs.append(layer._plans(8, 3, torch.complex64, torch.device("cpu")))
        (rep,) = layer.last_reports().values()  # one entry a shape: its latest executions
        assert (rep["forward"], rep["backward"]) == pairs[-1]
    assert pairs[0] is pairs[2] and pairs[1] is pairs[3]
    assert {id(p) for p in pairs[0]}.isdisjoint({id(p) for p in pairs[1]})
    for st, pair in ((11, pairs[0]), (22, pairs[1])):
        assert all(set(p.ran) == {st} for p in pair)


def test_backward_runs_with_the_plans_of_the_stream_it_is_called_on(layer):
    layer.at = 11
    _step(layer)
    x = torch.randn(3, 8, dtype=torch.complex64, requires_grad=True)
    y = layer.fft(x)
    layer.at = 22
    y.grad_fn.apply(torch.ones_like(y))  # outside autograd's engine
    assert layer._plans(8, 3, torch.complex64, torch.device("cpu"))[1].ran == [22]


def test_a_captured_graph_takes_over_the_warm_up_plans(layer):
    layer.at = 11
    _step(layer)
    warm = layer._plans(8, 3, torch.complex64, torch.device("cpu"))
    layer.at, FakePlan.capturing = 33, True
    _step(layer)
    assert layer._plans(8, 3, torch.complex64, torch.device("cpu")) is warm
    layer.at, FakePlan.capturing = 11, False
    _step(layer)  # replays and eager calls share nothing
    assert layer._plans(8, 3, torch.complex64, torch.device("cpu")) is not warm
    assert [p.ran for p in warm] == [[11, 33]] * 2


def test_forward_alone_on_another_stream_keeps_the_reports(layer):
    layer.at = 11
    _step(layer)
    _, adj = layer._plans(8, 3, torch.complex64, torch.device("cpu"))
    layer.at = 22
    with torch.no_grad():
        layer.fft(torch.randn(3, 8, dtype=torch.complex64))
    fwd, _ = layer._plans(8, 3, torch.complex64, torch.device("cpu"))
    (rep,) = layer.last_reports().values()
    assert (rep["forward"], rep["backward"]) == (fwd, adj)
