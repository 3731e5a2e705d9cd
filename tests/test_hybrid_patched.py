"""Models whose parts are patched, hooked or computed in fewer bits: the field derivatives follow what the
model computes, and hooks see the calls they saw before.  (CPU, the circuit replaced by a closed form.)"""
import pytest
import torch
from torch import nn

import workloads as W
from paper_2506_23246_amd import hybrid as H
from paper_2506_23246_amd.train import hybrid_total_loss


def _model(dtype=torch.float64):
    circ = W.basic_entangling(4, 1, "rot", enc=W.Encoding(kind=W.ENC_ANGLES, gate=W.ENC_RX))
    fn = lambda p, th, jac: (torch.cos(th)[:, :3], -torch.sin(th)[:, :3, None] * jac[:, :3])
    return H.HybridQPINN(circ, scale=H.SCALE_ACOS, n_freq=5, hidden=(7, 6), circuit_fn=fn, dtype=dtype, seed=2)


def _points(P=6, seed=3):
    return torch.rand(P, 3, dtype=torch.float64, generator=torch.Generator().manual_seed(seed)) - 0.5


def _angles_on_instance(m):
    orig = m.angles
    m.angles = lambda x: 0.7 * orig(x) + 0.1 * x[:, :1]


def _forward_on_layer(m):
    lin = m.layers[1]
    orig = lin.forward
    lin.forward = lambda h: orig(h) + 0.3 * torch.sin(orig(h))


def _layer_subclass(m):
    class Bent(nn.Linear):
        def forward(self, h):
            return super().forward(h) ** 2
    b = Bent(7, 6, dtype=torch.float64)
    b.load_state_dict(m.layers[1].state_dict())
    m.layers[1] = b


def _forward_on_class(m, monkeypatch):
    orig = nn.Linear.forward
    monkeypatch.setattr(nn.Linear, "forward", lambda self, h: orig(self, h) + 0.2 * (orig(self, h) ** 2 if self is not m.head else 0))


def _global_hook(m):
    return nn.modules.module.register_module_forward_hook(
        lambda mod, i, o: o * 1.5 + 0.1 * o * o if mod in list(m.layers) else None)


class _BentLinear(torch.overrides.TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        out = func(*args, **(kwargs or {}))
        return torch.sinh(out) if func is nn.functional.linear and out.shape[1] == 6 else out


class _BentWeight(torch.Tensor):
    """A weight that has linear() do something else (as quantised weights do)."""
    @classmethod
    def __torch_function__(cls, func, types, args=(), kwargs=None):
        with torch._C.DisableTorchFunctionSubclass():
            out = func(*args, **(kwargs or {}))
            return torch.sinh(out) if func is nn.functional.linear else out


def _weight_subclass(m):
    m.layers[1]._parameters["weight"] = m.layers[1].weight.detach().clone().as_subclass(_BentWeight).requires_grad_(True)


@pytest.mark.parametrize("patch", ["none", "angles", "layer", "subclass", "class", "global hook", "mode", "weight"])
def test_derivatives_are_those_of_the_fields(patch, monkeypatch):
    m, pts = _model(), _points()
    handle, mode = None, None
    if patch == "angles": _angles_on_instance(m)
    elif patch == "layer": _forward_on_layer(m)
    elif patch == "subclass": _layer_subclass(m)
    elif patch == "class": _forward_on_class(m, monkeypatch)
    elif patch == "global hook": handle = _global_hook(m)
    elif patch == "weight": _weight_subclass(m)
    elif patch == "mode": mode = _BentLinear()
    try:
        if mode: mode.__enter__()
        assert m.plain_network() == (patch == "none")
        f, d = m(pts)
        torch.testing.assert_close(f, m.fields(pts), rtol=1e-12, atol=1e-13)
        h = 1e-6
        for c in range(3):
            e = torch.zeros(3, dtype=torch.float64)
            e[c] = h
            fd = (m.fields(pts + e) - m.fields(pts - e)) / (2 * h)
            # central differences: h^2 of truncation and rounding / h, both about 1e-10
            torch.testing.assert_close(d[:, :, c].detach(), fd.detach(), rtol=1e-7, atol=1e-8)
    finally:
        if mode: mode.__exit__(None, None, None)
        if handle: handle.remove()


def test_a_default_device_keeps_the_short_way():
    m = _model()
    with torch.device("cpu"):
        assert m.plain_network()


@pytest.mark.parametrize("how", ["bfloat16", "autocast"])
def test_fewer_bits_keep_autograd(how):
    """1 - tanh^2 of a 16-bit activation would lose what tanh's own backward keeps."""
    m = _model(torch.float32)
    pts = _points().float()
    if how == "bfloat16":
        m, pts = m.bfloat16(), pts.bfloat16()
    with torch.autocast("cpu", dtype=torch.bfloat16, enabled=how == "autocast"):
        _, d = m(pts)
        x = pts.clone().requires_grad_(True)
        th = m.angles(x)
        _, tan = m.quantum(th, H.input_jacobian(th, x))
        ref = torch.einsum("fi,pic->pfc", m.head.weight, tan.to(m.head.weight.dtype))
    assert torch.equal(d, ref)


@pytest.mark.parametrize("part", ["quantum", "head", "head forward", "none"])
def test_hooks_see_each_point_set(part):
    m, pts, ic = _model(), _points(5), _points(4)[:, :2]
    ref = hybrid_total_loss(m, pts, ic, W.TotalLossDesc())
    sizes = []
    if part == "head forward":
        orig = m.head.forward
        m.head.forward = lambda x: (sizes.append(len(x)), orig(x))[1]
    elif part != "none":
        getattr(m, part).register_forward_hook(lambda mod, i, o: sizes.append(len(i[0])))
    t = hybrid_total_loss(m, pts, ic, W.TotalLossDesc())
    if part != "none":
        assert sizes == [5, 5, 5, 4]      # collocation points, y-mirror, x-mirror, initial plane
    else:
        assert m.plain_model()
    for k in ref:
        torch.testing.assert_close(t[k], ref[k], rtol=1e-12, atol=1e-13)
