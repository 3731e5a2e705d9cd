"""The hybrid model's angle Jacobian carried forward with the activations, against the one of a backward
pass per qubit, in 64 bits: values and weight gradients, every input scaling, and the ways back to it."""
import pytest
import torch

import workloads as W
from paper_2506_23246_amd import hybrid as H


def _model(scale, n=4):
    circ = W.basic_entangling(n, 1, "rot", enc=W.Encoding(kind=W.ENC_ANGLES, gate=W.ENC_RX))
    fn = lambda p, th, jac: (torch.cos(th)[:, :3], -torch.sin(th)[:, :3, None] * jac[:, :3])
    return H.HybridQPINN(circ, scale=scale, n_freq=5, hidden=(7, 6), circuit_fn=fn, dtype=torch.float64, seed=scale)


@pytest.mark.parametrize("scale", range(5))
@pytest.mark.parametrize("P", [0, 1, 9])
def test_forward_jacobian(scale, P):
    m = _model(scale)
    pts = torch.rand(P, 3, dtype=torch.float64, generator=torch.Generator().manual_seed(P)) * 2 - 1
    ws = [p for l in m.layers for p in l.parameters()]
    th, jac = m.angles_jacobian(pts)
    x = pts.clone().requires_grad_(True)
    ref_th = m.angles(x)
    ref = H.input_jacobian(ref_th, x)
    assert jac.shape == ref.shape == (P, 4, 3)
    tol = dict(rtol=1e-11, atol=1e-12)    # 64-bit rounding through four layers
    torch.testing.assert_close(th, ref_th, **tol)
    torch.testing.assert_close(jac, ref, **tol)
    w = torch.linspace(-1, 1, jac.numel(), dtype=torch.float64).reshape(jac.shape)
    g = torch.autograd.grad((th.sum() + (w * jac * jac).sum()), ws, allow_unused=True)
    r = torch.autograd.grad((ref_th.sum() + (w * ref * ref).sum()), ws, allow_unused=True)
    for a, b in zip(g, r):
        torch.testing.assert_close(a if a is not None else torch.zeros(()).double().expand_as(b), b, rtol=1e-9, atol=1e-10)


def test_other_networks_keep_the_general_path():
    m = _model(4)
    assert m.plain_network()
    seen = []
    h = m.layers[1].register_forward_hook(lambda mod, i, o: seen.append(1))
    assert not m.plain_network()
    pts = torch.rand(6, 3, dtype=torch.float64) - 0.5
    f, d = m(pts)
    assert seen
    h.remove()
    f2, d2 = m(pts)
    torch.testing.assert_close(f, f2, rtol=1e-11, atol=1e-12)
    torch.testing.assert_close(d, d2, rtol=1e-11, atol=1e-12)

    class Other(H.HybridQPINN):
        def angles(self, x):
            return 0.5 * super().angles(x)
    o = Other(m.quantum.desc, scale=1, n_freq=5, hidden=(7, 6), circuit_fn=m.quantum._fn, dtype=torch.float64)
    assert not o.plain_network()
    with torch.no_grad(), pytest.raises(RuntimeError):
        m(pts)
