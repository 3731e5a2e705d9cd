"""Circuits whose layers rotate few qubits: groups of positions (lanes, swap slots, wave bits) left out layer by
layer, exchanges put in to bring the gates together, next to full layers, CZ and CRZ between them, with every
call that runs layers, against the CPU oracle (GPU only)."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import qpinn_oracle as O
from tests.gpu_helpers import TOL, rel, t2n

pytestmark = pytest.mark.gpu


def _circuit(n, counts, ent, enc, first_ring):
    """Layers with the given numbers of rotated qubits (each layer's start where the last one's ended)."""
    gates, p, at = (W.ring(n, W.CNOT, 1) if first_ring else []), 0, 1
    for l, k in enumerate(counts):
        for i in range(k):
            q = (at + i * (2 if n % 2 else 1)) % n
            for kind in ((W.RY, W.RZ) if l % 2 else (W.RZ, W.RY, W.RX)):
                gates.append((kind, q, -1, p))
                p += 1
        at += k
        gates += {"cnot": W.ring(n, W.CNOT, 1), "cz": W.ring(n, W.CZ, 1 + l % 2),
                  "one": [(W.CNOT, l % n, (l + 2) % n, -1)]}.get(ent, [])
        if ent == "crz":
            gates += [(W.CRZ, l % n, (l + 1) % n, p), (W.CZ, 0, n - 1, -1)]
            p += 1
    return W.Circuit(n, gates, p, enc=enc, out_qubits=[0, n - 1, n // 2])


CASES = [(5, [3, 1, 2, 3, 1, 3, 2, 1, 2, 3, 1, 1]), (6, [1, 2, 3, 6, 1, 2, 3, 1, 2, 1]), (7, [3, 1, 7, 2, 4, 1, 1, 3, 2, 1]),
         (8, [1, 3, 5, 8, 2, 7, 1, 3, 1, 2]), (9, [3, 1, 8, 2, 9, 1, 3, 7, 1, 2]), (10, [2, 1, 7, 3, 10, 1, 8, 3, 1]),
         (11, [1, 3, 7, 11, 2, 1, 8, 3, 1]), (12, [3, 1, 7, 2, 12, 8, 1, 3, 1])]


@pytest.mark.parametrize("ent", ["cnot", "cz", "one", "crz"])
@pytest.mark.parametrize("n,counts", CASES)
def test_points(n, counts, ent):
    from paper_2506_23246_amd.api import Batch, Circuit, Context
    ctx = Context(0)
    rng = np.random.default_rng(n)
    circ = _circuit(n, counts, ent, W.Encoding(), first_ring=ent == "one")
    prm = rng.uniform(0, 2 * math.pi, circ.n_params).astype(np.float32)
    P = 2 * (256 >> (n - 3)) + 1 if n < 8 else 3
    pts = rng.uniform(-1, 1, (P, 3)).astype(np.float32)
    sf, sg = rng.standard_normal((P, 3)).astype(np.float32), rng.standard_normal((P, 3, 3)).astype(np.float32)
    f, g, loss, grad = O.maxwell_eval(circ, prm, pts, W.MaxwellDesc())
    ref = O.grad_reverse(circ, prm, pts, sf.astype(np.float64), sg.astype(np.float64))
    shapes = [None] + ([(2, 1), (4, 1)] if n >= 10 and ent != "crz" else [])
    for shape in shapes:                                   # both exchange depths
        c = Circuit(ctx, circ)
        if shape:
            c.set_launch(*shape)
        out, tan = c.simulate(prm, pts)
        pk, _ = c.simulate(prm, pts, tangents=False)
        r = c.maxwell(prm, pts, W.MaxwellDesc())
        v = c.vjp(prm, pts, sf, sg)
        errs = {"out": rel(t2n(out), f), "tan": rel(t2n(tan), g), "packed": rel(t2n(pk), f), "loss": rel(t2n(r["loss"]), [loss]),
                "grad": rel(t2n(r["grad"]), grad), "vjp": rel(t2n(v), ref)}
        print(n, ent, shape, {k: f"{x:.1e}" for k, x in errs.items()}, flush=True)
        assert all(x < TOL for x in errs.values()), errs
    b = Batch(ctx, [circ], [P])
    arr, bufs = b.io([prm], [pts])
    b.run(arr, W.MaxwellDesc())
    assert rel(t2n(bufs[0]["grad"]), grad) < TOL and rel(t2n(bufs[0]["tan"]), g) < TOL


@pytest.mark.parametrize("first_ring", [False, True])
@pytest.mark.parametrize("n,counts", CASES)
def test_input_grads(n, counts, first_ring):
    from paper_2506_23246_amd.api import Circuit, Context
    rng = np.random.default_rng(100 + n)
    circ = _circuit(n, counts, "cnot", W.Encoding(kind=W.ENC_ANGLES, gate=W.ENC_RX), first_ring)
    P = 5 if n < 10 else 2
    prm = rng.uniform(0, 2 * math.pi, circ.n_params).astype(np.float32)
    ang = rng.uniform(-math.pi, math.pi, (P, n)).astype(np.float32)
    jac = rng.uniform(-1, 1, (P, n, 3)).astype(np.float32)
    sf, sg = rng.standard_normal((P, 3)).astype(np.float32), rng.standard_normal((P, 3, 3)).astype(np.float32)
    c = Circuit(Context(0), circ)
    g, ga, gj = c.vjp(prm, None, sf, sg, angles=ang, jac=jac, input_grads=True)
    rg, ra, rj = O.grad_reverse(circ, prm, None, sf.astype(np.float64), sg.astype(np.float64), ang, jac, inputs=True)
    assert rel(t2n(g), rg) < TOL and rel(t2n(ga), ra) < TOL and rel(t2n(gj), rj) < TOL


SHALLOW = [(n, c) for n in (10, 11, 12) for c in ([1, 1, 1, 2], [3, 1, 2, 1], [n // 2, 1, 2, 1], [8, 2, 1, 1], [n, 1, 1, 2])]


@pytest.mark.parametrize("n,counts", SHALLOW)
def test_shallow(n, counts):
    """The fewest layers that leave positions out, behind opening layers that take register bits, lanes, slots and
    wave bits."""
    test_points(n, counts, "cnot")
    for first_ring in (False, True):
        test_input_grads(n, counts, first_ring)
