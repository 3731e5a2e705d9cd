"""Outputs alone of 3-qubit circuits on both sides of the rule that has shallow ones run by rounds (layers,
points, CRZ phases, gates formed in FP32), against the same points with tangents, which always run by layers,
and against the CPU oracle (GPU only)."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import qpinn_oracle as O
from tests.gpu_helpers import TOL, rel, t2n

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [1, 1025, 262144, 262145])
@pytest.mark.parametrize("kind", ["L1", "L3", "L4", "crz", "rff", "angles", "first ring"])
def test_both_sides(kind, P):
    from paper_2506_23246_amd import _lib as L
    from paper_2506_23246_amd.api import Circuit, Context
    rng = np.random.default_rng(P)
    enc = {"rff": W.Encoding(kind=W.ENC_RFF, rff_B=rng.standard_normal((5, 3)).astype(np.float32),
                             rff_W=rng.standard_normal((3, 10)).astype(np.float32)),
           "angles": W.Encoding(kind=W.ENC_ANGLES, gate=W.ENC_RX)}.get(kind, W.Encoding())
    circ = W.cross_mesh(3, 2, "x") if kind == "crz" else W.layered(
        3, {"L1": 1, "L3": 3, "L4": 4}.get(kind, 2), "xyz", lambda l: W.ring(3, W.CNOT, 1) + W.ring(3, W.CZ, 1), enc=enc)
    if kind == "first ring":
        circ.gates = W.ring(3, W.CNOT, 1) + list(circ.gates)
    prm = rng.uniform(0, 2 * math.pi, circ.n_params).astype(np.float32)
    pts = rng.uniform(-1, 1, (P, 3)).astype(np.float32)
    ang, jac = (None, None) if kind != "angles" else (rng.uniform(-3, 3, (P, 3)).astype(np.float32),
                                                      rng.uniform(-1, 1, (P, 3, 3)).astype(np.float32))
    x = None if kind == "angles" else pts
    c = Circuit(Context(0), circ)
    pk, _ = c.simulate(prm, x, ang, jac, tangents=False)
    out, _ = c.simulate(prm, x, ang, jac)
    p32, _ = c.simulate(prm, x, ang, jac, tangents=False, flags=L.QP_FLAG_GATES_FP32)
    # both forwards are of the order of 20 FP32 roundings per layer from the exact one
    assert rel(t2n(pk), t2n(out)) < TOL and rel(t2n(p32), t2n(out)) < TOL
    s = slice(max(0, P - 20), P)
    f, _ = O.simulate(circ, prm, None if x is None else pts[s], None if ang is None else ang[s], None if jac is None else jac[s])
    assert rel(t2n(pk)[s], f) < TOL
