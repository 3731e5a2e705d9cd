"""Gradients with respect to the per-point angles and their Jacobian at every place a qubit can have
(register bits, lane bits, swap slots, waves), with and without an opening rotation stage, against the
CPU oracle (GPU only)."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import qpinn_oracle as O
from tests.gpu_helpers import TOL, rel, t2n

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", list(range(3, 12)))
@pytest.mark.parametrize("head,gate", [(True, W.ENC_RX), (False, W.ENC_RY)])
def test_input_grads_every_position(n, head, gate):
    from paper_2506_23246_amd.api import Circuit, Context
    rng = np.random.default_rng(950 + n)
    circ = W.layered(n, 2, "xyz", lambda l: W.ring(n, W.CNOT, 1), out_qubits=[0, n - 1, n // 2],
                     enc=W.Encoding(kind=W.ENC_ANGLES, gate=gate))
    if not head:
        circ.gates = W.ring(n, W.CZ, 1) + list(circ.gates)
    P = 2 * (256 // (1 << (n - 3))) + 1 if n < 8 else 5
    prm = rng.uniform(0, 2 * math.pi, circ.n_params).astype(np.float32)
    ang = rng.uniform(-math.pi, math.pi, (P, n)).astype(np.float32)
    jac = rng.uniform(-1, 1, (P, n, 3)).astype(np.float32)
    sf = rng.standard_normal((P, 3)).astype(np.float32)
    sg = rng.standard_normal((P, 3, 3)).astype(np.float32)
    c = Circuit(Context(0), circ)
    g, ga, gj = c.vjp(prm, None, sf, sg, angles=ang, jac=jac, input_grads=True)
    rg, ra, rj = O.grad_reverse(circ, prm, None, sf.astype(np.float64), sg.astype(np.float64), ang, jac, inputs=True)
    assert rel(t2n(g), rg) < TOL and rel(t2n(ga), ra) < TOL and rel(t2n(gj), rj) < TOL
