"""Gradients of circuits with more layers than the table kernel scans at a time (1024), against the CPU oracle (GPU
only): one gate a layer, so that the statistics of all gates fit a workgroup's LDS.

Tolerance: a state or adjoint state of L layers is off by at most 6 roundings a layer, tol = 6 * 2^-24 * L of its
norm; a gradient component is a sum of products of the two, so off by 2 tol (2 more for the sums) of the product of
their norms, at most the sum over points of |sf| and |sg| * 3 pi (the angles' derivatives are pi, 3 coordinates)."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import qpinn_oracle as O
from tests.gpu_helpers import t2n

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,L", [(3, 1024), (3, 1025), (3, 1100), (5, 1026), (8, 1026), (11, 1026)])
def test_deep_adjoint(n, L):
    from paper_2506_23246_amd.api import Circuit, Context
    rng = np.random.default_rng(L + n)
    gates = []
    for l in range(L):
        gates += [((W.RX, W.RY)[l % 2], l % n, -1, l)] + (W.ring(n, W.CNOT, 1 + l % 2) if l % 3 else W.ring(n, W.CZ, 1))
    circ = W.Circuit(n, gates, L, out_qubits=[0, n - 1])
    params = rng.uniform(0, 2 * math.pi, L).astype(np.float32)
    pts = rng.uniform(-1, 1, (2, 3)).astype(np.float32)
    sf, sg = rng.standard_normal((2, 2)).astype(np.float32), rng.standard_normal((2, 2, 3)).astype(np.float32)
    g = t2n(Circuit(Context(0), circ).vjp(params, pts, sf, sg))
    ref = O.grad_reverse(circ, params, pts, sf.astype(np.float64), sg.astype(np.float64))
    tol = 4 * 6 * 2.0 ** -24 * L * (np.abs(sf).sum() + 3 * math.pi * np.abs(sg).sum())
    err = np.abs(g - ref).max()
    print(n, L, f"{err:.2e} of {np.abs(ref).max():.2e}, tolerance {tol:.2e}", flush=True)
    assert err < tol
    # one wrong sign of a layer's gate or mask would show: the gradient's components are well above the tolerance
    assert np.abs(ref).max() > 4 * tol
