"""Outputs of circuits with more layers than the table kernel scans at a time (1024), against the CPU
oracle (GPU only).  A wrong X mask would change them by order one; the tolerance is the rounding of six
FP32 operations a layer, added up."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import qpinn_oracle as O
from tests.gpu_helpers import t2n

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1023, 1024, 1025, 1026, 2100])
def test_deep_circuit(L):
    from paper_2506_23246_amd.api import Circuit, Context
    rng = np.random.default_rng(L)
    circ = W.layered(3, L, "x", lambda l: W.ring(3, W.CNOT, 1 + l % 2))
    params = rng.uniform(0, 2 * math.pi, circ.n_params).astype(np.float32)
    pts = rng.uniform(-1, 1, (5, 3)).astype(np.float32)
    out, tan = Circuit(Context(0), circ).simulate(params, pts)
    f, g = O.simulate(circ, params, pts)
    tol = 6 * 2.0 ** -24 * L
    assert np.abs(t2n(out) - f).max() < tol and np.abs(t2n(tan) - g).max() < math.pi * 3 * tol
