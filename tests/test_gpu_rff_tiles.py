"""Random-Fourier-feature angles at the edges of their kernel's tiles (32 points, 32 features, 8 qubits per
step) against the CPU oracle (GPU only)."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import qpinn_oracle as O
from tests.gpu_helpers import TOL, rel, t2n

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,F", [(3, 1), (4, 32), (8, 33), (9, 31), (12, 70)])
def test_rff_tile_edges(n, F):
    from paper_2506_23246_amd.api import Circuit, Context
    rng = np.random.default_rng(970 + n)
    B = rng.standard_normal((F, 3)).astype(np.float32)
    Wm = (rng.standard_normal((n, 2 * F)) / math.sqrt(F)).astype(np.float32)
    circ = W.layered(n, 1, "rot", lambda l: W.ring(n, W.CZ, 1), out_qubits=[0, n - 1],
                     enc=W.Encoding(kind=W.ENC_RFF, gate=W.ENC_RY, scale=W.SCALE_NONE, rff_B=B, rff_W=Wm))
    params = rng.uniform(0, 2 * math.pi, circ.n_params).astype(np.float32)
    c = Circuit(Context(0), circ)
    for P in (1, 32, 33):
        pts = rng.uniform(-1, 1, (P, 3)).astype(np.float32)
        out, tan = c.simulate(params, pts)
        f, g = O.simulate(circ, params, pts)
        assert rel(t2n(out), f) < TOL and rel(t2n(tan), g) < TOL
