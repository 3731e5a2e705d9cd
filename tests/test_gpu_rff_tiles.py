"""Random-Fourier-feature angles at the edges of their kernel's tiles (32 points, 32 features, 8 qubits per
step): features of zero weight and the other points of a call change no bit (GPU only; the values
themselves are held against the oracle by the forward tests)."""
import math

import numpy as np
import pytest

import workloads as W
from tests.gpu_helpers import t2n

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,F", [(3, 1), (4, 32), (8, 33), (9, 31), (12, 70)])
def test_rff_tile_edges(n, F):
    """Adding w = 0 times a feature adds a zero to every sum, and a point's angles are formed alone, so the
    padded and the single-point calls agree exactly."""
    from paper_2506_23246_amd.api import Circuit, Context
    ctx = Context(0)
    rng = np.random.default_rng(970 + n)
    B = rng.standard_normal((F, 3)).astype(np.float32)
    Wm = (rng.standard_normal((n, 2, F)) / math.sqrt(F)).astype(np.float32)

    def circuit(pad):
        Bp = np.concatenate([B, np.zeros((pad, 3), np.float32)])
        Wp = np.concatenate([Wm, np.zeros((n, 2, pad), np.float32)], axis=2).reshape(n, 2 * (F + pad))
        return Circuit(ctx, W.layered(n, 1, "rot", lambda l: W.ring(n, W.CZ, 1), out_qubits=[0, n - 1],
                                      enc=W.Encoding(kind=W.ENC_RFF, gate=W.ENC_RY, scale=W.SCALE_NONE, rff_B=Bp,
                                                     rff_W=Wp)))
    params = rng.uniform(0, 2 * math.pi, 3 * n).astype(np.float32)
    pts = rng.uniform(-1, 1, (33, 3)).astype(np.float32)
    out, tan = (t2n(x) for x in circuit(0).simulate(params, pts))
    for pad in (-F % 32, 32, 1):
        o, t = (t2n(x) for x in circuit(pad).simulate(params, pts))
        assert np.array_equal(o, out) and np.array_equal(t, tan)
    for i in (0, 31, 32):
        o, t = (t2n(x) for x in circuit(0).simulate(params, pts[i:i + 1]))
        assert np.array_equal(o[0], out[i]) and np.array_equal(t[0], tan[i])
