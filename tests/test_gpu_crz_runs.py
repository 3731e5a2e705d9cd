"""CRZ runs longer than the table kernel takes at a time (256 gates), and more phase coefficients than that, against
the CPU oracle (GPU only)."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import qpinn_oracle as O
from tests.gpu_helpers import TOL, rel, t2n

pytestmark = pytest.mark.gpu


def _run_of(n, count):
    """A run of `count` CRZ gates over all ordered pairs in turn, rotations around it, twice."""
    pairs = [(a, b) for a in range(n) for b in range(n) if a != b]
    gates, p = [], 0
    for _ in range(2):
        for q in range(n):
            gates.append((W.RX if q % 2 else W.RY, q, -1, p))
            p += 1
        for k in range(count):
            gates.append((W.CRZ, *pairs[k % len(pairs)], p))
            p += 1
    gates.append((W.RY, 0, -1, p))
    return W.Circuit(n, gates, p + 1)


@pytest.mark.parametrize("n,count", [(3, 256), (3, 257), (4, 600), (9, 300), (12, 0)])
def test_crz_runs(n, count):
    from paper_2506_23246_amd.api import Circuit, Context
    circ = _run_of(n, count) if count else W.cross_mesh(n, 4, "x")   # 12 qubits: 4 x 78 coefficients
    rng = np.random.default_rng(n + count)
    prm = rng.uniform(0, 2 * math.pi, circ.n_params).astype(np.float32)
    pts = rng.uniform(-1, 1, (3, 3)).astype(np.float32)
    c = Circuit(Context(0), circ)
    f, g, loss, grad = O.maxwell_eval(circ, prm, pts, W.MaxwellDesc())
    out, tan = c.simulate(prm, pts)
    r = c.maxwell(prm, pts, W.MaxwellDesc())
    errs = {"out": rel(t2n(out), f), "tan": rel(t2n(tan), g), "loss": rel(t2n(r["loss"]), [loss]), "grad": rel(t2n(r["grad"]), grad)}
    print(n, count, {k: f"{v:.1e}" for k, v in errs.items()}, flush=True)
    assert all(v < TOL for v in errs.values()), errs
