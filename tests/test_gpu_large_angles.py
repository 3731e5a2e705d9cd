"""Parameters of many turns (up to the largest float), where theta / (2 pi) cannot be rounded to 64 bits
before it is reduced, against the CPU oracle (GPU only): rotations and CRZ phases, the forward by layers and
by rounds, and the adjoint.  The bar is that of every other FP32 result."""
import numpy as np
import pytest

import workloads as W
from oracle import qpinn_oracle as O
from tests.gpu_helpers import TOL, rel, t2n

pytestmark = pytest.mark.gpu

CASES = {
    "4q xyz cnot": lambda: W.layered(4, 3, "xyz", lambda l: W.ring(4, W.CNOT, 1)),
    "7q x crz": lambda: W.cross_mesh(7, 2, "x"),
    "8q rot cz": lambda: W.layered(8, 2, "rot", lambda l: W.ring(8, W.CZ, 1 + l)),
    "10q xz crz": lambda: W.cross_mesh(10, 2, "xz"),
    "12q xyz cnot": lambda: W.layered(12, 2, "xyz", lambda l: W.ring(12, W.CNOT, 1)),
}


@pytest.mark.parametrize("lo,hi", [(5.8, 6.3), (8, 14), (20, 38)])
@pytest.mark.parametrize("case", CASES)
def test_large_angles(case, lo, hi):
    from paper_2506_23246_amd.api import Circuit, Context
    circ = CASES[case]()
    rng = np.random.default_rng(circ.n)
    prm = (rng.choice([-1.0, 1.0], circ.n_params) * 10 ** rng.uniform(lo, hi, circ.n_params)).astype(np.float32)
    P = 9 if circ.n < 10 else 3
    pts = rng.uniform(-1, 1, (P, 3)).astype(np.float32)
    sf, sg = rng.standard_normal((P, 3)).astype(np.float32), rng.standard_normal((P, 3, 3)).astype(np.float32)
    c = Circuit(Context(0), circ)
    p64 = prm.astype(np.float64)
    f, g = O.simulate(circ, p64, pts)
    out, tan = c.simulate(prm, pts)
    r = c.maxwell(prm, pts, W.MaxwellDesc())
    _, _, loss, grad = O.maxwell_eval(circ, p64, pts, W.MaxwellDesc())
    vjp = c.vjp(prm, pts, sf, sg)
    ref = O.grad_reverse(circ, p64, pts, sf.astype(np.float64), sg.astype(np.float64))
    errs = {"out": rel(t2n(out), f), "tan": rel(t2n(tan), g), "rounds out": rel(t2n(r["out"]), f),
            "loss": rel(t2n(r["loss"]), [loss]), "grad": rel(t2n(r["grad"]), grad), "vjp": rel(t2n(vjp), ref)}
    print(case, lo, hi, {k: f"{v:.1e}" for k, v in errs.items()}, flush=True)
    assert all(v < TOL for v in errs.values()), errs
