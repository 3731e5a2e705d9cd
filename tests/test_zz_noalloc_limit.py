"""The one comparison that decides whether a call fits the no-allocation entry point's scratch, on both
sides of the limit (GPU only)."""
import ctypes as C

import numpy as np
import pytest

import workloads as W
from oracle import qpinn_oracle as O
from tests.gpu_helpers import TOL, rel, t2n

pytestmark = pytest.mark.gpu


def test_documented_limit():
    import torch
    from paper_2506_23246_amd import _lib as L
    from paper_2506_23246_amd.api import Circuit, Context
    ctx = Context(0)
    w = W.config(2)                     # random Fourier features: scratch grows with the points
    c = Circuit(ctx, w.circuit)
    cap, tables = int(L.qp_noalloc_scratch_bytes()), c.info(14)
    counted = lambda P: int(L.qp_workspace_bytes(c.h, P, 0)) - tables
    al = lambda x: (x + 255) // 256 * 256
    n, F, grid = w.circuit.n, c.info(3), 4 * ctx.cu_count
    for P in (0, 1, 1000, 100003):      # the gate matrices, counts, angles and Jacobian, partials, sums
        assert counted(P) == (al(32 * (F + 1)) + al(8) + al(4 * n * P) + al(12 * n * P) + al(16 * F * grid)
                              + al(4 * grid) + al(32 * F))
    S = w.circuit.n_params // (3 * n)   # rotation layers, each with its phases, tangents and scales
    assert tables >= (8 << n) * S and tables < (8 << n) * (S + 1) + 4096 + 32 * F + 100 * S
    lo, hi = 1, cap // (16 * n)
    assert counted(lo) <= cap < counted(hi)
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if counted(mid) <= cap else (lo, mid)
    rng = np.random.default_rng(5)
    pts = torch.tensor(rng.uniform(-1, 1, (hi, 3)).astype(np.float32), device=ctx.dev)
    r = c.maxwell_noalloc(w.params, pts[:lo], w.loss)
    ref = c.maxwell(w.params, pts[:lo], w.loss)
    for k in ("out", "tan", "loss", "grad"):
        assert torch.equal(r[k], ref[k]), k
    f, g = O.simulate(w.circuit, w.params, pts[lo - 8:lo].cpu().numpy())
    assert rel(t2n(r["out"][lo - 8:]), f) < TOL and rel(t2n(r["tan"][lo - 8:]), g) < TOL
    assert counted(hi) > cap
    with pytest.raises(Exception, match="scratch"):
        c.maxwell_noalloc(w.params, pts, w.loss)
