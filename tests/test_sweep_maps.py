"""Index maps of the sweep layers: the turn between the rounds' last mapping and the layers' (forward of the calls
with an FP64 loss), and thin layers, which leave swaps out and exchange without an entangler, checked address by
address in the planner's image (no GPU)."""
import ctypes as C
import math
import os

import numpy as np
import pytest

import workloads as W
from oracle import qpinn_oracle as O

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_23246_amd",
                   "libqpinn.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")

XCHG, POS, LANES = 1, 256, 0xfff


def _thin(n, k, layers, ent):
    """`layers` layers of k rotated qubits each, a ring of CNOT or CZ gates behind each."""
    gates, p = [], 0
    for l in range(layers):
        for i in range(k):
            for kind in (W.RX, W.RY, W.RZ):
                gates.append((kind, (l * k + i) % n, -1, p))
                p += 1
        gates += W.ring(n, ent, 1)
    return W.Circuit(n, gates, p)


def _full(n):
    return W.layered(n, 3, "xyz", lambda l: W.ring(n, W.CNOT, 1 + l % 2))


def _index(n, t):
    """Basis index of every (thread, register) under the layers' mapping t."""
    u, r = np.arange(1 << (n - 3))[:, None], np.arange(8)[None, :]
    v = u ^ (((u >> 2) & 1) * 3) if n >= 6 else u
    j = sum(((r >> k) & 1) << int(t[k]) for k in range(3))
    return j + sum(((v >> (k - 3)) & 1) << int(t[k]) for k in range(3, n))


def _parity(x):
    x = np.asarray(x, np.int64)
    for s in (8, 4, 2, 1):
        x = x ^ (x >> s)
    return x & 1


def _entangle(rows, j):
    """Rows of an index map over GF(2), applied."""
    return sum(_parity(j & int(rows[k])) << k for k in range(16))


def _carries(waddr, raddr, wj, rj):
    """An exchange hands the amplitude at basis index wj, written at waddr, to who reads that index."""
    assert len(set(waddr.ravel())) == waddr.size and waddr.max() < 8 * waddr.size
    at = dict(zip(waddr.ravel().tolist(), wj.ravel().tolist()))
    assert [at[a] for a in raddr.ravel().tolist()] == rj.ravel().tolist()


@pytest.mark.parametrize("n", range(3, 13))
@pytest.mark.parametrize("kind", ["full", "thin"])
def test_turn(n, kind):
    from paper_2506_23246_amd import _lib as L
    from paper_2506_23246_amd.api import make_desc
    from tests.plan_emulator import _deposit, _regoff, plan_image
    from tests.test_sweep_plan import _image
    circ = _full(n) if kind == "full" else _thin(n, 2, 24, W.CNOT)
    h = _image(circ)[0]
    d, keep = make_desc(circ)
    nb = C.c_size_t(0)
    L.qp_plan_image(C.byref(d), None, 0, C.byref(nb))
    buf = (C.c_ubyte * nb.value)()
    assert L.qp_plan_image(C.byref(d), buf, nb.value, C.byref(nb)) == 0
    turn = np.frombuffer(bytes(buf), "<u4", 16, int(h["off_turn"]))
    lanes = np.frombuffer(bytes(buf), "<u4", 2 << (n - 3), int(h["off_tlanes"])).reshape(-1, 2)
    rpos = plan_image(circ)["rounds"][-1]["tpost"]
    wj = np.array([[_deposit(u, rpos, n) | _regoff(r, rpos) for r in range(8)] for u in range(1 << (n - 3))])
    _carries(lanes[:, :1] ^ turn[:8], lanes[:, 1:] ^ turn[8:], wj, _index(n, h["ftpos"]))


@pytest.mark.parametrize("ent", [W.CNOT, W.CZ])
@pytest.mark.parametrize("n,k", [(n, k) for n in range(5, 13) for k in (1, 3, 6) if k < n])
def test_thin_layers(n, k, ent):
    from tests.test_sweep_plan import _image
    h, sw, lanes = _image(_thin(n, k, 48, ent))[:3]
    first = int(h["first"])
    words = [int(L["flags"]) // POS for L in sw]
    thin = any(w != LANES for w in words)
    assert thin == (k <= 3 or n >= 9)    # 6 gates take all lanes of 7 qubits, and leave out the two slots of more
    cur = h["etpos"] if first else sw[0]["tin"]
    for l in range(first, len(sw)):
        L, w = sw[l], words[l]
        if int(L["flags"]) & XCHG:
            wj, rj = _index(n, cur), _index(n, L["tin"])
            # amplitude j after the entangler is amplitude A j before it
            _carries(lanes[l][:, :1] ^ L["woff"], lanes[l][:, 1:2] ^ L["roff"], wj, _entangle(L["arow"], rj))
            _carries(lanes[l][:, 2:3] ^ L["bwoff"], lanes[l][:, 3:] ^ L["broff"], _entangle(L["arow"], rj), wj)
        else:
            assert list(L["tin"][:n]) == list(cur[:n])
        assert all((w >> p) & 1 for p in range(n) if int(L["gate"][p]) >= 0)     # what has a gate is run
        out = list(L["tin"][:n])
        for lo, count in ((7, min(max(n - 7, 0), 2)), (9, max(n - 9, 0))):
            if (w >> lo) & ((1 << max(count, 0)) - 1):
                for i in range(count):
                    out[i], out[lo + i] = out[lo + i], out[i]
        assert out == list(L["tout"][:n])
        cur = L["tout"]
    assert list(h["ftpos"][:n]) == list(cur[:n])


@pytest.mark.parametrize("n,k,ent", [(5, 1, W.CNOT), (5, 3, W.CZ), (6, 2, W.CZ), (7, 1, W.CZ), (7, 3, W.CNOT), (7, 5, W.CZ)])
def test_thin_layers_match_oracle(n, k, ent):
    """Without slots a layer that leaves lanes out runs as a full one does: the emulated layers, forced exchanges
    among them, against the oracle."""
    from tests.test_sweep_plan import _run
    rng = np.random.default_rng(n * 10 + k)
    circ = _thin(n, k, 40, ent)
    params, pts = rng.uniform(0, 2 * math.pi, circ.n_params), rng.uniform(-1, 1, (1, 3))
    theta, J = O.encoding_angles(circ, pts)
    f, g = O.simulate(circ, params, pts)
    seeds = O.maxwell_seeds(g, pts, W.MaxwellDesc())
    fe, ge, grad = _run(circ, params, theta[0], J[0], seeds[0])
    np.testing.assert_allclose(fe, f[0], atol=1e-12)
    np.testing.assert_allclose(ge, g[0], atol=1e-11)
    np.testing.assert_allclose(grad, O.grad_reverse(circ, params, pts, None, seeds), atol=1e-10)
