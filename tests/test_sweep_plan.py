"""The sweep layers the fused kernels run (ZYZ split, phase tables, X masks, DPP/permlane/wave
positions, index-map exchanges), executed thread by thread in complex128 from the planner's image,
against the oracle: outputs, tangents and parameter gradients."""
import math
import os

import numpy as np
import pytest

import workloads as W
from oracle import qpinn_oracle as O
from tests.circuit_cases import opening_stage_cases

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_23246_amd",
                   "libqpinn.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")

XCHG = 1


def _image(circ):
    import ctypes as C
    from paper_2506_23246_amd import _lib as L
    from paper_2506_23246_amd.api import make_desc
    from tests.plan_emulator import HDR
    hdr = np.dtype(HDR.descr + [("n_phase", "<i4"), ("off_phase", "<i4"), ("off_phase_gates", "<i4"),
                                ("n_phase_coef", "<i4"), ("n_moments", "<i4"), ("off_pcsr_ptr", "<i4"),
                                ("off_pcsr_idx", "<i4"), ("n_sweeps", "<i4"), ("first", "<i4"), ("off_sweeps", "<i4"),
                                ("off_slanes", "<i4"), ("off_terms", "<i4"), ("hgate", "<i4", 16), ("etpos", "<i4", 16),
                                ("ftpos", "<i4", 16), ("gtpos", "<i4", 16), ("off_turn", "<i4"),
                                ("off_tlanes", "<i4")])
    sweep = np.dtype([("gate", "<i4", 12), ("flags", "<i4"), ("phase", "<i4"), ("term0", "<i4"), ("nterms", "<i4"),
                      ("tin", "<i4", 16), ("tout", "<i4", 16), ("woff", "<u4", 8), ("roff", "<u4", 8),
                      ("bwoff", "<u4", 8), ("broff", "<u4", 8), ("arow", "<u4", 16)])
    assert sweep.itemsize == 384
    from tests.plan_emulator import FUSED
    fused = np.dtype(FUSED.descr[:-1] + [("layer", "<i4"), ("head", "<i4"), ("pad", "<i4")])
    d, keep = make_desc(circ)
    nb = C.c_size_t(0)
    L.qp_plan_image(C.byref(d), None, 0, C.byref(nb))
    buf = (C.c_ubyte * nb.value)()
    assert L.qp_plan_image(C.byref(d), buf, nb.value, C.byref(nb)) == 0
    raw = bytes(buf)
    h = np.frombuffer(raw, hdr, 1)[0]
    S, TP = int(h["n_sweeps"]), 1 << (circ.n - 3)
    return (h, np.frombuffer(raw, sweep, S, int(h["off_sweeps"])),
            np.frombuffer(raw, "<u4", S * TP * 4, int(h["off_slanes"])).reshape(S, TP, 4) if S else None,
            np.frombuffer(raw, fused, int(h["n_fused"]), int(h["off_fused"])),
            np.frombuffer(raw, "<u4", (int(h["off_turn"]) - int(h["off_terms"])) // 4, int(h["off_terms"])).reshape(-1, 2),
            np.frombuffer(raw, "<i4", 4 * sum(g[0] == W.CRZ for g in circ.gates), int(h["off_phase_gates"])).reshape(-1, 4),
            np.frombuffer(raw, "<i4", 4 * int(h["n_phase"]), int(h["off_phase"])).reshape(-1, 4))


def _rot(kind, th):
    c, s = math.cos(th / 2), math.sin(th / 2)
    return np.array([[[c, -1j * s], [-1j * s, c]], [[c, -s], [s, c]], [[c - 1j * s, 0], [0, c + 1j * s]]][kind], complex)


def _par(x):
    return bin(int(x)).count("1") & 1


def _rows(rows, x):
    return sum(_par(int(rows[k]) & x) << k for k in range(16))


def _run(circ, params, theta, J, seeds_g):
    """(f, g, grad) of one point, as the kernel computes them."""
    h, sw, lanes, fused, terms, pgates, pst = _image(circ)
    n, TP, N = circ.n, 1 << (circ.n - 3), 1 << circ.n
    first, S = int(h["first"]), len(sw)
    U, ab = [], []
    for f in fused:
        u = np.eye(2, dtype=complex)
        for c in range(int(f["ncomp"])):
            u = _rot(int(f["kind"][c]), float(params[int(f["param"][c])])) @ u
        U.append(u)
        r0, r1 = abs(u[0, 0]), abs(u[1, 0])
        a0, a1 = np.angle(u[0, 0]), np.angle(u[1, 0])
        flip = r1 > r0
        t = -r0 / r1 if flip else r1 / r0
        ab.append((a1 - a0, -(a0 + a1), t, flip))       # RZ(a), RZ(c), tan, X flip
    assert all(abs(x[2]) <= 1 for x in ab)
    v = [u ^ (((u >> 2) & 1) * 3) if n >= 6 else u for u in range(TP)]

    def index(u, r, t):
        j = sum(((r >> k) & 1) << int(t[k]) for k in range(3))
        return j | sum(((v[u] >> (k - 3)) & 1) << int(t[k]) for k in range(3, n))

    def mapped(t):
        return np.array([[index(u, r, t) for r in range(8)] for u in range(TP)])

    def gate_of(l, q):                                    # layer l's gate on qubit q (not the folded layer's)
        return next((g for g, f in enumerate(fused) if f["layer"] == l and f["qubit"] == q and not f["head"]), -1)

    # X masks, coefficients, tables
    xs, tab, x = [0] * S, [None] * S, 0                   # the mask is zero at the readout
    for l in range(S - 1, first - 1, -1):
        for q in range(n):
            if gate_of(l, q) >= 0 and ab[gate_of(l, q)][3]:
                x ^= 1 << (n - 1 - q)
        xs[l] = x
        x = _rows(sw[l]["arow"], x)
    xe = x                                                # of the product state
    if first:
        xs[0] = xe
    for l in range(first, S):
        L = sw[l]
        j = mapped(L["tin"]) ^ xs[l]
        ph = np.zeros(j.shape)
        amp = 1.0
        for q in range(n):
            b = (j >> (n - 1 - q)) & 1
            gc, gp = gate_of(l, q), gate_of(l - 1, q)
            if gc >= 0:
                ph += (b - 0.5) * ab[gc][1]
                amp /= math.sqrt(1 + ab[gc][2] ** 2)
            if gp >= 0:
                ob = np.vectorize(lambda i: (_rows(L["arow"], int(i)) >> (n - 1 - q)) & 1)(j)
                ph += (ob - 0.5) * ab[gp][0] + (np.pi * (1 - ob) if ab[gp][3] else 0)
        for (mu, mv) in terms[int(L["term0"]):int(L["term0"]) + int(L["nterms"])]:
            ph += np.pi * np.vectorize(lambda i: _par(int(mu) & int(i)) & _par(int(mv) & int(i)))(j)
        if int(L["phase"]) >= 0:
            p0, cnt = pst[int(L["phase"])][:2]
            for (c, t, p, _) in pgates[p0:p0 + cnt]:
                ph += params[p] * ((j >> (n - 1 - c)) & 1) * (((j >> (n - 1 - t)) & 1) - 0.5)
        tab[l] = amp * np.exp(1j * ph)
    # encoding
    c, s = np.cos(theta / 2), np.sin(theta / 2)
    rx = circ.enc.gate == W.ENC_RX
    e = [np.array([c[q], -1j * s[q] if rx else s[q]], complex) for q in range(n)]
    d = [np.array([-s[q] / 2, -0.5j * c[q] if rx else c[q] / 2], complex) for q in range(n)]
    for q in range(n):
        if int(h["hgate"][q]) >= 0:
            e[q], d[q] = U[int(h["hgate"][q])] @ e[q], U[int(h["hgate"][q])] @ d[q]
    st = np.zeros((8, TP, 8), complex)
    for u in range(TP):
        for r in range(8):
            j = index(u, r, h["etpos"]) ^ xe
            a, D = 1 + 0j, np.zeros(3, complex)
            for q in range(n):
                b = (j >> (n - 1 - q)) & 1
                D, a = D * e[q][b] + a * J[q] * d[q][b], a * e[q][b]
            st[0, u, r], st[1:4, u, r] = a, D

    def exchange(st, wb, rb, wo, ro):
        buf = {}
        for u in range(TP):
            for r in range(8):
                buf[int(wb[u]) ^ int(wo[r])] = st[:, u, r].copy()
        assert len(buf) == N and max(buf) < 8 * N
        out = np.zeros_like(st)
        for u in range(TP):
            for r in range(8):
                out[:, u, r] = buf[int(rb[u]) ^ int(ro[r])]
        return out

    def swap(st, i, wave):
        out = np.zeros_like(st)
        k = 6 + i if wave else 4 + i                      # thread bit
        for u in range(TP):
            for r in range(8):
                rb, ub = (r >> i) & 1, (u >> k) & 1
                out[:, (u & ~(1 << k)) | (rb << k), (r & ~(1 << i)) | (ub << i)] = st[:, u, r]
        return out

    def partner(st, pos):
        if pos < 3:
            return st[:, :, [r ^ (1 << pos) for r in range(8)]]
        k = pos - 3
        return st[:, [u ^ (7 if k == 2 else 1 << k) for u in range(TP)]]

    def bit(pos):
        if pos < 3:
            return np.array([[(r >> pos) & 1 for r in range(8)]] * TP)
        return np.array([[(v[u] >> (pos - 3)) & 1] * 8 for u in range(TP)])

    def gate(st, pos, t):
        return st + np.where(bit(pos), t, -t) * partner(st, pos)

    def tcoef(l, g, flipped=0):
        q = int(fused[g]["qubit"])
        return ab[g][2] * (-1 if (xs[l] >> (n - 1 - q)) & 1 else 1)

    def groups(L):
        """Gate lists in forward order: the positions reached in place, the slots, the wave bits."""
        base = [(k, int(L["gate"][k])) for k in range(min(n, 7))]
        slots = [(i, int(L["gate"][7 + i])) for i in range(max(0, min(n - 7, 2)))]
        wave = [(i, int(L["gate"][9 + i])) for i in range(max(0, n - 9))]
        return base, slots, wave

    for l in range(first, S):
        L = sw[l]
        if int(L["flags"]) & XCHG:
            st[:4] = exchange(st[:4], lanes[l][:, 0], lanes[l][:, 1], L["woff"], L["roff"])
        st[:4] *= tab[l]
        for gi, grp in enumerate(groups(L)):
            if gi and grp:
                for i, _ in grp:
                    st[:4] = swap(st[:4], i, gi == 2)
            for pos, g in grp:
                if g >= 0:
                    st[:4] = gate(st[:4], pos, tcoef(l, g))
    j = mapped(h["ftpos"])
    m = int(h["n_out"])
    z = np.array([[[1.0 - 2 * _par(int(h["zmask"][i]) & int(jj)) for jj in row] for row in j] for i in range(m)])
    f = np.array([np.sum(z[i] * np.abs(st[0]) ** 2) for i in range(m)])
    gg = np.array([[2 * np.sum(z[i] * np.real(np.conj(st[0]) * st[1 + k])) for k in range(3)] for i in range(m)])
    D = [sum(seeds_g[i, k] * z[i] for i in range(m)) for k in range(3)]
    st[4] = sum(D[k] * st[1 + k] for k in range(3))
    for k in range(3):
        st[5 + k] = D[k] * st[0]
    Sxy, Sz, mom = np.zeros((len(fused), 2)), np.zeros(len(fused)), {}

    def stats(pos, g, sc):
        y = partner(st[:4], pos)
        xx = np.conj(st[4:])
        b = bit(pos)
        Sxy[g] = sc * np.sum(np.imag(xx * y)), sc * np.sum(np.where(b, 1, -1) * np.real(xx * y))

    for l in range(S - 1, -1, -1):
        L, pull = sw[l], l >= first
        base, slots, wave = groups(L)
        sc = 1.0
        for gi, grp in ((2, wave), (1, slots), (0, base)):
            for pos, g in grp:
                if g >= 0 and pull:
                    st = gate(st, pos, -tcoef(l, g))
                    sc /= 1 + ab[g][2] ** 2
            for pos, g in grp:
                if g >= 0:
                    stats(pos, g, sc)
            if gi and grp:
                for i, _ in grp:
                    st = swap(st, i, gi == 2)
        w = np.sum(np.imag(np.conj(st[4:]) * st[:4]), axis=0) * sc
        ji = mapped(L["tin"]) ^ xs[l]                     # basis index
        sgn = lambda q: 1 - 2 * ((ji >> (n - 1 - q)) & 1)  # noqa: E731
        for g in {int(x) for x in L["gate"]} - {-1}:
            Sz[g] = np.sum(w * sgn(int(fused[g]["qubit"])))
            if (xs[l] >> (n - 1 - int(fused[g]["qubit"]))) & 1:
                Sxy[g, 1] *= -1                           # X Y X = -Y
        if int(L["phase"]) >= 0:
            p0, cnt = pst[int(L["phase"])][:2]
            for (c, t, p, _) in pgates[p0:p0 + cnt]:
                mom[p] = mom.get(p, 0.0) + 0.5 * np.sum(w * (sgn(t) - sgn(c) * sgn(t)))
        if pull:
            st = st * np.conj(tab[l])
            if int(L["flags"]) & XCHG:
                st = exchange(st, lanes[l][:, 2], lanes[l][:, 3], L["bwoff"], L["broff"])
    # gradient: axis of the generator at the statistic's place
    P = [np.array([[0, 1], [1, 0]]), np.array([[0, -1j], [1j, 0]]), np.diag([1.0, -1.0])]
    grad = np.zeros(len(params))
    for g, fu in enumerate(fused):
        for ci in range(int(fu["ncomp"])):
            Wm = np.eye(2, dtype=complex)
            for c2 in range(ci):
                Wm = _rot(int(fu["kind"][c2]), float(params[int(fu["param"][c2])])) @ Wm
            G = Wm.conj().T @ P[int(fu["kind"][ci])] @ Wm
            R = U[g] if int(fu["head"]) else _rot(2, ab[g][1])
            G = R @ G @ R.conj().T
            nv = [0.5 * np.real(np.trace(p @ G)) for p in P]
            grad[int(fu["param"][ci])] += nv[0] * Sxy[g, 0] + nv[1] * Sxy[g, 1] + nv[2] * Sz[g]
    for p, val in mom.items():
        grad[p] += val
    return f, gg, grad


def _cases():
    out = [(name, c) for name, c, _ in opening_stage_cases()]
    for n in range(3, 13):
        rings = [W.ring(n, W.CNOT, 1) + W.ring(n, W.CZ, 2), W.ring(n, W.CZ, 1), W.ring(n, W.CNOT, 2)]
        out.append((f"mixed {n}", W.layered(n, 3 if n < 11 else 2, "xyz", lambda l, r=rings: r[l],
                                            out_qubits=[0, n - 1, n // 2])))
    out.append(("crz 5", W.cross_mesh(5, 3, "xz")))
    out.append(("crz 10", W.cross_mesh(10, 2, "x")))
    gates = [(W.CRZ, 0, 3, 0), (W.CZ, 2, 5, -1)] + [(W.RX, q, -1, 1 + q) for q in range(6)] + W.ring(6, W.CNOT, 1) + [
        (W.CRZ, 1, 2, 7), (W.CZ, 0, 4, -1), (W.CRZ, 2, 1, 7), (W.RY, 4, -1, 8)]
    out.append(("crz mixed", W.Circuit(6, gates, 9)))
    gates = [(W.RX, 3, -1, 0)] + W.ring(11, W.CNOT, 1) + [(W.RY, 9, -1, 1), (W.CNOT, 9, 0, -1), (W.RZ, 9, -1, 2),
                                                           (W.RX, 1, -1, 3)]
    out.append(("sparse 11", W.Circuit(11, gates, 4)))
    out.append(("no rotation", W.Circuit(5, W.ring(5, W.CNOT, 1), 0)))
    return out


@pytest.mark.parametrize("case", range(len(_cases())))
def test_sweep_layers_match_oracle(case):
    name, circ = _cases()[case]
    rng = np.random.default_rng(900 + case)
    params = rng.uniform(0, 2 * math.pi, circ.n_params)
    if circ.n_params > 3:
        params[1] = 0.0            # a degenerate rotation
    pts = rng.uniform(-1, 1, (1, 3))
    theta, J = O.encoding_angles(circ, pts)
    f, g = O.simulate(circ, params, pts)
    Wg = O.maxwell_seeds(g, pts, W.MaxwellDesc())
    fe, ge, grad = _run(circ, params, theta[0], J[0], Wg[0])
    np.testing.assert_allclose(fe, f[0], atol=1e-12)
    np.testing.assert_allclose(ge, g[0], atol=1e-11)
    if circ.n_params:
        np.testing.assert_allclose(grad, O.grad_reverse(circ, params, pts, None, Wg), atol=1e-11)
