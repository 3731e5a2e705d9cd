"""The planner rates an exchange's LDS layout by the banks that four lane bits span; counted lane by lane here,
every group of 16 lanes of a workgroup has as many distinct banks as any other, on both sides."""
import numpy as np
import pytest

import workloads as W
from tests.test_sweep_plan import LIB, _image, pytestmark  # noqa: F401


def _swz(x):
    return x ^ ((x >> 4 ^ x >> 8 ^ x >> 12 ^ x >> 16) & 15)


def _banks(words, n, T):
    """Distinct banks of each group of 16 lanes; words: 8 x the entry of thread u of a point."""
    TP = 1 << (n - 3)
    t = np.arange(T)
    e = (words[t % TP] // 8) ^ _swz((t // TP) << n)
    return [len(set(g & 15)) for g in e.reshape(-1, 16)]


@pytest.mark.parametrize("ent", ["cnot", "mixed"])
@pytest.mark.parametrize("n", range(3, 13))
def test_every_group_alike(n, ent):
    rings = {"cnot": lambda l: W.ring(n, W.CNOT, 1), "mixed": lambda l: W.ring(n, W.CNOT, 1 + l % 2) + W.ring(n, W.CZ, 2)}
    h, sw, lanes, *_ = _image(W.layered(n, 4, "xyz", rings[ent]))
    T = 64 if n <= 9 else (512 if n == 12 else 256)
    worst = 16
    for l, L in enumerate(sw):
        if not int(L["flags"]) & 1:
            continue
        for k in range(4):              # forward and reverse, writer and reader
            d = _banks(lanes[l][:, k], n, T)
            assert len(set(d)) == 1, (l, k, d)
            worst = min(worst, d[0])
    assert worst >= 8                   # the search always finds a layout with at most two lanes a bank
