"""Layers of more rotations than a pass takes (19 generic ones): the first pass's images per term
choose how the layer's other passes run. Few of them, many, and few in one part and many in
the other: the terms are those without gathered rounds, bit for bit."""
import numpy as np
import pytest

from _compare import compare_fp64, oracle_arrays
import oracle
from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Simulator

pytestmark = pytest.mark.gpu

G = W.Gate


def _circuit(n, wires, seed):
    """An X string over the given wires (generator of the first), then a rotation of every wire, twice."""
    rng = np.random.default_rng(seed)
    g = [(G.H, wires[0], wires[0], 0.0)] + [(G.CX, a, b, 0.0) for a, b in zip(wires, wires[1:])]
    for _ in range(2):
        g += [(k, q, q, rng.uniform(0.2, 2.9)) for q in range(n) for k in (G.RX, G.RY, G.RZ)]
        g += [(G.CZ, 0, n - 1, 0.0)]
    gate, a, b, t = zip(*g)
    return W.Circuit(n, np.array(gate, np.uint8), np.array(a, np.uint32), np.array(b, np.uint32), np.array(t),
                     np.array([len(g)], np.int64), 0.0, f"wide(n={n},{len(wires)})")


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n,wires", [(20, [0, 3]), (24, [20, 21, 22, 23]), (24, [0, 5, 7, 12, 15, 18]), (33, [1, 2, 30, 32]),
                                     (40, [36, 37, 38, 39]), (64, [0, 20, 40, 60])])
def test_passes_of_one_layer(monkeypatch, n, wires, precision):
    c = _circuit(n, wires, n)
    got = []
    for v in "01":
        monkeypatch.setenv("QIMAX_GATHER", v)
        with Simulator(n, precision=precision) as s:
            for _ in range(2):
                s.reset()
                s.run(c).flush()
            got.append((s.generators(), s.stats()))
    for x, y in zip(got[0][0], got[1][0]):
        assert np.array_equal(x, y)
    for k in ("term_updates", "images", "passes", "terms"):
        assert got[0][1][k] == got[1][1][k]
    if precision == 64:
        compare_fp64(got[1][0], oracle_arrays(oracle.propagate(c), n))
