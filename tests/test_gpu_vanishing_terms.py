"""Rotations by multiples of pi / 2 leave entries of 6e-17 where they mean none: products of a
few of them vanish in FP32 (of twenty, in FP64), and terms of weight zero go at the end of every
pass. Passes that leave their images unsorted must hold no more terms than sorted ones."""
import numpy as np
import pytest

from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Batch, Simulator

pytestmark = pytest.mark.gpu


def _circuit(n, k, theta, seed=1):
    """k rotations about different axes between random Clifford moments."""
    c = W.c2_clifford_rz(seed, n, 4 * k, k)
    t = np.where(np.isin(c.gate, [int(g) for g in W.ROTATIONS]), theta, 0.0)
    return W.Circuit(c.n, c.gate, c.q0, c.q1, t, c.layer_end, c.eps, c.name)


def _run(monkeypatch, value, c, precision):
    monkeypatch.setenv("QIMAX_MERGE_FREE", value)
    with Simulator(c.n, precision=precision) as s:
        s.run(c)
        return s.generators(), s.stats()


@pytest.mark.parametrize("n", [16, 32, 48])
@pytest.mark.parametrize("k,theta,precision", [(16, np.pi / 2, 32), (16, np.pi, 32), (12, 1e-12, 32), (12, 2e-38, 32),
                                               (16, 1e-25, 64), (12, 1e-300, 64)])
def test_products_that_vanish(monkeypatch, n, k, theta, precision):
    c = _circuit(n, k, theta)
    (g0, s0), (g1, s1) = (_run(monkeypatch, v, c, precision) for v in "01")
    for x, y in zip(g0, g1):
        assert np.array_equal(x, y)
    for key in ("images", "term_updates", "terms", "rounds"):
        assert s0[key] == s1[key], key


@pytest.mark.parametrize("max_n", [16, 48])
def test_batch(monkeypatch, max_n):
    cs = [_circuit(max_n - i, 10 + i, np.pi / 2, i) for i in range(4)]
    got = []
    for v in "01":
        monkeypatch.setenv("QIMAX_MERGE_FREE", v)
        with Batch(precision=32, max_n=max_n) as b:
            ids = [b.submit(c) for c in cs]
            b.run()
            got.append(([b.circuit_updates(i) for i in ids], [x for i in ids for x in b.fetch(i)]))
    assert got[0][0] == got[1][0]
    for x, y in zip(got[0][1], got[1][1]):
        assert np.array_equal(x, y)


def test_ordinary_angles_stay_unsorted(monkeypatch):
    """Random angles are far from vanishing: the passes before the last are not sorted."""
    c = W.c2_clifford_rz(5, 32, 120, 24)
    for precision in (64, 32):
        (_, s0), (_, s1) = (_run(monkeypatch, v, c, precision) for v in "01")
        assert s1["sort_elems"] < s0["sort_elems"]
