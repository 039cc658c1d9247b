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


PATHS = {"groups": {}, "small rounds": {"QIMAX_SMALL_GROUPS": "0"}, "rounds": {"QIMAX_SMALL_ROUNDS": "0"}}


def _run(monkeypatch, value, c, precision, path="groups"):
    monkeypatch.setenv("QIMAX_MERGE_FREE", value)
    for k, v in PATHS[path].items():
        monkeypatch.setenv(k, v)
    with Simulator(c.n, precision=precision) as s:
        s.run(c)
        return s.generators(), s.stats()


@pytest.mark.parametrize("path", sorted(PATHS))
@pytest.mark.parametrize("n", [16, 32, 48])
@pytest.mark.parametrize("k,theta,precision", [(16, np.pi / 2, 32), (16, np.pi, 32), (12, 1e-12, 32), (12, 2e-38, 32),
                                               (16, 1e-25, 64), (12, 1e-300, 64)])
def test_products_that_vanish(monkeypatch, n, k, theta, precision, path):
    c = _circuit(n, k, theta)
    (g0, s0), (g1, s1) = (_run(monkeypatch, v, c, precision, path) for v in "01")
    for x, y in zip(g0, g1):
        assert np.array_equal(x, y)
    for key in ("images", "term_updates", "terms", "rounds"):
        assert s0[key] == s1[key], key


@pytest.mark.parametrize("spins", ["0", "64"])
@pytest.mark.parametrize("path", sorted(PATHS))
@pytest.mark.parametrize("max_n", [16, 32, 48])
def test_batch(monkeypatch, max_n, path, spins):
    monkeypatch.setenv("QIMAX_DEFER_SPINS", spins)
    for k, v in PATHS[path].items():
        monkeypatch.setenv(k, v)
    cs = [_circuit(max_n - i, 10 + i, np.pi / 2, i) for i in range(4)] + [W.c2_clifford_rz(7, max_n, 60, 12)]
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


def test_a_recorded_step(monkeypatch):
    """A recording of rounds that are run again, replayed."""
    monkeypatch.setenv("QIMAX_SMALL_ROUNDS", "0")
    c = _circuit(20, 12, np.pi / 2)
    with Simulator(20, precision=32) as s:
        s.run(c).flush()
        want = s.generators()
        with s.record_step(c) as g:
            for _ in range(3):
                s.reset()
                g.launch()
                s.sync()
                for x, y in zip(s.generators(), want):
                    assert np.array_equal(x, y)


def test_ordinary_angles_stay_unsorted(monkeypatch):
    """Random angles are far from vanishing: the passes before the last are not sorted."""
    c = W.c2_clifford_rz(5, 32, 120, 24)
    for precision in (64, 32):
        (_, s0), (_, s1) = (_run(monkeypatch, v, c, precision) for v in "01")
        assert s1["sort_elems"] < s0["sort_elems"]
