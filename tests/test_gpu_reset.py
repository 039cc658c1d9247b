"""A reset after the terms have shrunk to fewer than the generators, by pruning, in buffers that were
sized for those few: the generators of the start, and a circuit run from them."""
import numpy as np
import pytest

from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Simulator

pytestmark = pytest.mark.gpu


def _pair(t):
    """exp(-i t XX / 2) as a PTM, order I, X, Y, Z."""
    x, i2 = np.array([[0, 1], [1, 0]]), np.eye(4)
    u = np.cos(t / 2) * i2 - 1j * np.sin(t / 2) * np.kron(x, x)
    p = [np.eye(2), x, np.array([[0, -1j], [1j, 0]]), np.diag([1, -1])]
    b = [np.kron(a, c) for a in p for c in p]
    return np.array([[np.trace(a @ u @ c @ u.conj().T).real / 4 for c in b] for a in b])


@pytest.mark.parametrize("env", [{}, {"QIMAX_SMALL_GROUPS": "0"}, {"QIMAX_SMALL_ROUNDS": "0"}, {"QIMAX_SORT_CLASSIC": "1"}])
@pytest.mark.parametrize("keep", [0, 1, 3])
@pytest.mark.parametrize("n,precision", [(16, 32), (20, 64), (64, 64), (64, 32)])
def test_reset_after_pruning(monkeypatch, n, precision, keep, env):
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    turn = np.array([[1, 0, 0, 0], [0, 1, 0, 0], [0, 0, np.cos(1.2), -np.sin(1.2)], [0, 0, np.sin(1.2), np.cos(1.2)]])
    c = W.c2_clifford_rz(3, n, 30, 6)
    with Simulator(n, precision=precision) as s:
        want = s.run(c).generators()
    with Simulator(n, precision=precision, prune_eps=0.95) as s:
        for rep in range(3):
            # weights of cos 1.2 and sin 1.2 go; `keep` generators are not turned
            s.apply_layer([(q, turn) for q in range(keep, n)])
            assert s.num_terms() <= keep
            for _ in range(2):  # several passes a call, each in another of the buffers
                s.apply_layer([((0, 1), _pair(0.1)), ((1, 2), _pair(0.1)), ((0, 2), _pair(0.1))][:2 + rep % 2])
            s.reset()
            off, keys, w = s.generators()
            assert np.array_equal(off, np.arange(n + 1)) and np.all(w == 1.0)
    with Simulator(n, precision=precision) as s:
        s.apply_layer([(0, turn)])
        s.reset()
        got = s.run(c).generators()
    for x, y in zip(got, want):
        assert np.array_equal(x, y)
