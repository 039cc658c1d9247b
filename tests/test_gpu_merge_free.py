"""Passes whose images all differ leave them unsorted: the results are those of sorting and
merging every pass, bit for bit, whatever the operators (rotations on independent and on
dependent axes, two-qubit rotations, generic two-qubit operators, maps that are no conjugation),
key class, precision and split into calls; and the rule does apply where the axes are
independent (fewer elements sorted)."""
import numpy as np
import pytest

from _compare import compare_fp64, oracle_arrays
import oracle
from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Batch, Simulator

pytestmark = pytest.mark.gpu


def _with(monkeypatch, value, make, **env):
    monkeypatch.setenv("QIMAX_MERGE_FREE", value)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    r = make()
    monkeypatch.delenv("QIMAX_MERGE_FREE")
    for k in env:
        monkeypatch.delenv(k)
    return r


def _same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def _run(c, precision=64, layers=True):
    with Simulator(c.n, precision=precision, prune_eps=c.eps) as s:
        s.run(c) if layers else s.apply_circuit(c)
        return s.generators(), s.stats()


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n,depth,rz", [(2, 30, 12), (5, 60, 24), (9, 80, 24), (16, 100, 24), (17, 100, 24),
                                        (32, 120, 26), (33, 120, 24), (48, 150, 26), (64, 100, 20)])
def test_clifford_rz(monkeypatch, n, depth, rz, precision):
    c = W.c2_clifford_rz(n, n, depth, rz)
    (g0, s0), (g1, s1) = (_with(monkeypatch, v, lambda: _run(c, precision)) for v in "01")
    _same(g0, g1)
    for k in ("term_updates", "images", "passes", "rounds", "terms"):
        assert s0[k] == s1[k]
    if n >= 32:  # few rotations against 2n key bits: passes before the last stay unsorted
        assert s1["sort_elems"] < s0["sort_elems"]


@pytest.mark.parametrize("groups", ["0", "1"])
@pytest.mark.parametrize("seed", range(6))
def test_full_gate_set(monkeypatch, seed, groups):
    """Two-qubit rotations, angles that merge and axes that become dependent, in layers."""
    n = (4, 7, 9, 18, 34, 40)[seed]
    c = W.random_layered(seed, n, 3, 40 if n > 10 else 50, 0.0, 0.12)
    g0, g1 = (_with(monkeypatch, v, lambda: _run(c)[0], QIMAX_SMALL_GROUPS=groups) for v in "01")
    _same(g0, g1)
    compare_fp64(g1, oracle_arrays(oracle.propagate(c), n))


def _haar(rng, d):
    q, r = np.linalg.qr(rng.normal(size=(d, d)) + 1j * rng.normal(size=(d, d)))
    return q * (np.diag(r) / np.abs(np.diag(r)))


def _ptm(u):
    p = [np.eye(2), np.array([[0, 1], [1, 0]]), np.array([[0, -1j], [1j, 0]]), np.diag([1, -1])]
    d = u.shape[0]
    basis = p if d == 2 else [np.kron(a, b) for a in p for b in p]
    return np.array([[np.trace(a @ u @ b @ u.conj().T).real / d for b in basis] for a in basis])


@pytest.mark.parametrize("n", [6, 20, 36])
def test_generic_operators(monkeypatch, n):
    """Generic one- and two-qubit operators (differences of rank 2 and 4) and a signed
    permutation that is no conjugation, in one call and over several."""
    rng = np.random.default_rng(n)
    reflect = np.diag([1.0, 1.0, 1.0, -1.0])
    u1, u2 = _ptm(_haar(rng, 2)), _ptm(_haar(rng, 4))
    ops = [((0, n - 1), u2), (1, reflect), (1, u1), ((2, 3), u2), (0, u1), ((1, 2), u2), (n - 1, reflect), (3, u1)]

    def make(parts):
        with Simulator(n) as s:
            for p in parts:
                s.apply_layer(p)
            return s.generators()
    for parts in ([ops], [ops[:3], ops[3:]], [[o] for o in ops]):
        _same(_with(monkeypatch, "0", lambda: make(parts)), _with(monkeypatch, "1", lambda: make(parts)))


@pytest.mark.parametrize("max_n", [16, 32, 64])
def test_batch(monkeypatch, max_n):
    cs = [W.c2_clifford_rz(i, max_n - 3 * i, 60 + 20 * i, 14 + i) for i in range(4)]
    cs.append(W.random_layered(3, 6, 3, 30, 1e-7))
    cs.append(W.c2_clifford_rz(9, max_n, 80, 16, layer_per_moment=True))

    def make():
        with Batch(max_n=max_n) as b:
            ids = [b.submit(c) for c in cs]
            b.run()
            return [b.fetch(i) for i in ids]
    for x, y in zip(_with(monkeypatch, "0", make), _with(monkeypatch, "1", make)):
        _same(x, y)


def test_calls_after_a_replay(monkeypatch):
    """A replayed step leaves the state it recorded, the span of its keys included: a circuit
    applied after it (and after a reset in between) merges as it must."""
    c, d = W.c2_clifford_rz(3, 10, 60, 16), W.c2_clifford_rz(4, 10, 60, 14)

    def make():
        with Simulator(10) as s:
            g = s.record_step(c)
            s.reset()
            g.launch()
            s.apply_circuit(d)
            r = s.generators()
            g.close()
            return r
    _same(_with(monkeypatch, "0", make), _with(monkeypatch, "1", make))


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("spins", ["0", "64"])
@pytest.mark.parametrize("sizes", [[(12, 14), (9, 12), (16, 6)], [(30, 12), (21, 5), (18, 13)], [(40, 11), (64, 13), (33, 4)]])
def test_small_rounds(monkeypatch, sizes, spins, precision):
    """Segments that fit a chunk leave it as they come beside others that are sorted, at once and
    deferred: the terms of sorting every pass."""
    cs = [W.c2_clifford_rz(seed=70 + i, n=n, depth=40 + 25 * i, n_rz=k) for i, (n, k) in enumerate(sizes)]
    monkeypatch.setenv("QIMAX_DEFER_SPINS", spins)
    monkeypatch.setenv("QIMAX_SMALL_GROUPS", "0")

    def make():
        with Batch(precision=precision, max_n=max(c.n for c in cs)) as b:
            ids = [b.submit(c) for c in cs]
            while b.step():
                pass
            return [x for i in ids for x in b.fetch(i)]
    got = [_with(monkeypatch, v, make) for v in "01"]
    for x, y in zip(*got):
        assert np.array_equal(x, y)
