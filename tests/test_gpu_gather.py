"""Rounds of large fan-out merge before they expand: the results are those of expanding,
sorting and merging every image, bit for bit, over operators of every block form (and of forms
that are not gathered), chains before and after them, key classes, weights and thresholds."""
import numpy as np
import pytest

from _compare import compare_fp64, oracle_arrays
import oracle
from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Batch, Simulator

pytestmark = pytest.mark.gpu


def _both(monkeypatch, make, **env):
    out = []
    for v in "01":
        monkeypatch.setenv("QIMAX_GATHER", v)
        for k, x in env.items():
            monkeypatch.setenv(k, x)
        out.append(make())
        for k in ("QIMAX_GATHER", *env):
            monkeypatch.delenv(k)
    return out


def _same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("eps", [0.0, 1e-3])
@pytest.mark.parametrize("precision,merge", [(64, 0), (32, 0), (32, 1)])
@pytest.mark.parametrize("n,layers", [(3, 1), (3, 6), (5, 4), (6, 3), (7, 3), (9, 2), (11, 2), (13, 2)])
def test_ansatz(monkeypatch, n, layers, precision, merge, eps):
    c = W.c3_hea(n, n, layers, eps)

    def make():
        with Simulator(n, precision=precision, fp32_merge=merge, prune_eps=eps) as s:
            s.run(c)
            return s.generators(), s.stats()
    (g0, s0), (g1, s1) = _both(monkeypatch, make)
    _same(g0, g1)
    for k in ("term_updates", "images", "passes", "rounds", "terms"):
        assert s0[k] == s1[k]
    if eps == 0.0 and precision == 64:
        compare_fp64(g1, oracle_arrays(oracle.propagate(c), n))


@pytest.mark.parametrize("env", [{"QIMAX_LOCAL_SORT": "0"}, {"QIMAX_LOCAL_SORT_M": "1"}, {"QIMAX_LOCAL_SORT_M": "2"},
                                 {"QIMAX_CLASSIC_PASSES": "1"}, {"QIMAX_AUTOTUNE": "0"}, {"QIMAX_XCD_RANGES": "0"}])
def test_sort_variants(monkeypatch, env):
    c = W.c3_hea(2, 10, 2, 1e-9)

    def make():
        with Simulator(10, prune_eps=1e-9) as s:
            return s.run(c).generators()
    _same(*_both(monkeypatch, make, **env))


def _rotation(rng, form):
    a = rng.uniform(0.2, 2.8, 3)

    def r(ax, t):
        m = np.eye(4)
        u, v = ax % 3 + 1, (ax % 3 + 1) % 3 + 1
        m[u, u] = m[v, v] = np.cos(t)
        m[v, u], m[u, v] = np.sin(t), -np.sin(t)
        return m
    if form == "generic":
        return r(1, a[0]) @ r(2, a[1]) @ r(3, a[2])
    if form == "axis":  # blocks {I}, {axis}, the other two
        return r(int(rng.integers(1, 4)), a[0])
    if form == "axis then Clifford":  # the lone digit moves, with a sign
        return np.round(r(int(rng.integers(1, 4)), np.pi / 2)) @ r(int(rng.integers(1, 4)), a[0])
    return r(1, a[0]) @ r(2, a[1])  # an entry is zero: no full block


CHAINS = {"none": 0, "ops": 5, "table": 30}


@pytest.mark.parametrize("chain", list(CHAINS))
@pytest.mark.parametrize("form", ["generic", "axis", "axis then Clifford", "zero entry", "mixed"])
@pytest.mark.parametrize("n", [4, 8, 16, 17, 21, 32, 33, 40, 64])
def test_forms(monkeypatch, n, form, chain):
    rng = np.random.default_rng(n * 7 + len(form) + CHAINS[chain])
    forms = ["generic", "axis", "axis then Clifford"] if form == "mixed" else [form]
    parts = []
    for _ in range(3):
        wires = rng.choice(n, size=min(n, 6), replace=False)
        parts.append([(int(q), _rotation(rng, forms[int(rng.integers(len(forms)))])) for q in wires])
    cliff = [W.random_circuit(int(rng.integers(1000)), n, CHAINS[chain] or 1,
                              gates=list(W.CLIFFORD_1Q) + [W.Gate.CX, W.Gate.CZ]) for _ in parts]

    def make():
        with Simulator(n) as s:
            for ops, c in zip(parts, cliff):
                s.apply_layer(ops)
                if CHAINS[chain]:
                    s.apply_circuit(c)
            return s.generators()
    _same(*_both(monkeypatch, make))


@pytest.mark.parametrize("n", [8, 20, 36])
def test_chain_after_the_rotations_in_one_call(monkeypatch, n):
    """B chains of the pass itself: op lists (few operators) and tables."""
    for k, seed in ((2, 1), (9, 2), (60, 3)):
        rng = np.random.default_rng(seed)
        ops = [(int(q), _rotation(rng, "generic")) for q in range(6)]
        c = W.random_circuit(seed, n, k, gates=[W.Gate.H, W.Gate.S, W.Gate.CX])
        more = [(int(q), _rotation(rng, "axis")) for q in range(6)]

        def make():
            with Simulator(n) as s:
                cl = s.group(c)[0]
                return s.apply_layer(ops + cl + more + cl + ops).generators()
        _same(*_both(monkeypatch, make))


@pytest.mark.parametrize("max_n", [16, 32, 64])
def test_batch_and_replay(monkeypatch, max_n):
    cs = [W.c3_hea(i, 5 + i, 1 + i % 3, 1e-9) for i in range(5)] + [W.c2_clifford_rz(1, 12, 40, 8)]

    def make():
        with Batch(max_n=max_n) as b:
            ids = [b.submit(c) for c in cs]
            b.run()
            got = [b.fetch(i) for i in ids]
        with Simulator(9, prune_eps=1e-9) as s:
            g = s.record_step(W.c3_hea(4, 9, 2, 1e-9))
            for _ in range(3):
                s.reset()
                s.run(W.c3_hea(5, 9, 1)).sync()
                g.launch()
            got.append(s.generators())
            g.close()
        return got
    for x, y in zip(*_both(monkeypatch, make)):
        _same(x, y)


def test_segments_too_large_to_group(monkeypatch):
    """Generators above what a block groups take the general path (n = 8, saturated)."""
    c = W.c3_hea(1, 8, 3, 1e-9)
    d = W.Circuit(8, c.gate[:3 * 3], c.q0[:9], c.q1[:9], c.theta[:9], np.array([9]), 1e-9)

    def make():
        with Simulator(8, prune_eps=1e-9) as s:
            s.run(c)
            assert s.num_terms() > 8 * 16384
            return s.run(d).generators()
    _same(*_both(monkeypatch, make))


@pytest.mark.parametrize("n,weight", [(10, 1), (10, 6), (10, 7), (10, 8), (17, 8), (33, 6), (33, 7), (64, 7)])
def test_first_layer_of_single_strings(monkeypatch, n, weight):
    """A rotation of every wire while every generator is one string: strings whose images fit a
    block's capacity (3^7 for the shorter keys, 3^6 for 16-byte ones) go through it in one
    launch, heavier ones through a round."""
    rng = np.random.default_rng(n + weight)
    spread = W.Circuit(n, np.full(weight - 1, W.Gate.CX, np.uint8), np.zeros(weight - 1, np.uint32),
                       np.arange(1, weight, dtype=np.uint32), np.zeros(weight - 1), np.array([weight - 1]), 0.0)
    ops = [(q, _rotation(rng, "generic")) for q in range(min(n, 12))]

    def make():
        with Simulator(n) as s:
            if weight > 1:
                s.apply_circuit((np.array([W.Gate.H], np.uint8), np.zeros(1, np.uint32), np.zeros(1, np.uint32), np.zeros(1)))
                s.apply_circuit(spread)
            s.apply_layer(ops)
            st = s.stats()
            return (*s.generators(), np.array([st["images"], st["term_updates"], st["rounds"]]))
    g = [_both(monkeypatch, make, QIMAX_SMALL_GROUPS=v) for v in "01"]
    for x in (g[0][1], g[1][0], g[1][1]):
        _same(g[0][0], x)


@pytest.mark.parametrize("precision,merge", [(64, 0), (32, 0), (32, 1)])
@pytest.mark.parametrize("n,layers", [(1, 3), (2, 5), (3, 6), (4, 5), (6, 4), (9, 2), (18, 1), (36, 1)])
def test_teams_of_waves(monkeypatch, n, layers, precision, merge):
    """Parents a chunk of the team's, fewer and more; units of one group and of several in a wave."""
    c = W.c3_hea(n, n, layers, 0.0) if n < 16 else W.random_circuit(1, n, 3 * n)
    got = []
    for v in "01":
        monkeypatch.setenv("QIMAX_GATHER_TEAM", v)
        with Simulator(n, precision=precision, fp32_merge=merge) as s:
            got.append(s.run(c).generators())
    _same(*got)
