"""Expectation values from the device statevector around the sizes where its work is laid out
differently (amplitudes per block, state in LDS, parts per generator, strings per launch)
against dense statevectors."""
import numpy as np
import pytest

from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Simulator

import _dense as D

pytestmark = pytest.mark.gpu


def _pauli(v, s):
    n = len(s)
    u = v.reshape((2,) * n)
    for q, ch in enumerate(s):
        if ch == "I":
            continue
        m = {"X": np.array([[0, 1], [1, 0]]), "Y": np.array([[0, -1j], [1j, 0]]), "Z": np.diag([1, -1])}[ch]
        u = np.moveaxis(np.tensordot(m, u, axes=(1, q)), 0, q)
    return float(np.vdot(v, u.reshape(-1)).real)


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n,layers", [(1, 1), (2, 2), (5, 3), (9, 2), (10, 2), (11, 2), (12, 1), (13, 1), (14, 1), (15, 1)])
def test_expectations(n, layers, precision):
    c = W.c3_hea(n, n, layers, eps=0.0)
    v = D.statevector(c)
    rng = np.random.default_rng(n)
    strings = ["".join(rng.choice(list("IXYZ"), n)) for _ in range(40)]
    strings += ["I" * q + "Z" + "I" * (n - q - 1) for q in range(n)]
    want = np.array([_pauli(v, s) for s in strings])
    with Simulator(n, precision=precision) as s:
        s.run(c)
        got, p0 = s.expect_many(strings), s.prob_zero_all()
        one = s.expect(strings[3])
    # the generators hold to about 1e-15 (FP64) or 1e-6 (FP32) per projection, n of them
    tol = n * (1e-14 if precision == 64 else 2e-6)
    assert np.max(np.abs(got - want)) <= tol
    assert np.max(np.abs(p0 - 0.5 * (1 + want[40:]))) <= tol
    assert abs(one - got[3]) <= 1e-13


def test_many_strings_and_a_memory_cap():
    n = 6
    c = W.c3_hea(3, n, 2, eps=0.0)
    rng = np.random.default_rng(5)
    strings = ["".join(rng.choice(list("IXYZ"), n)) for _ in range(20000)]
    with Simulator(n) as s:
        s.run(c)
        a = s.expect_many(strings)
        cap = s.stats()["alloc_bytes"]
    v = D.statevector(c)
    for i in (0, 1, 16383, 16384, 19999):
        assert abs(a[i] - _pauli(v, strings[i])) <= n * 1e-14
    with Simulator(n, mem_cap_bytes=cap) as s:  # fewer strings at a time
        s.run(c)
        assert np.max(np.abs(s.expect_many(strings) - a)) <= 1e-13


@pytest.mark.parametrize("n", [6, 8, 12])
def test_generators_of_many_terms(n):
    """Terms over one group of a block's waves and over four (16384 terms and more), amplitudes in
    LDS and not: generators below, near and past the line in one state."""
    c = W.random_circuit(3 * n, n, 330)
    v = D.statevector(c)
    rng = np.random.default_rng(n)
    strings = ["".join(rng.choice(list("IXYZ"), n)) for _ in range(20)]
    want = np.array([_pauli(v, s) for s in strings])
    with Simulator(n) as s:
        s.run(c)
        print("[expect] terms per generator", np.diff(s.generators()[0]), flush=True)
        got = s.expect_many(strings)
    assert np.max(np.abs(got - want)) <= n * 1e-14
