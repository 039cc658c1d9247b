"""Long Clifford chains compiled into tables, against the stabilizer tableau: chain lengths
around the table minimum, the run length and one and two levels of joins, on every key class
and at its first and last qubit counts."""
import numpy as np
import pytest

from _keys import xz_to_index
from _tableau import Tableau
from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Batch, Simulator

pytestmark = pytest.mark.gpu

CLIFFORD = list(W.CLIFFORD_1Q) + [W.Gate.CX, W.Gate.CZ, W.Gate.ISWAP]


def _expected(c):
    rows = Tableau(c.n).run(c).rows()
    keys = np.concatenate([xz_to_index(np.array([x], np.uint64), np.array([z], np.uint64), c.n) for x, z, _ in rows])
    return keys, np.array([s for _, _, s in rows])


def _check(got, c):
    off, keys, w = got
    rk, rw = _expected(c)
    assert np.array_equal(off, np.arange(c.n + 1))
    assert np.array_equal(keys.reshape(rk.shape), rk)
    assert np.array_equal(w, rw)


@pytest.mark.parametrize("n", [2, 16, 17, 32, 33, 48, 64])
@pytest.mark.parametrize("m", [12, 40, 190, 400, 6000])
def test_chain_lengths(n, m):
    c = W.random_circuit(m + n, n, m, gates=CLIFFORD)
    with Simulator(n) as s:
        _check(s.run(c).generators(), c)


@pytest.mark.parametrize("n", [13, 29, 61])
def test_two_levels_of_joins(n):
    c = W.random_circuit(n, n, 130_000, gates=CLIFFORD)  # more than 24 * 24 * 128 operators
    with Simulator(n) as s:
        assert s.group_counts(c)[0] > 24 * 24 * 128
        _check(s.run(c).generators(), c)


@pytest.mark.parametrize("n", [16, 32, 64])
def test_chains_of_a_batch(n):
    cs = [W.random_circuit(7 + i, n - i, 5000 * i + 30, gates=CLIFFORD) for i in range(3)]
    with Batch(max_n=n) as b:
        ids = [b.submit(c) for c in cs]
        b.run()
        for cid, c in zip(ids, cs):
            _check(b.fetch(cid), c)


@pytest.mark.parametrize("n", [32, 64])
def test_memory_cap_without_room_for_the_scratch(n):
    """The chain's joins take device scratch that the cap may not leave: the result is the same
    (one run per chain, or the ops one by one)."""
    c = W.random_circuit(5, n, 60_000, gates=CLIFFORD)
    with Simulator(n) as s:
        s.run(c).flush()
        full = s.stats()["alloc_bytes"]
    for spare in (1_500_000, 3_000_000):
        with Simulator(n, mem_cap_bytes=full - spare) as s:
            _check(s.run(c).generators(), c)
