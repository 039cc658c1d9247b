"""The chunk-local sort's plan where a key's top digit is partial (2n not a multiple of 8) and
where circuits of a batch have keys of different width: the same terms bit for bit as sorting by
global passes over every digit."""
from __future__ import annotations

import sys

import numpy as np
import pytest

import oracle
from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Batch, Simulator

from _compare import compare_fp64, oracle_arrays

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n", [9, 10, 11])
def test_partial_top_digit(monkeypatch, n, precision):
    c = W.random_layered(40 + n, n, layers=3, gates_per_layer=100)
    print("[sort plan]", n, precision, file=sys.stderr, flush=True)
    got = []
    for local in ("1", "0"):
        monkeypatch.setenv("QIMAX_LOCAL_SORT", local)
        with Simulator(c.n, prune_eps=c.eps, precision=precision) as s:
            s.run(c)
            s.reset()
            s.run(c)
            got.append(s.generators())
            print("  terms", int(got[-1][0][-1]), "redos", s.stats()["sort_redos"], file=sys.stderr, flush=True)
    for x, y in zip(*got):
        assert np.array_equal(x, y)


def test_keys_of_different_width(monkeypatch):
    """(Segments past a block's size, the narrower keys in the larger segments.)"""
    cs = [W.c2_clifford_rz(seed=s, n=n, depth=120, n_rz=k) for s, (n, k) in enumerate([(35, 22), (43, 10), (38, 20)])]
    got = []
    for local in ("1", "0"):
        monkeypatch.setenv("QIMAX_LOCAL_SORT", local)
        with Batch(max_n=43) as b:
            ids = [b.submit(c) for c in cs]
            b.run()
            got.append([b.fetch(i) for i in ids])
    print("[sort plan] terms", [int(g[0][-1]) for g in got[0]], file=sys.stderr, flush=True)
    for x, y in zip(*got):
        for p, q in zip(x, y):
            assert np.array_equal(p, q)


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n,local", [(6, "1"), (12, "1"), (12, "0"), (20, "0"), (40, "0"), (40, "1")])
def test_sort_tiles(monkeypatch, n, local, precision):
    """Tiles of 1024 and 4096 elements, every key size, global passes and chunks: the same terms
    bit for bit, and the oracle's."""
    c = W.random_circuit(50 + n, n, 260) if n < 16 else W.c2_clifford_rz(seed=n, n=n, depth=120, n_rz=22)
    print("[sort plan] tiles", n, local, precision, file=sys.stderr, flush=True)
    monkeypatch.setenv("QIMAX_LOCAL_SORT", local)
    monkeypatch.setenv("QIMAX_SMALL_ROUNDS", "0")
    monkeypatch.setenv("QIMAX_MERGE_FREE", "0")
    got = []
    for tile in ("1024", "4096", ""):
        monkeypatch.setenv("QIMAX_SORT_TILE", tile)
        with Simulator(c.n, prune_eps=c.eps, precision=precision) as s:
            s.run(c)
            got.append(s.generators())
    for g in got[1:]:
        for x, y in zip(got[0], g):
            assert np.array_equal(x, y)
    if precision == 64:
        compare_fp64(got[0], oracle_arrays(oracle.propagate(c), c.n), label=c.name)
