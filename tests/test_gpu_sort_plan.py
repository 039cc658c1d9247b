"""The chunk-local sort's plan where a key's top digit is partial (2n not a multiple of 8) and
where circuits of a batch have keys of different width: the same terms bit for bit as sorting by
global passes over every digit."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Batch, Simulator

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n", [9, 10, 11, 13])
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
