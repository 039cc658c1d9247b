"""Batch.run takes several small passes of every circuit in one launch; Batch.step takes one.
Both give the same terms bit for bit, the same updates, and leave the array empty."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Batch

pytestmark = pytest.mark.gpu


def circuits(kind):
    if kind == "16":  # passes of different numbers; pruned segments; a circuit without operators
        return [W.c2_clifford_rz(seed=s, n=5 + s, depth=20 + 9 * s, n_rz=k) for s, k in enumerate([1, 2, 7, 9])] + \
               [W.c3_hea(seed=2, n=4, layers=3, eps=1e-2), W.random_circuit(3, 6, 0)]
    if kind == "32":
        return [W.c2_clifford_rz(seed=s, n=32 - 3 * s, depth=60, n_rz=4 * s + 1) for s in range(4)]
    if kind == "64":
        return [W.c2_clifford_rz(seed=s, n=64 - 15 * s, depth=40, n_rz=3 * s + 1) for s in range(4)]
    # more segments than a group takes, and just as many
    n = {"segs256": 16, "segs272": 17}[kind]
    return [W.c2_clifford_rz(seed=s, n=16, depth=30, n_rz=3) for s in range(n)]


@pytest.mark.parametrize("kind,precision,cap", [("16", 64, 0), ("16", 32, 0), ("32", 64, 0), ("64", 64, 0), ("64", 32, 0),
                                                ("segs256", 64, 0), ("segs272", 64, 0), ("32", 64, 64 << 20)])
def test_run_equals_steps(kind, precision, cap):
    cs = circuits(kind)
    max_n = max(c.n for c in cs)
    print("[batch groups]", kind, precision, cap, len(cs), file=sys.stderr, flush=True)
    opts = {"mem_cap_bytes": cap} if cap else {}
    with Batch(precision=precision, max_n=max_n, **opts) as a, Batch(precision=precision, max_n=max_n, **opts) as b:
        for rep in range(2):  # (new circuits, then the same again in the buffers that are there)
            ia, ib = [a.submit(c) for c in cs], [b.submit(c) for c in cs]
            a.run()
            while b.step():
                pass
            assert set(a.poll()) == set(ia)
            for c, x, y in zip(cs, ia, ib):
                for p, q in zip(a.fetch(x), b.fetch(y)):
                    assert np.array_equal(p, q), (c.name, rep)
            ja, jb = a.info(), b.info()
            for k in ("active", "queued", "terms"):
                assert ja[k] == jb[k] == 0
            assert ja["rounds"] == jb["rounds"]
