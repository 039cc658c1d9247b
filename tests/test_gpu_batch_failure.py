"""A batch call that fails for want of memory leaves the batch usable: the same call made again
goes on where it failed, and every circuit's terms are those of a run without the failure."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Batch, QimaxError, Simulator

pytestmark = pytest.mark.gpu


def _alone(c, precision):
    with Simulator(c.n, precision=precision, prune_eps=c.eps) as s:
        return s.run(c).generators()


@pytest.mark.parametrize("how", ["run", "step"])
@pytest.mark.parametrize("max_n,precision", [(16, 64), (16, 32), (32, 64), (64, 64)])
@pytest.mark.parametrize("k", [1, 2, 4])
def test_result_without_host_memory(monkeypatch, k, max_n, precision, how):
    """The k-th result finds no host memory: circuits that finish at the same pass as it, later
    than it (with passes of theirs behind them in the same round) and before it."""
    cs = [W.c2_clifford_rz(seed=s, n=max_n - 2 * s, depth=30, n_rz=rz) for s, rz in enumerate([2, 9, 2, 6])]
    want = [_alone(c, precision) for c in cs]
    monkeypatch.setenv("QIMAX_FAIL_RESULT", str(k))
    print("[batch failure]", how, max_n, precision, k, file=sys.stderr, flush=True)
    with Batch(precision=precision, max_n=max_n) as b:
        ids = [b.submit(c) for c in cs]
        done, failed = [], 0
        for _ in range(100):
            try:
                left = b.run() if how == "run" else b.step()
            except QimaxError as e:
                assert e.status == -2
                failed += 1
                done += b.poll()
                assert len(done) == k - 1 and b.info()["active"] == len(cs) - len(done)
                for i in ids:
                    if i not in done:
                        with pytest.raises(QimaxError, match="ESTATE"):
                            b.fetch(i)
                continue
            if how == "run" or not left:
                break
        done += b.poll()
        assert failed == 1 and sorted(done) == sorted(ids)
        for i, w in zip(ids, want):
            for x, y in zip(b.fetch(i), w):
                assert np.array_equal(x, y)
        info = b.info()
        assert info["active"] == info["queued"] == info["terms"] == 0


def _circuits(max_n):
    """Several of them small (they advance in groups of passes), with chains long enough for
    tables, and one whose last passes are rounds."""
    return [W.c2_clifford_rz(seed=s, n=max_n - s, depth=60, n_rz=rz) for s, rz in enumerate([3, 5, 14, 4])]


@pytest.mark.parametrize("how", ["run", "step"])
@pytest.mark.parametrize("max_n,precision", [(16, 32), (32, 64), (64, 64)])
@pytest.mark.parametrize("m", [1, 3])
def test_device_allocation_fails(monkeypatch, m, max_n, precision, how):
    """m device allocations from the k-th on fail, for every k: the call falls back on another way,
    or is refused and made again."""
    cs = _circuits(max_n)
    want = [_alone(c, precision) for c in cs]
    print("[batch failure]", how, max_n, precision, m, file=sys.stderr, flush=True)
    refused = 0
    for k in range(5, 100):
        monkeypatch.setenv("QIMAX_FAIL_ALLOC", f"{k}:{m}")
        with Batch(precision=precision, max_n=max_n) as b:
            monkeypatch.delenv("QIMAX_FAIL_ALLOC")
            ids = [b.submit(c) for c in cs]
            for _ in range(200):
                try:
                    if how == "run":
                        b.run()
                        break
                    if not b.step():
                        break
                except QimaxError as e:
                    assert e.status == -2
                    refused += 1
            for i, w in zip(ids, want):
                for x, y in zip(b.fetch(i), w):
                    assert np.array_equal(x, y), k
    assert refused <= m * 95
