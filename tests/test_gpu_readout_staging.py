"""The pinned staging that readouts go through: without it they give the same results."""
import numpy as np
import pytest

from _keys import xz_to_index
from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Batch, Simulator

pytestmark = pytest.mark.gpu


def _readouts(c, precision):
    """Two readouts of either form, and a batch's result."""
    with Simulator(c.n, precision=precision, prune_eps=c.eps) as s:
        s.run(c)
        out = [s.generators(), s.generators_xz(), s.generators(), s.generators_xz()]
    with Batch(precision=precision, max_n=c.n) as b:
        i, j = b.submit(c), b.submit(c)
        b.run()
        return out + [b.fetch(i), b.fetch(j)]


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n", [1, 9, 16, 17, 32, 33, 64])
def test_without_staging(monkeypatch, n, precision):
    c = W.c2_clifford_rz(3, n, 50, 10)
    want = _readouts(c, precision)
    off, x, z, w = want[1]
    assert np.array_equal(xz_to_index(x, z, n), want[0][1]) and np.array_equal(w, want[0][2])
    for k in (1, 2, 3, 100):  # the first k readouts find none, the next ones do
        monkeypatch.setenv("QIMAX_FAIL_READS", str(k))
        got = _readouts(c, precision)
        monkeypatch.delenv("QIMAX_FAIL_READS")
        for a, b in zip(got, want):
            for p, q in zip(a, b):
                assert np.array_equal(p, q)
