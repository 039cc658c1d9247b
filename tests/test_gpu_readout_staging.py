"""The pinned staging that readouts go through: without it they give the same results; it is shared
by the contexts of a process, whatever their number, and by its threads."""
import threading

import numpy as np
import pytest

from _keys import xz_to_index
from test_gpu_readout_sizes import _tensor_circuit
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


def _mapped_kb():
    with open("/proc/self/status") as f:
        return next(int(line.split()[1]) for line in f if line.startswith("VmSize"))


def test_contexts_share_it():
    """Long readouts (2^21 terms: all sixteen slots) of ten contexts that stay open."""
    c = _tensor_circuit(24, 21)
    sims = [Simulator(24).run(c) for _ in range(10)]
    try:
        grown, want = [], None
        for s in sims:
            a = _mapped_kb()
            got = s.generators()
            want = want or got
            assert all(np.array_equal(x, y) for x, y in zip(got, want))
            del got
            grown.append(_mapped_kb() - a)
        # after the first two (threads, the arrays compared with) no context adds its own 32 MB
        assert sum(grown[2:]) < 40 << 10, grown
    finally:
        for s in sims:
            s.close()


def test_threads_read_at_once():
    """Readouts of several sizes on four threads, contexts opened and closed between them."""
    cs = [_tensor_circuit(16, 4), _tensor_circuit(17, 15), _tensor_circuit(33, 16), _tensor_circuit(24, 20)]
    want = []
    for c in cs:
        with Simulator(c.n) as s:
            want.append(s.run(c).generators())
    bad = []

    def work(k):
        for rep in range(6):
            i = (k + rep) % len(cs)
            with Simulator(cs[i].n) as s:
                s.run(cs[i])
                for _ in range(3):
                    if not all(np.array_equal(x, y) for x, y in zip(s.generators(), want[i])):
                        bad.append((k, rep, i))
    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
