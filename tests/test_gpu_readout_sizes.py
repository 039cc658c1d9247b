"""The readout in one slot, in a few chunks and in more chunks than slots, around the sizes
where that changes: every form against the others and against the terms' own invariants."""
import numpy as np
import pytest

from _keys import xz_to_index
from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Batch, Simulator

pytestmark = pytest.mark.gpu


def _tensor_circuit(n, digits):
    """X strings spread over `digits` qubits: generator 0 ends with 2^digits terms (Rz on every
    one of them after a CX fan-out of an X)."""
    g = [W.Gate.H] + [W.Gate.CX] * digits
    q0, q1 = [0] + [0] * digits, [0] + list(range(1, digits + 1))
    g += [W.Gate.RZ] * digits
    q0 += list(range(1, digits + 1))
    q1 += list(range(1, digits + 1))
    th = [0.0] * (1 + digits) + [0.3 + 0.01 * k for k in range(digits)]
    return W.Circuit(n, np.array(g, np.uint8), np.array(q0, np.uint32), np.array(q1, np.uint32), np.array(th),
                     np.array([len(g)], np.int64), 0.0, f"spread(n={n},k={digits})")


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n,digits", [(16, 3), (16, 15), (17, 16), (32, 16), (33, 17), (64, 17), (24, 20), (40, 21)])
def test_sizes(n, digits, precision):
    c = _tensor_circuit(n, digits)
    with Simulator(n, precision=precision) as s:
        s.run(c)
        off, keys, w = s.generators()
        off2, x, z, w2 = s.generators_xz()
        again = s.generators()
    assert int(off[1]) == 2 ** digits and np.array_equal(off, off2)
    assert np.array_equal(xz_to_index(x, z, n), keys) and np.array_equal(w, w2)
    assert all(np.array_equal(a, b) for a, b in zip(again, (off, keys, w)))
    a, b = int(off[0]), int(off[1])
    # every qubit 1..digits holds X or Y, so each term's weight is a product of cosines and sines
    t = c.theta[1 + digits:]
    expect = np.ones(1)
    for q in range(digits):
        expect = np.concatenate([expect * np.cos(t[q]), expect * np.sin(t[q])])
    code = np.zeros(b - a, dtype=np.int64)
    for q in range(1, digits + 1):  # Y on qubit q: the sine was taken
        code |= (((x[a:b] & z[a:b]) >> np.uint64(q)) & np.uint64(1)).astype(np.int64) << (q - 1)
    assert np.array_equal(np.sort(code), np.arange(2 ** digits))
    tol = digits * (2.0 ** -52 if precision == 64 else 2.0 ** -22)
    assert np.max(np.abs(np.abs(w[a:b]) - np.abs(expect[code]))) <= tol
    if precision == 64 and n <= 32:
        with Batch(max_n=n) as bt:
            i = bt.submit(c)
            bt.run()
            assert all(np.array_equal(p, q) for p, q in zip(bt.fetch(i), (off, keys, w)))
