"""Rounds of more images than a round can have, or than memory holds, are refused before anything
that grows with them is allocated, and leave the state as it was."""
import numpy as np
import pytest

from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import QimaxError, Simulator

pytestmark = pytest.mark.gpu

G = W.Gate
TOO_LARGE, NO_MEMORY = -4, -2


def _apply(s, gates):
    g, a, b, t = zip(*gates)
    s.apply_circuit((np.array(g, np.uint8), np.array(a, np.uint32), np.array(b, np.uint32), np.array(t)))


# 2^k strings with an X or Y on every wire, apart on the last k wires; then a rotation of every wire: 3^19
# outputs for each of them in the first pass (a pass's fan-out is below 2^31)
@pytest.mark.parametrize("n,k,cap,status", [(32, 13, 0, TOO_LARGE), (64, 12, 0, TOO_LARGE), (30, 10, 40 << 30, NO_MEMORY),
                                            (32, 13, 1 << 30, TOO_LARGE), (40, 9, 1 << 30, NO_MEMORY)])
@pytest.mark.parametrize("gather", ["1", "0"])
def test_rotations_of_every_wire(monkeypatch, gather, n, k, cap, status):
    monkeypatch.setenv("QIMAX_GATHER", gather)
    with Simulator(n, mem_cap_bytes=cap) as s:
        _apply(s, [(G.H, 0, 0, 0.0)] + [(G.CX, i, i + 1, 0.0) for i in range(n - 1)] +
               [(G.RZ, q, q, 0.3 + 0.01 * q) for q in range(n - k, n)])
        s.flush()
        want = s.generators()
        assert int(want[0][1]) == 2 ** k
        before = s.stats()["peak_bytes"]
        print("[huge rounds]", n, k, cap, gather, flush=True)
        with pytest.raises(QimaxError) as e:
            _apply(s, [(g, q, q, 0.4 + 0.1 * i) for q in range(n) for i, g in enumerate((G.RX, G.RY, G.RZ))])
        assert e.value.status == status
        assert s.stats()["peak_bytes"] - before < 64 << 20
        for x, y in zip(s.generators(), want):
            assert np.array_equal(x, y)
