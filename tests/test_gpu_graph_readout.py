"""Reading a recorded step's results in any form leaves the recording as it is: expectation values
of many strings between replays, whatever staging they need."""
import numpy as np
import pytest

from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Simulator

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("clifford", [False, True])
def test_replay_after_readouts(clifford):
    n = 10
    c = W.graph_state(3, n, 2) if clifford else W.c3_hea(2, n, 1, 1e-9)
    rng = np.random.default_rng(1)
    with Simulator(n, prune_eps=c.eps) as s:
        for _ in range(12):
            s.reset()
            s.run(c)
            s.flush()
        want = s.generators()
        with s.record_step(c) as g:
            for k in (3, 500, 20000):  # (32 bytes of staging a string)
                strings = ["".join(rng.choice(list("IXYZ"), n)) for _ in range(k)]
                a = np.array(s.expect_many(strings))
                s.prob_zero_all()
                s.generators_xz()
                s.reset()
                g.launch()
                s.sync()
                for x, y in zip(s.generators(), want):
                    assert np.array_equal(x, y)
                assert np.allclose(np.array(s.expect_many(strings)), a, rtol=0, atol=1e-12)
