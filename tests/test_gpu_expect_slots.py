"""The statevector's place during its projections: it changes with every generator of a few terms and
stays for those whose terms are dealt over several parts, in whatever order they come."""
import numpy as np
import pytest

from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Simulator

import _dense as D
from test_gpu_expect_sizes import _pauli

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [False, True])
@pytest.mark.parametrize("n,m", [(5, 8), (6, 8), (8, 9), (9, 9), (10, 9), (12, 6), (13, 6)])
def test_generators_of_few_and_many_terms(n, m, cap):
    seen = set()
    for seed in range(6 if n <= 10 else 2):
        c = W.random_circuit(40 * n + seed, n, m * n)
        v = D.statevector(c)
        rng = np.random.default_rng(seed)
        strings = ["".join(rng.choice(list("IXYZ"), n)) for _ in range(20)]
        want = np.array([_pauli(v, s) for s in strings])
        z = np.array([_pauli(v, "I" * q + "Z" + "I" * (n - q - 1)) for q in range(n)])
        with Simulator(n) as s:
            s.run(c).flush()
            held, terms = s.stats()["alloc_bytes"], s.num_terms()
        with Simulator(n, mem_cap_bytes=held + 2 * (16 << n) + 32 * terms + 512 if cap else 0) as s:
            s.run(c)
            sizes = np.diff(s.generators()[0].astype(np.int64))
            got, p0 = s.expect_many(strings), s.prob_zero_all()
        assert np.max(np.abs(got - want)) <= n * 1e-14
        assert np.max(np.abs(p0 - 0.5 * (1 + z))) <= n * 1e-14
        at = 0  # the slot in which each generator finds the state: parts of 16 terms, as many as fit
        for t in sizes:
            parts = min((t + 15) // 16, max(1, 2 * terms >> n))
            seen.add((at, bool(parts > 1)))
            at ^= parts <= 1
    assert len(seen) == 4 or n > 10
