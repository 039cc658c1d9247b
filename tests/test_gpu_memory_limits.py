"""Calls short of memory: what fits without groups of small passes, gathered rounds, unsorted passes
and small sort tiles fits with them too (they are left out where there is no room), with the
same terms; and a call that is refused, or that had to leave them out, costs later ones nothing."""
import numpy as np
import pytest

from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import QimaxError, Simulator

pytestmark = pytest.mark.gpu

OFF = {"groups": {"QIMAX_SMALL_GROUPS": "0"},
       "all": {"QIMAX_SMALL_GROUPS": "0", "QIMAX_GATHER": "0", "QIMAX_MERGE_FREE": "0", "QIMAX_SORT_TILE": "4096"}}


def _run(c, cap, precision):
    """The generators under the cap, or None where the call is refused for memory."""
    with Simulator(c.n, precision=precision, prune_eps=c.eps, mem_cap_bytes=cap) as s:
        try:
            s.run(c).flush()
        except QimaxError as e:
            assert e.status == -2
            s.sync()
            return None
        assert not cap or s.stats()["peak_bytes"] <= cap
        return s.generators()


def _least_cap(c, precision):
    lo, hi = 1 << 12, 1 << 30
    while hi - lo > max(2048, lo // 64):
        mid = (lo + hi) // 2
        if _run(c, mid, precision) is None:
            lo = mid
        else:
            hi = mid
    return hi


CASES = {"layer16": lambda: W.c3_hea(1, 16, 1), "layer40": lambda: W.c3_hea(1, 40, 1), "layer64": lambda: W.c3_hea(1, 64, 1),
         "ansatz8": lambda: W.c3_hea(1, 8, 2), "rz24": lambda: W.c2_clifford_rz(1, 24, 60, 14),
         "rz48": lambda: W.c2_clifford_rz(1, 48, 60, 12), "one48": lambda: W.c2_clifford_rz(1, 48, 40, 1),
         "graph48": lambda: W.graph_state(1, 48, 20), "graph20": lambda: W.graph_state(1, 20, 60),
         "random9": lambda: W.random_layered(3, 9, 3, 40, 1e-9), "deep5": lambda: W.c3_hea(2, 5, 6)}


@pytest.mark.parametrize("off", sorted(OFF))
@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("case", sorted(CASES))
def test_what_fits_without_fits_with(monkeypatch, case, precision, off):
    c = CASES[case]()
    for k, v in OFF[off].items():
        monkeypatch.setenv(k, v)
    cap = _least_cap(c, precision)
    want = _run(c, cap, precision)
    for k in OFF[off]:
        monkeypatch.delenv(k)
    print("[memory limits]", case, precision, off, cap, flush=True)
    for room in (1.0, 1.05, 1.3, 2.0, 4.0, 16.0):
        got = _run(c, int(cap * room), precision)
        assert got is not None, f"refused with {room} times the memory it needs"
        for x, y in zip(got, want):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("n", [20, 48])
def test_a_refused_call_costs_later_ones_nothing(n):
    """After a call that does not fit, long chains are compiled in parallel runs into tables again."""
    chain = W.graph_state(1, n, 60)
    big = W.c2_clifford_rz(2, n, 400, 40)
    with Simulator(n) as s:
        s.run(chain).flush()
        cap = s.stats()["alloc_bytes"] + (8 << 20)
    with Simulator(n, mem_cap_bytes=cap) as s:
        def launches():
            s.reset()
            s.profile(True)
            s.run(chain).flush()
            s.profile(False)
            return {k: v["launches"] for k, v in s.profile_read().items()}, s.generators()
        first, want = launches()
        assert "chain_tables" in first
        allocated = s.stats()["alloc_bytes"]
        s.reset()
        with pytest.raises(QimaxError, match="ENOMEM"):
            s.run(big)
        s.sync()
        again, got = launches()
        assert again == first and s.stats()["alloc_bytes"] >= allocated * 0.9
        for x, y in zip(got, want):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("n", [20, 48])
def test_a_call_short_of_memory_once(monkeypatch, n):
    """One allocation that fails: that call runs again without tables of 16-byte keys, the calls
    after it have them."""
    c = W.graph_state(2, n, 60)
    monkeypatch.setenv("QIMAX_FAIL_ALLOC", "8")
    with Simulator(n) as s:
        monkeypatch.delenv("QIMAX_FAIL_ALLOC")
        launched, want = [], None
        for _ in range(4):
            s.reset()
            s.profile(True)
            s.run(c).flush()
            s.profile(False)
            launched.append("chain_tables" in s.profile_read())
            got = s.generators()
            want = want or got
            for x, y in zip(got, want):
                assert np.array_equal(x, y)
        assert launched == [n <= 32, True, True, True]


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("case", sorted(CASES))
def test_device_allocation_fails(monkeypatch, case, precision):
    """One, then four device allocations from the k-th on fail, for every k: the terms are those of
    an undisturbed run, where a call is refused once it is made again."""
    c = CASES[case]()
    want = _run(c, 0, precision)
    print("[memory limits]", case, precision, flush=True)
    for m in (1, 4):
        for k in range(5, 75):
            monkeypatch.setenv("QIMAX_FAIL_ALLOC", f"{k}:{m}")
            with Simulator(c.n, precision=precision, prune_eps=c.eps) as s:
                monkeypatch.delenv("QIMAX_FAIL_ALLOC")
                for a, b in c.layers():
                    for _ in range(m + 1):
                        try:
                            s.apply_circuit((c.gate[a:b], c.q0[a:b], c.q1[a:b], c.theta[a:b]))
                            break
                        except QimaxError as e:
                            assert e.status == -2 and m > 1
                for _ in range(m + 1):
                    try:
                        got = s.generators()
                        break
                    except QimaxError as e:
                        assert e.status == -2 and m > 1
                for x, y in zip(got, want):
                    assert np.array_equal(x, y), (m, k)
