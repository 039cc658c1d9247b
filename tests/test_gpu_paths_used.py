"""The paths that the on/off comparisons of the other tests compare are the ones that run: gathered
rounds, groups of small passes, unsorted passes and chain tables, by the kernels launched."""
import pytest

from paper_2505_03307_amd import workloads as W
from paper_2505_03307_amd.qimax import Batch, Simulator

pytestmark = pytest.mark.gpu


def _launched(c, precision=64, **opts):
    with Simulator(c.n, precision=precision, prune_eps=c.eps, **opts) as s:
        s.profile(True)
        s.run(c).flush()
        s.profile(False)
        return {k: v["launches"] for k, v in s.profile_read().items()}, s.stats()


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n,layers", [(5, 4), (6, 3), (7, 3), (9, 2), (11, 2), (13, 2)])
def test_gathered_rounds(monkeypatch, n, layers, precision):
    c = W.c3_hea(n, n, layers, 0.0)
    on, s1 = _launched(c, precision)
    monkeypatch.setenv("QIMAX_GATHER", "0")
    off, s0 = _launched(c, precision)
    assert on["gather"] >= layers - 1 and "gather" not in off
    assert s1["sort_elems"] < s0["sort_elems"] and s1["images"] == s0["images"]


@pytest.mark.parametrize("n", [12, 32, 48, 64])
def test_small_passes_and_tables(monkeypatch, n):
    c = W.c2_clifford_rz(1, n, 60, 6)
    on, s1 = _launched(c)
    assert on["small_passes"] >= 1 and on["chain_tables"] >= 1
    monkeypatch.setenv("QIMAX_SMALL_GROUPS", "0")
    off, s0 = _launched(c)
    assert "small_passes" not in off and s1["syncs"] < s0["syncs"]


@pytest.mark.parametrize("max_n,precision", [(16, 64), (16, 32), (32, 64), (64, 64)])
def test_groups_of_a_batch(max_n, precision):
    cs = [W.c2_clifford_rz(seed=s, n=max_n - 3 * s, depth=50, n_rz=3 + s) for s in range(3)]
    launched = []
    for how in ("run", "step"):
        with Batch(precision=precision, max_n=max_n) as b:
            b.profile(True)
            for c in cs:
                b.submit(c)
            if how == "run":
                b.run()
            else:
                while b.step():
                    pass
            b.profile(False)
            launched.append(b.profile_read())
    run, step = launched
    assert run["small_passes"]["launches"] >= 1 and "small_passes" not in step
    assert run.get("chunk_sort", {"launches": 0})["launches"] < step["chunk_sort"]["launches"]
