"""Search by halves (chm_halves_kernel.h) where its float times, its limit and its shares of work can go wrong: times beyond 2^24 (sums are
rounded there), fetch times that outweigh the steps or cost nothing, untouched pipelines that decide the step time, stages that lost nodes at
every place of the walk, an odd and a small number of layers above the lanes' cuts.  Against the range kernel over the same space in two
windows, the winner's cost against the oracle.  Whole numbers, compared exactly."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2508_21613_amd import synth


def _case(L, PP, DP, M, failed, cap_x=4.0, act=False, slowest=1, **kw):
    fwd, bwd, mem = synth.layer_tables(41 * L + PP, L)
    fwd[L // 2] *= slowest                               # (a layer that takes longer than all others together: times beyond 2^24 whatever the cuts)
    bwd[L // 2] *= slowest
    sc = synth.scenario(L, PP, DP, M, fwd, bwd, mem, failed, 150, int(cap_x * mem.sum() / PP), **kw)
    return synth.with_activations(sc, 5, cap_scale=1.1) if act else sc


CASES = {
    "8 stages, times beyond 2^24": _case(34, 8, 2, 24, [4], slowest=600),
    "11 stages, times beyond 2^24": _case(26, 11, 2, 30, [4], slowest=500, cap_x=5.0),
    "7 stages, times beyond 2^24, no memory limit": dict(_case(40, 7, 2, 20, [2], slowest=700), mem_cap_mib=2 ** 31 - 1),
    "6 stages, fetching outweighs the steps": _case(55, 6, 3, 8, [7], horizon_steps=1, xfer_us_per_mib=5000),
    "10 stages, fetching costs nothing": _case(30, 10, 2, 11, [13], xfer_us_per_mib=0),
    "8 stages, untouched pipelines decide": _case(36, 9, 12, 10, [4], cap_x=5.0),
    "9 stages, communication rounds weigh": _case(33, 9, 3, 12, [0, 17], allreduce_us=9000),
    "12 stages, little above the lanes' cuts": _case(25, 12, 2, 12, [11], cap_x=6.0),
    "16 stages, few layers more than stages": _case(26, 16, 2, 16, [15], cap_x=6.0, act=True),
}
CASES["13 stages, assignment open"] = _case(27, 14, 3, 15, [0], cap_x=5.0, transfer_assign=1, allreduce_us=300)
CASES["7 stages, assignment open, two pipelines hit"] = _case(40, 8, 3, 10, [3, 14], transfer_assign=1, xfer_us_per_mib=3000)
CASES.update({"8 stages, stages %d and %d lost" % (s, (s + 3) % 8): _case(35, 8, 4, 9, [s, 8 + (s + 3) % 8]) for s in range(8)})
CASES.update({"11 stages, stage %d lost" % s: _case(27, 11, 3, 12, [s], cap_x=5.0) for s in (5, 6, 7, 8, 9, 10)})


# strategies of each case that go by halves
ALL = ("10 stages, fetching costs nothing", "8 stages, untouched pipelines decide", "16 stages, few layers more than stages",
       "7 stages, assignment open, two pipelines hit", *("11 stages, stage %d lost" % s for s in range(5, 11)))
WITHOUT_0 = ("9 stages, communication rounds weigh", "13 stages, assignment open")


@pytest.mark.parametrize("name", CASES)
def test_the_cases_go_by_halves(name):
    from paper_2508_21613_amd import binding as B
    want = [0, 1, 2] if name in ALL else [1, 2] if name in WITHOUT_0 else [0, 2]
    assert [k for k in range(3) if B.halves_selection(CASES[name], k)[0]] == want


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_walk_finds_what_the_range_kernel_finds(name):
    from paper_2508_21613_amd import binding as B
    sc = CASES[name]
    o, g = O.Scenario(sc), B.Scenario(sc)
    g.set_timing(True)
    each = []
    for f in g.families:
        k, half = f["strategy"], f["n_part"] // 2
        got, fit = [], 0
        for first, count in ((0, half), (half, f["n_part"] - half)):
            got.append(g.search_range(k, first, count))
            fit += g.get_timing()["feasible"][k]
        found = [b for b in got if b[0] == 0]
        want = min(found, key=lambda x: (x[1]["cost"], x[1]["index"])) if found else got[0]
        assert g.search_best(1 << k) == want, k
        assert g.get_timing()["feasible"][k] == fit, k
        if want[0] == 0:
            assert int(o.score(want[1]["index"], 1)[0]) == want[1]["cost"]
            each.append(want)
    best = min(each, key=lambda v: (v[1]["cost"], v[1]["index"]))
    g.set_timing(False)
    assert g.search_best(7) == best
    g.set_bounded_search(1)
    assert g.search_best(7) == best
    g.close()

