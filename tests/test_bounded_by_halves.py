"""Bounded searches that take families by halves, whose loops leave out what the cuts placed so far make too slow: the same plan as the
exhaustive search over the same family (which test_search_by_halves.py and test_halves_nodes.py hold against the range kernel), per
strategy and all together, over the cases of those files and over every width and depth, rounds of communication, several chunks and
families that are enumerated beside them.  Whole numbers, compared exactly."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2508_21613_amd import synth
from tests import test_halves_nodes, test_search_by_halves


def _case(L, PP, DP, M, failed, cap_x=4.0, act=False, **kw):
    fwd, bwd, mem = synth.layer_tables(23 * L + PP, L)
    sc = synth.scenario(L, PP, DP, M, fwd, bwd, mem, failed, 150, int(cap_x * mem.sum() / PP), **kw)
    return synth.with_activations(sc, 5, cap_scale=1.1) if act else sc


CASES = {"nodes: " + name: sc for name, (_, sc) in test_halves_nodes.CASES.items()}
CASES.update({"halves: " + name: sc for name, sc in test_search_by_halves.CASES.items()})
for _s in range(9):
    CASES["9 stages, stage %d gone" % _s] = _case(32, 9, 2, 11, [_s, 9 + (_s + 4) % 9], act=_s % 3 == 0)
for _s in range(0, 12):
    CASES["12 stages, stage %d gone" % _s] = _case(25, 12, 2, 12, [_s], cap_x=5.0, allreduce_us=250 if _s % 4 == 0 else 0)
for _s in (0, 5, 11, 12, 13, 14, 15):
    CASES["16 stages, stage %d gone" % _s] = _case(25, 16, 2, 17, [_s], cap_x=5.0, act=_s % 2 == 0)
CASES.update({
    "6 stages, rounds": _case(60, 6, 3, 7, [1, 8], allreduce_us=200, act=True),
    "10 stages, rounds, chunks of 2^16": _case(29, 10, 2, 11, [4], allreduce_us=500, horizon_steps=1 << 21),
    "13 stages, short horizon": _case(26, 13, 2, 14, [6], cap_x=5.0, horizon_steps=1, xfer_us_per_mib=4000, transfer_assign=1),
    "14 stages, equal layers (ties)": dict(_case(25, 14, 2, 15, [2], cap_x=5.0), fwd_us=np.full(25, 900, np.int32),
                                           bwd_us=np.full(25, 1800, np.int32), mem_mib=np.full(25, 500, np.int32)),
    "10 stages": _case(30, 10, 3, 11, [4, 15]),
    "11 stages, 10 left": _case(30, 11, 2, 13, [8]),
    "8 stages, 7 left": _case(41, 8, 2, 9, [2], allreduce_us=100),
    "6 stages, 5 left": _case(100, 6, 2, 9, [5]),
    "15 stages, every pipeline hit": _case(26, 15, 3, 16, [3, 21, 44], cap_x=5.0),
})


def test_the_cases_cover_every_depth():
    from paper_2508_21613_amd import binding as B
    seen = {(k, stages, B.halves_selection(sc, k)[0]) for sc in CASES.values()
            for k, stages in ((0, sc["PP"]), (1, sc["PP"] - 1), (2, sc["PP"]))}
    depths = {k: {stages for j, stages, up in seen if j == k and up} for k in range(3)}
    assert depths[0] >= set(range(5, 17)) and depths[2] >= set(range(5, 17)) and depths[1] >= set(range(5, 16))
    for k in (0, 2):
        assert {2, 3, 4} <= {up for j, _, up in seen if j == k}


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_bounded_search_finds_what_the_exhaustive_one_finds(name):
    from paper_2508_21613_amd import binding as B
    g = B.Scenario(CASES[name])
    masks = [1 << f["strategy"] for f in g.families] + [7]
    want, fit = {}, {}
    for mask in masks:
        want[mask] = g.search_best(mask)
        fit[mask] = g.get_timing()["feasible"]
    g.set_bounded_search(1)
    for mask in masks + [7]:
        assert g.search_best(mask) == want[mask], mask
        assert all(a <= b for a, b in zip(g.get_timing()["feasible"], fit[mask])), mask
    (rc, best), = B.search_best_batch([g], 7)
    assert (rc, best) == want[7]
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("PP,L", [(8, 48), (9, 44)])
def test_families_by_halves_beside_one_that_is_not(PP, L):
    """communication rounds keep strategy 0 from going by halves: the others start with the cost the seeds found all the same"""
    from paper_2508_21613_amd import binding as B
    g = B.Scenario(_case(L, PP, 3, 16, [3], allreduce_us=300))
    assert g.family(0)["n_part"] >= 1 << 25
    want = {mask: g.search_best(mask) for mask in (2, 4, 6, 7)}
    g.set_bounded_search(1)
    looked_at = {}
    for mask in (2, 4, 6, 7):
        assert g.search_best(mask) == want[mask], mask
        looked_at[mask] = g.get_timing()["feasible"]
    assert looked_at[7][1] <= 2 * looked_at[2][1] < g.family(1)["n_part"] // 2
    assert looked_at[7][2] <= 2 * looked_at[6][2] + 100000 < g.family(2)["n_part"] // 2
    assert int(O.Scenario(_case(L, PP, 3, 16, [3], allreduce_us=300)).score(want[7][1]["index"], 1)[0]) == want[7][1]["cost"]
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("PP,L,masks", [(16, 30, (7, 4, 2)), (11, 40, (7, 4, 2)), (9, 52, (7, 4)), (12, 34, (7, 4, 2))])
@pytest.mark.parametrize("assign", [0, 1])
def test_families_of_many_lower_halves(PP, L, masks, assign):
    """calls whose lower halves would take longer to set up than candidates take to count are enumerated, but for a family that is left
    with many candidates: next to nothing is looked at where all strategies are searched"""
    from paper_2508_21613_amd import binding as B
    g = B.Scenario(_case(L, PP, 3, 16, [3], transfer_assign=assign))
    for mask in masks:
        g.set_bounded_search(0)
        want = g.search_best(mask)
        g.set_bounded_search(1)
        assert g.search_best(mask) == want, mask
        if mask == 7:
            looked_at = g.get_timing()["feasible"]
            assert looked_at[0] + looked_at[2] <= 1 << 17, looked_at
    g.close()
