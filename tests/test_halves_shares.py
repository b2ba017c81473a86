"""Search by halves in the layouts that sizes alone seldom ask for.  Two choices of the lower cuts a lane (by themselves only from 2^24 units of
work on, a third of 10^9 partitions): every depth from 10 stages on under every strategy, with every second lane idle and with none, ties,
open assignments, rounds of communication, times beyond 2^24.  Shares of work that end anywhere within the walked cuts, two, three and four of
them, from one wavefront for all to a million of a unit or two each: where every partition fits, the number of those that fit tells
that each is walked once.  Against the range kernel over the same space, the winner's cost against the oracle.  Whole numbers, compared exactly."""
from math import comb

import pytest

from oracle import oracle as O
from paper_2508_21613_amd import synth
from tests import test_bounded_by_halves, test_halves_nodes, test_halves_walk


def _case(L, PP, DP, M, failed, cap_x=5.0, act=False, **kw):
    fwd, bwd, mem = synth.layer_tables(37 * L + PP, L)
    sc = synth.scenario(L, PP, DP, M, fwd, bwd, mem, failed, 150, int(cap_x * mem.sum() / PP), **kw)
    return synth.with_activations(sc, 5, cap_scale=1.1) if act else sc


TWO = {"%d stages" % PP: _case(L, PP, 3, PP + 5, [PP // 3, PP + PP // 2], act=PP % 2 == 0)
       for PP, L in ((10, 29), (11, 28), (12, 27), (13, 27), (14, 27), (15, 27), (16, 27))}
TWO["17 stages, 16 left"] = _case(27, 17, 2, 20, [6])
TWO["17 stages, 16 left, assignment open"] = _case(28, 17, 2, 18, [16], transfer_assign=1, allreduce_us=400)
for _module in (test_halves_walk, test_halves_nodes, test_bounded_by_halves):
    for _name, _sc in _module.CASES.items():
        _sc = _sc[1] if isinstance(_sc, tuple) else _sc
        if _sc["PP"] >= 10 and comb(_sc["L"] - 1, _sc["PP"] - 1) >= 1 << 21 and not _name.startswith(("nodes: ", "halves: ")):
            TWO["%s: %s" % (_module.__name__.split("test_")[-1], _name)] = _sc


def _takes(sc):
    """strategies of a case that go by halves, with their stages"""
    from paper_2508_21613_amd import binding as B
    return {k: stages for k, stages in ((0, sc["PP"]), (1, sc["PP"] - 1), (2, sc["PP"])) if B.halves_selection(sc, k)[0]}


def _by_range(g, f):
    """(winner, partitions that fit) of a family, by the range kernel in two windows"""
    k, half = f["strategy"], f["n_part"] // 2
    got, fit = [], 0
    for first, count in ((0, half), (half, f["n_part"] - half)):
        got.append(g.search_range(k, first, count))
        fit += g.get_timing()["feasible"][k]
    found = [b for b in got if b[0] == 0]
    return (min(found, key=lambda x: (x[1]["cost"], x[1]["index"])) if found else got[0]), fit


def test_two_choices_reach_every_depth_and_strategy():
    from paper_2508_21613_amd import binding as B
    seen = set()
    for sc in TWO.values():
        for k, stages in _takes(sc).items():
            seen.add((k, stages))
            assert B.halves_work(sc, k)["choices"] == 1              # of this size only when asked for
    assert seen >= {(k, stages) for k in range(3) for stages in range(10, 17)}
    large = synth.config2()                                          # by size, where the search takes milliseconds
    large = dict(large, PP=11, failed_nodes=[3])
    assert B.halves_work(large, 2)["choices"] == 2 and B.halves_work(dict(large, PP=9), 2)["choices"] == 1


@pytest.mark.gpu
@pytest.mark.parametrize("name", TWO)
def test_two_choices_a_lane(name):
    from paper_2508_21613_amd import binding as B
    sc = TWO[name]
    o, g = O.Scenario(sc), B.Scenario(sc)
    takes = _takes(sc)
    assert takes
    g.set_timing(True)
    for f in g.families:
        k = f["strategy"]
        if takes.get(k, 0) < 10:
            continue
        want, fit = _by_range(g, f)
        for choices in (2, 1):
            g.set_halves_shares(choices)
            assert g.search_best(1 << k) == want, (k, choices)
            assert g.get_timing()["feasible"][k] == fit, (k, choices)
        if want[0] == 0:
            assert int(o.score(want[1]["index"], 1)[0]) == want[1]["cost"]
    g.close()


SHARES = {
    "two walked cuts": _case(52, 6, 2, 9, [2]),
    "two walked cuts, long model": _case(120, 5, 2, 7, []),
    "three walked cuts": _case(34, 8, 2, 9, [6]),
    "three walked cuts, few lanes": _case(29, 10, 2, 13, [1]),
    "four walked cuts": _case(27, 12, 2, 12, [11]),
    "four walked cuts, little above": _case(27, 16, 2, 16, [8]),
}


def test_the_cases_walk_as_many_cuts_as_they_name():
    from paper_2508_21613_amd import binding as B
    for name, sc in SHARES.items():
        walked = {"two": 2, "three": 3, "four": 4}[name.split()[0]]
        assert B.halves_work(sc, 2)["walked_cuts"] == walked and B.halves_selection(sc, 2)[0] > 0, name


@pytest.mark.gpu
@pytest.mark.parametrize("limit", [False, True], ids=["everything fits", "a limit"])
@pytest.mark.parametrize("name", SHARES)
def test_shares_cover_every_partition_once(name, limit):
    from paper_2508_21613_amd import binding as B
    sc = SHARES[name] if limit else dict(SHARES[name], mem_cap_mib=2 ** 31 - 1)
    takes = _takes(sc)
    g = B.Scenario(sc)
    g.set_timing(True)
    for f in g.families:
        k = f["strategy"]
        if k not in takes:
            continue
        want, fit = _by_range(g, f)
        assert limit or fit == f["n_part"]
        units = B.halves_work(sc, k)["units"]
        for choices in (1, 2) if takes[k] >= 10 else (1,):
            for wavefronts in (1, 7, 1000, 65537, units // 3, min(units, 1 << 20)):
                g.set_halves_shares(choices, wavefronts)
                assert g.search_best(1 << k) == want, (k, choices, wavefronts)
                assert g.get_timing()["feasible"][k] == fit, (k, choices, wavefronts)
                if choices == 1:
                    g.set_bounded_search(1)
                    assert g.search_best(1 << k) == want, (k, "bounded", wavefronts)
                    g.set_bounded_search(0)
    g.close()


@pytest.mark.gpu
def test_shares_out_of_range_are_refused():
    from paper_2508_21613_amd import binding as B
    g = B.Scenario(SHARES["two walked cuts"])
    for args in ((-1, 0), (3, 0), (0, (1 << 24) + 1)):
        with pytest.raises(B.ChmError) as e:
            g.set_halves_shares(*args)
        assert e.value.code == B.ERR_ARG
    g.close()
