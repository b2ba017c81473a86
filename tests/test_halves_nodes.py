"""Search by halves where a pipeline is short of nodes: the class that is timed for every partition lacks a node in every position
it can lack it (two and four walked cuts; every pipeline hit), more than three classes, and a long model.  Against the range kernel over the same space in two windows, the winner's cost against
the oracle.  Whole numbers, compared exactly."""
import pytest

from oracle import oracle as O
from paper_2508_21613_amd import synth


def _case(L, PP, DP, M, failed, cap_x=4.0, act=False, **kw):
    fwd, bwd, mem = synth.layer_tables(31 * L + PP, L)
    sc = synth.scenario(L, PP, DP, M, fwd, bwd, mem, failed, 150, int(cap_x * mem.sum() / PP), **kw)
    return synth.with_activations(sc, 5, cap_scale=1.1) if act else sc


# (upper cuts of strategy 0, scenario)
CASES = {"two cuts, stage %d gone" % s: (2, _case(39, 7, 2, 8, [s, 7 + (s + 3) % 7], act=s % 2 == 0)) for s in range(7)}
CASES.update({"four cuts, stage %d gone" % s: (4, _case(27, 12, 2, 13, [s, 12 + (s + 5) % 12], cap_x=5.0)) for s in (0, 1, 7, 8, 9, 10, 11)})
CASES["four cuts, activations, ring pair"] = (4, _case(27, 12, 2, 12, [8, 23], cap_x=5.0, act=True, transfer_assign=1))
CASES["five classes"] = (2, _case(40, 7, 5, 9, [1, 9, 17, 25], cap_x=3.5))
CASES["7 stages, more than 120 layers"] = (2, _case(121, 7, 2, 8, [3], act=True))


@pytest.mark.parametrize("name", CASES)
def test_the_cases_have_the_width_they_name(name):
    from paper_2508_21613_amd import binding as B
    up, sc = CASES[name]
    assert B.halves_selection(sc, 0)[0] == up


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_halves_with_nodes_gone_against_the_range_kernel(name):
    from paper_2508_21613_amd import binding as B
    _, sc = CASES[name]
    o, g = O.Scenario(sc), B.Scenario(sc)
    g.set_timing(True)
    for f in g.families:
        k, half = f["strategy"], f["n_part"] // 2
        got, fit = [], 0
        for first, count in ((0, half), (half, f["n_part"] - half)):
            got.append(g.search_range(k, first, count))
            fit += g.get_timing()["feasible"][k]
        found = [b for b in got if b[0] == 0]
        want = min(found, key=lambda x: (x[1]["cost"], x[1]["index"])) if found else got[0]
        assert g.search_best(1 << k) == want, k
        assert g.get_timing()["feasible"][k] == fit
        if want[0] == 0:
            assert int(o.score(want[1]["index"], 1)[0]) == want[1]["cost"]
    g.close()
