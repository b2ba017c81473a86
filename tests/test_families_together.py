"""Small searches, whose families are searched in one launch: stages of the re-partitioned pipelines one, two and three fewer than
the grid's (the last without a common instance), the shallowest and deepest grids with one, families that are missing, the seeds
of large families.  Against the oracle, one mask after the other; whole numbers, compared exactly."""
import pytest

from oracle import oracle as O
from paper_2508_21613_amd import synth


def _case(L, PP, DP, M, failed, cap_x=4.0, act=False, hetero=False, **kw):
    fwd, bwd, mem = synth.layer_tables(13 * L + PP, L)
    sc = synth.scenario(L, PP, DP, M, fwd, bwd, mem, failed, 150, max(int(cap_x * mem.sum() / PP), 3 * int(mem.max())),
                        speed=synth.speed_factors(L, DP, PP) if hetero else None, **kw)
    return synth.with_activations(sc, 5, cap_scale=1.1) if act else sc


CASES = {
    "3 stages": _case(9, 3, 3, 4, [1]),
    "4 stages, two fewer": _case(12, 4, 3, 5, [1, 3], hetero=True),
    "6 stages, three fewer": _case(13, 6, 3, 5, [0, 2, 4]),
    "8 stages, one fewer": _case(14, 8, 3, 6, [3, 12], act=True, hetero=True),
    "9 stages, two fewer": _case(14, 9, 2, 9, [2, 5]),
    "12 stages": _case(16, 12, 2, 5, [7], hetero=True),
    "13 stages, two fewer": _case(17, 13, 2, 14, [1, 9]),
    "16 stages": _case(19, 16, 2, 20, [15]),
    "17 stages": _case(20, 17, 2, 6, [4]),
    "24 stages": _case(26, 24, 2, 30, [11]),
    "25 stages": _case(27, 25, 2, 5, [11]),
    "two stages, one left": _case(9, 2, 2, 4, [1]),
    "no re-partition": _case(14, 6, 3, 6, [1, 6, 8]),
    "nothing lost": _case(12, 5, 2, 6, []),
    "nothing fits": dict(_case(12, 5, 2, 6, [2]), mem_cap_mib=1),
    "families of several chunks": _case(25, 7, 2, 6, [3], horizon_steps=1 << 22),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_families_of_a_call_against_the_oracle(name):
    from paper_2508_21613_amd import binding as B
    sc = CASES[name]
    o, g = O.Scenario(sc), B.Scenario(sc)
    for mask in (7, 5, 3, 6):
        assert any(mask >> f["strategy"] & 1 for f in g.families)
        want = o.search(mask)
        assert g.search_best(mask) == want, mask
        assert g.search_best(mask) == want, mask                 # the words of the first search, put back by its end
    (rc, best), = B.search_best_batch([g], 7)
    assert (rc, best) == o.search(7) and g.search_best_static(7) == (rc, best)
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("failed", [[3], [3, 5], [3, 9]], ids=str)
def test_seeds_of_large_families(failed):
    from paper_2508_21613_amd import binding as B
    sc = _case(32, 8, 3, 9, failed)
    g = B.Scenario(sc)
    g.set_timing(True)                                           # (families and their seeds one by one)
    apart = g.search_best(7)
    g.set_timing(False)
    assert g.search_best(7) == apart and apart[0] == 0
    assert int(O.Scenario(sc).score(apart[1]["index"], 1)[0]) == apart[1]["cost"]
    g.close()
