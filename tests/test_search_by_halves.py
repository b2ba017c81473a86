"""Exhaustive search of large families by halves (from 2^21 partitions on) against the range kernel over the same space in
two windows (which test_gpu_random.py and test_closed_forms.py hold against the oracle; test_gpu_full_space.py holds the
search by halves itself against whole-space results of the oracle), the winner's cost against the oracle: two to four walked cuts, the smallest and largest number of stages, failed nodes that cross between the halves,
one to three pipeline classes, every modelling option it takes, several chunks, no failure, no memory limit, ties.  Whole numbers,
compared exactly."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2508_21613_amd import synth


def _case(L, PP, DP, M, failed, cap_x=4.0, act=False, **kw):
    fwd, bwd, mem = synth.layer_tables(17 * L + PP, L)
    sc = synth.scenario(L, PP, DP, M, fwd, bwd, mem, failed, 150, int(cap_x * mem.sum() / PP), **kw)
    return synth.with_activations(sc, 5, cap_scale=1.1) if act else sc


CASES = {
    "5 stages, long model": _case(96, 5, 2, 5, [3]),
    "5 stages, longest model, nothing lost": _case(128, 5, 2, 9, []),
    "6 stages, first stage lost": _case(53, 6, 2, 7, [0], cap_x=3.0),
    "7 stages, options": _case(39, 7, 3, 8, [10], act=True, transfer_assign=1, allreduce_us=400),
    "7 stages, long model": _case(68, 7, 2, 9, [8]),
    "8 stages, crossing node lost, three classes": _case(32, 8, 3, 9, [4, 11], transfer_assign=1),
    "8 stages, every pipeline hit": _case(32, 8, 3, 8, [3, 12, 23], cap_x=3.0),
    "8 stages, nothing lost": _case(32, 8, 2, 16, []),
    "11 stages, last stage lost": _case(26, 11, 2, 12, [21], cap_x=3.0),
    "16 stages": _case(26, 16, 2, 17, [12], cap_x=5.0),
    "8 stages, chunks of 2^16": _case(32, 8, 2, 8, [7], horizon_steps=1 << 22),
    "8 stages, next to nothing fits": _case(32, 8, 3, 9, [4], cap_x=2.1),
    "8 stages, nothing of one strategy fits": _case(32, 8, 3, 9, [4], cap_x=1.5),
    "6 stages, no memory limit": dict(_case(53, 6, 2, 7, [2]), mem_cap_mib=2 ** 31 - 1),
    "8 stages, no memory limit, chunks of 2^16": dict(_case(32, 8, 2, 8, [7], horizon_steps=1 << 22), mem_cap_mib=2 ** 31 - 1),
    "8 stages, equal layers (ties)": dict(_case(32, 8, 2, 8, [6]), fwd_us=np.full(32, 900, np.int32), bwd_us=np.full(32, 1800, np.int32),
                                          mem_mib=np.full(32, 500, np.int32)),
}


def _large(L, PP, DP, M, failed):
    fwd, bwd, mem = synth.layer_tables(L, L)
    return synth.scenario(L, PP, DP, M, fwd, bwd, mem, failed, 150, int(mem.sum()))


def test_families_searched_by_halves_and_their_lanes():
    """from 2^21 partitions on, whatever the depth; the steps reported are those of the cuts that are walked, with 64 choices of the others a
    block, and the units of work those and what set-up and rows take (a few lanes idle where a last cut leaves few choices)"""
    from math import comb
    from paper_2508_21613_amd import binding as B
    walked, choices = set(), set()
    for PP in range(5, 17):
        for L in range(PP + 6, 129, 3):
            sc = _large(L, PP, 3, PP + 4, [PP // 2])
            if comb(L - 1, PP - 1) >= 1 << 36:
                continue
            for k, stages in ((0, PP), (1, PP - 1), (2, PP)):
                n, (up, steps) = comb(L - 1, stages - 1), B.halves_selection(sc, k)
                assert (up > 0) == (n >= 1 << 21 and stages >= 5), (L, stages, k)
                if up == 0:
                    continue
                walked.add((stages, up))
                work, kept = B.halves_work(sc, k), stages - 1 - up
                blocks = {c: {v: -(-comb(v - 1, kept - 1) // (64 * c)) for v in range(kept, L - up)} for c in (1, 2)}
                assert work["walked_cuts"] == up and steps == sum(b * comb(L - 1 - v, up) for v, b in blocks[1].items()), (L, stages, k)
                assert work["units"] > sum(b * comb(L - 1 - v, up) for v, b in blocks[work["choices"]].items())
                share = n / (64 * steps)                     # lanes that keep a choice
                assert share > (0.3 if stages == 5 else 0.7), (L, stages, k, share)
                assert work["choices"] == 1 or (stages >= 10 and n > 1 << 28), (L, stages, k)
                choices.add((stages, work["choices"]))
    assert walked == {(s, 2 if s <= 7 else 3 if s <= 10 else 4) for s in range(5, 17)}
    assert choices == {(s, 1) for s in range(5, 17)} | {(s, 2) for s in range(10, 17)}
    assert B.halves_selection(dict(_large(48, 8, 3, 8, [3]), speed_q16=np.full(24, 65537, np.uint32)), 2)[0] == 0


def test_tables_take_no_more_memory_than_promised():
    """under 0.7 MB a strategy (chm_search_best), whatever the model"""
    from paper_2508_21613_amd import binding as B
    largest = 0
    for L in range(40, 129, 8):
        sc = _large(L, 6, 2, 9, [3])
        for k in range(3):
            work = B.halves_work(sc, k)
            assert (work["table_bytes"] > 0) == (B.halves_selection(sc, k)[0] > 0)
            largest = max(largest, work["table_bytes"])
    assert 129 * 129 * 32 < largest < 700000


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_search_by_halves_finds_what_the_range_kernel_finds(name):
    from paper_2508_21613_amd import binding as B
    sc = CASES[name]
    o, g = O.Scenario(sc), B.Scenario(sc)
    assert max(f["n_part"] for f in g.families) >= 1 << 21
    g.set_timing(True)

    def range_search(k, first, count):
        got = g.search_range(k, first, count)
        return got, g.get_timing()["feasible"][k]

    each = []
    for f in g.families:
        k, half = f["strategy"], f["n_part"] // 2
        (rc_a, a), fit_a = range_search(k, 0, half)
        (rc_b, b), fit_b = range_search(k, half, f["n_part"] - half)
        want = (rc_a, a) if rc_a == 0 and (rc_b != 0 or a["cost"] <= b["cost"]) else (rc_b, b)      # ties: the lower rank
        assert g.search_best(1 << k) == want, k
        assert g.get_timing()["feasible"][k] == fit_a + fit_b == g.get_timing()["evaluated"][k]
        if want[0] == 0:
            assert int(o.score(want[1]["index"], 1)[0]) == want[1]["cost"]
            each.append(want)
    best = min(each, key=lambda v: (v[1]["cost"], v[1]["index"]))
    assert g.search_best(7) == best                      # the tables laid out by the searches before
    assert g.search_best_static(7) == best
    fresh = B.Scenario(sc)
    assert fresh.search_best_static(7) == best           # nothing laid out yet: the range kernels
    assert fresh.search_best(7) == best
    g.close()
    fresh.close()
