"""Reroute penalties where a peer's scaled stage time rounds to 0: such a peer takes its micro-batches for nothing, but no more
of them than the reroute cap allows.  Searches, lists and bounded searches against the oracle on the specialised kernels (up
to 4, up to 15 peers) and on the generic one, with caps that bind and without.  Whole numbers, compared exactly."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2508_21613_amd import synth


def _case(L, PP, DP, M, failed, factors, cap, scale=1, slowest=None):
    """factors: per pipeline, the factor of its nodes (all stages); a factor of 1 makes every stage time below 32,768 us 0"""
    fwd, bwd, mem = synth.layer_tables(7 * L + DP, L)
    speed = np.repeat(np.array(factors, dtype=np.uint32), PP)
    if slowest is not None:
        speed[slowest] = 1 << 20
    return synth.scenario(L, PP, DP, M, fwd * scale, bwd * scale, mem, failed, 120, int(mem.sum()) * 4 // PP, speed=speed, reroute_cap=cap)


def _one_us(L, PP, DP, M, failed, factors, cap):
    sc = _case(L, PP, DP, M, failed, factors, cap)
    return dict(sc, fwd_us=np.ones(L, np.int32), bwd_us=np.ones(L, np.int32), comm_us=0)


# (specialised kernel, scenario)
CASES = {
    "one of two peers, cap binds": (True, _case(9, 3, 3, 4, [1], (65536, 1, 60000), 3)),
    "one of two peers, cap of all orphans": (True, _case(9, 3, 3, 4, [1], (65536, 1, 60000), 4)),
    "one of two peers, no cap": (True, _case(9, 3, 3, 4, [1], (65536, 1, 60000), 0)),
    "layers of one microsecond": (True, _one_us(9, 4, 3, 4, [2], (65536, 30000, 65536), 2)),
    "two of three peers": (True, _case(10, 4, 4, 6, [2], (65536, 1, 1, 70000), 3)),
    "all peers": (True, _case(10, 4, 3, 6, [2], (65536, 1, 1), 3)),
    "two stages lost": (True, _case(9, 4, 3, 4, [1, 6], (65536, 1, 60000), 3)),
    "four peers": (True, _case(8, 3, 5, 9, [1], (65536, 1, 60000, 61000, 90000), 4)),
    "five peers": (True, _case(8, 3, 6, 9, [1], (65536, 1, 60000, 61000, 90000, 65536), 3)),
    "nine peers": (True, _case(8, 3, 10, 6, [1], (65536, 1, 2, 60000, 61000, 1, 62000, 63000, 64000, 65000), 1)),
    "generic kernel, cap binds": (False, _case(10, 8, 3, 16, [3], (65536, 1, 65536), 9, scale=8, slowest=17)),
    "generic kernel, no cap": (False, _case(10, 8, 3, 16, [3], (65536, 1, 65536), 0, scale=8, slowest=17)),
}


@pytest.mark.parametrize("name", CASES)
def test_the_cases_are_on_the_kernel_they_name(name):
    from paper_2508_21613_amd import binding as B
    specialised, sc = CASES[name]
    assert B.kernel_selection(sc)["specialised"][2] == specialised
    dead = sc["failed_nodes"][0]
    stage = dead % sc["PP"]
    peers = [int(sc["speed_q16"][d * sc["PP"] + stage]) for d in range(sc["DP"]) if d * sc["PP"] + stage not in sc["failed_nodes"]]
    layer = int(min(sc["fwd_us"].min(), sc["bwd_us"].min()))
    assert any((layer * q + 32768) >> 16 == 0 for q in peers)


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_searches_and_lists_against_the_oracle(name):
    import torch
    from paper_2508_21613_amd import binding as B
    _, sc = CASES[name]
    o, g = O.Scenario(sc), B.Scenario(sc)
    n = g.family(2)["n_part"]
    each = [o.search_range(2, r, 1) for r in range(n)]
    want = np.array([b["cost"] if rc == O.OK else O.INF for rc, b, *_ in each])
    order = np.random.default_rng(3).permutation(n)
    costs = torch.empty(n, dtype=torch.int64, device="cuda")
    rc, best, at = g.search_ranks(2, torch.from_numpy(order.astype(np.int64)).cuda(), costs=costs)
    assert (costs.cpu().numpy() == want[order]).all()
    assert rc == 0 and at == int(np.argmin(want[order])) and best == each[order[at]][1]
    for mask in (4, 7):
        for bounded in (0, 1, 2):
            g.set_bounded_search(bounded)
            assert g.search_best(mask) == o.search(mask), (mask, bounded)
        g.set_bounded_search(0)
        assert g.search_best_static(mask) == o.search(mask)
    g.close()
