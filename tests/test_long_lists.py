"""Lists long enough that a workgroup takes eight rounds and more, where redundant computation leaves out the terms of rows that can no
longer win: 10 and 11 stages (from there on the next row is fetched ahead), the fewest and most stages a list takes, one and several
classes of pipelines, rows that do not fit and rows that are none, ties.  The winner and its position against the least of the
costs the same list stores, those against the oracle at sampled rows; whole numbers, compared exactly."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2508_21613_amd import synth


def _case(L, PP, DP, M, failed, cap_x=4.0, hetero=False, act=False, **kw):
    fwd, bwd, mem = synth.layer_tables(19 * L + PP, L)
    sc = synth.scenario(L, PP, DP, M, fwd, bwd, mem, failed, 150, int(cap_x * mem.sum() / PP),
                        speed=synth.speed_factors(L, DP, PP) if hetero else None, **kw)
    return synth.with_activations(sc, 5, cap_scale=1.1) if act else sc


CASES = {
    "2 stages": _case(60, 2, 3, 5, [1]),
    "5 stages, three classes": _case(40, 5, 4, 6, [1, 7], cap_x=3.0),
    "8 stages, every option": _case(33, 8, 3, 9, [3, 12], hetero=True, act=True, transfer_assign=1, allreduce_us=300),
    "10 stages": _case(48, 10, 2, 24, [3]),
    "11 stages": _case(48, 11, 2, 24, [3], cap_x=3.4),
    "16 stages, uneven": _case(40, 16, 2, 20, [3], cap_x=5.0, hetero=True),
    "short horizon": _case(40, 8, 3, 9, [4], horizon_steps=1, xfer_us_per_mib=5000),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_long_lists_find_the_least_of_the_costs_they_store(name):
    import torch
    from paper_2508_21613_amd import binding as B
    sc = CASES[name]
    o, g = O.Scenario(sc), B.Scenario(sc)
    n = (1 << 22) + 77
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    for f in g.families:
        k, width = f["strategy"], f["stages"] - 1
        if width == 0:
            continue
        keys = (torch.rand((min(1 << 19, n - i), sc["L"] - 1), generator=gen, device="cuda") for i in range(0, n, 1 << 19))
        rows = torch.cat([(x.topk(width, dim=1, sorted=False).indices + 1).sort(dim=1).values.to(torch.uint8) for x in keys])
        if width > 1:
            rows[5] = rows[5].flip(0)                            # decreasing: no partition
        costs = torch.empty(n, dtype=torch.int64, device="cuda")
        rc, best, pos = g.search_cuts(k, rows, costs=costs)
        least = int(costs.min())
        assert rc == 0 and least < B.INFEASIBLE and (best["cost"], pos) == (least, int((costs == least).nonzero()[0]))
        assert width == 1 or int(costs[5]) == B.INFEASIBLE
        ranks = O.partition_rank_batch(rows[torch.tensor([pos, 0, 3, n // 2, n - 1], device="cuda")].cpu().numpy())
        for at, r in zip((pos, 0, 3, n // 2, n - 1), ranks):
            code, plan, _ = o.search_range(k, int(r), 1)
            assert int(costs[at]) == (plan["cost"] if code == 0 else B.INFEASIBLE), at
        d_ranks = g.rank_partitions(k, rows)
        for mode in (0, 1):
            g.set_bounded_search(mode)
            assert g.search_cuts(k, rows) == (rc, best, pos) and g.search_ranks(k, d_ranks) == (rc, best, pos), mode
        g.set_bounded_search(0)
        # the same row at a lower and at a higher position: the lower one is the winner's
        rows[n - 1] = rows[pos]
        rows[2 * n // 3] = rows[pos]
        first = min(pos, 2 * n // 3)
        assert g.search_cuts(k, rows) == (rc, best, first)
    g.close()
