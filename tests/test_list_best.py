"""Long lists of cut positions without stored costs (chm_list.hip), where a row is worked out only if a lower bound of its time may still win:
the shortest list that goes there and the one before it, lists whose last workgroup is nearly empty, rows that are no partition (equal,
falling, zero, 128 and more, behind the last layer), 128 layers, every option of the bound, times too long for it, a list of one and
the same row, one in falling order of cost.  Winner, position and the number of rows that fit against the costs the same list stores; whole
numbers, compared exactly."""
import pytest

from paper_2508_21613_amd import synth


def _case(L, PP, DP, M, failed, cap_x=4.0, hetero=False, act=False, slowest=1, **kw):
    fwd, bwd, mem = synth.layer_tables(23 * L + PP, L)
    fwd[L // 2] *= slowest
    bwd[L // 2] *= slowest
    sc = synth.scenario(L, PP, DP, M, fwd, bwd, mem, failed, 150, int(cap_x * mem.sum() / PP),
                        speed=synth.speed_factors(L, DP, PP) if hetero else None, **kw)
    return synth.with_activations(sc, 5, cap_scale=1.1) if act else sc


CASES = {
    "2 stages, 128 layers": _case(128, 2, 3, 5, [1]),
    "3 stages, the first lost": _case(128, 3, 2, 9, [0]),
    "5 stages, every pipeline hit": _case(40, 5, 2, 12, [1, 8], cap_x=3.0),
    "5 stages, the last lost": _case(60, 5, 3, 7, [4], allreduce_us=400),
    "9 stages, every option": _case(33, 9, 3, 9, [3, 13], hetero=True, act=True, transfer_assign=1, allreduce_us=300),
    "13 stages, uneven": _case(64, 13, 2, 40, [8], cap_x=5.0, hetero=True, reroute_cap=40),
    "16 stages, one hit in each word of cuts": _case(48, 16, 5, 2, [3, 20, 40, 75], cap_x=5.0),
    "16 stages, nothing fits": dict(_case(40, 16, 2, 20, [3]), mem_cap_mib=1),
    "7 stages, times too long for the bound": _case(40, 7, 2, 4, [4], slowest=4000),
}
SHORTEST = 3 << 19


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_the_winner_is_the_least_of_the_stored_costs(name):
    import torch
    from paper_2508_21613_amd import binding as B
    sc = CASES[name]
    g = B.Scenario(sc)
    n = SHORTEST + 2049
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    for f in g.families:
        k, width = f["strategy"], f["stages"] - 1
        if width == 0:
            continue
        keys = (torch.rand((min(1 << 19, n - i), sc["L"] - 1), generator=gen, device="cuda") for i in range(0, n, 1 << 19))
        rows = torch.cat([(x.topk(width, dim=1, sorted=False).indices + 1).sort(dim=1).values.to(torch.uint8) for x in keys])
        for i, bad in enumerate((0, 128, 255, sc["L"])):                # one byte of a row of its own each, at every place
            for j in range(width):
                rows[100 * i + j, j] = bad
        rows[1000] = rows[1001, 0]                                       # equal cuts
        costs = torch.empty(n, dtype=torch.int64, device="cuda")
        g.search_cuts(k, rows, costs=costs)
        assert all(int(costs[100 * i + j]) == B.INFEASIBLE for i in range(4) for j in range(width))
        falling = rows[torch.argsort(costs, descending=True, stable=True)].contiguous()
        alike = rows[int(costs.argmin())].repeat(SHORTEST, 1)
        for what in (rows[:SHORTEST - 1], rows[:SHORTEST], rows[:SHORTEST + 1], rows, falling, alike):
            rc, best, pos = g.search_cuts(k, what.contiguous(), costs=costs[:len(what)])
            fit = g.get_timing()["feasible"][k]
            stored = costs[:len(what)]
            assert fit == int((stored < B.INFEASIBLE).sum())
            if fit:
                least = int(stored.min())
                assert (rc, best["cost"], pos) == (0, least, int((stored == least).nonzero()[0]))
            assert g.search_cuts(k, what.contiguous()) == (rc, best, pos), len(what)
            assert g.get_timing()["feasible"][k] == fit
            worked_out = g.get_timing()["evaluated"][k]
            assert (worked_out == 0) == (fit == 0) and worked_out <= fit
            if len(what) < SHORTEST or name.endswith("too long for the bound"):
                assert worked_out == fit
            elif what is rows and sc["PP"] >= 5 and sc["speed_q16"] is None and fit > n // 2:
                assert worked_out < fit                                  # (half of the six rounds a wavefront has: the first is worked out whole)
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("name,sc", [("8 stages", _case(48, 8, 4, 16, [5])), ("8 stages, uneven", _case(48, 8, 4, 16, [5], hetero=True)),
                                     ("15 stages left, uneven", _case(60, 16, 2, 24, [9], cap_x=5.0, hetero=True))], ids=lambda v: v if isinstance(v, str) else "")
def test_lists_whose_bound_leaves_nothing_out(name, sc):
    """neighbours of one plan, nearly all of which may win, so that rounds go by without a look at the bound; behind them random rows, for which
    it counts again; the best row first, last, and at both ends of a round"""
    import torch
    from paper_2508_21613_amd import binding as B
    g = B.Scenario(sc)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    n = 5 << 20
    for f in g.families:
        k, width = f["strategy"], f["stages"] - 1
        rc, best = g.search_range(k, f["n_part"] // 3, 1 << 18)
        assert rc == 0
        plan = torch.tensor(best["cuts"][:width], dtype=torch.int16, device="cuda")
        rows = plan.repeat(n, 1)
        rows += torch.randint(-1, 2, rows.shape, generator=gen, device="cuda", dtype=torch.int16)
        rising = (rows[:, 1:] > rows[:, :-1]).all(1) & (rows[:, 0] > 0) & (rows[:, -1] < sc["L"])
        rows = torch.where(rising[:, None], rows, plan[None]).to(torch.uint8)
        keys = torch.rand((1 << 19, sc["L"] - 1), generator=gen, device="cuda")
        rows[n // 2:n // 2 + (1 << 19)] = (keys.topk(width, dim=1, sorted=False).indices + 1).sort(dim=1).values.to(torch.uint8)
        costs = torch.empty(n, dtype=torch.int64, device="cuda")
        g.search_cuts(k, rows, costs=costs)
        fit = g.get_timing()["feasible"][k]
        assert fit == int((costs < B.INFEASIBLE).sum()) > n // 4
        lowest = rows[int(costs.argmin())].clone()
        least = int(costs.min())
        rows = rows[costs > least].contiguous()                          # no other row is as good as the one put in
        for at in (0, len(rows) - 1, 64 * 4000, 64 * 4000 + 63, len(rows) // 2 + 17):
            kept = rows[at].clone()
            rows[at] = lowest
            rc, got, pos = g.search_cuts(k, rows)
            assert (rc, got["cost"], pos) == (0, least, at), (k, at)
            rows[at] = kept
    g.close()


def test_the_case_of_long_times_is_one():
    """(24-bit multiplies do not do, but the specialised kernels still take it)"""
    from paper_2508_21613_amd import binding as B
    for name, sc in CASES.items():
        sel = B.kernel_selection(sc)
        sharp = not name.endswith("too long for the bound")
        for k, stages in ((0, sc["PP"]), (1, sc["PP"] - 1), (2, sc["PP"])):
            assert stages < 2 or (sel["specialised"][k] and sel["sharp_bound"][k] == sharp), (name, k)
