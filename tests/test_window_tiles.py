"""Costs of windows of rerouting plan indices where one stage lost nodes: tiles that begin and end inside a partition, the fewest and
most vectors a tile's table takes and one beyond on either side, rows of four and eight entries, odd starts and counts, an output
that is not 16-byte aligned, both tile sizes, few and many stages.  Against the oracle; whole numbers, compared exactly."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2508_21613_amd import synth

pytestmark = pytest.mark.gpu


def _case(L, PP, DP, M, failed, cap_x=3.0, hetero=False, **kw):
    fwd, bwd, mem = synth.layer_tables(11 * L + DP, L)
    return synth.scenario(L, PP, DP, M, fwd, bwd, mem, [failed], 150, int(cap_x * mem.sum() / PP),
                          speed=synth.speed_factors(L, DP, PP) if hetero else None, **kw)


# vectors: C(M + peers - 1, peers - 1)
CASES = {
    "15 vectors": (15, _case(20, 4, 3, 14, 1)),
    "16 vectors": (16, _case(30, 4, 3, 15, 1)),
    "17 vectors, 2 stages": (17, _case(90, 2, 3, 16, 1)),
    "63 vectors": (63, _case(24, 5, 3, 62, 3, hetero=True)),
    "64 vectors": (64, _case(24, 5, 3, 63, 3)),
    "153 vectors": (153, _case(22, 6, 4, 16, 2, hetero=True)),
    "five peers": (126, _case(20, 6, 6, 5, 2, hetero=True)),
    "five peers, 20 stages": (715, _case(23, 20, 6, 9, 7)),
    "five peers, eight orphans each": (495, _case(18, 4, 6, 8, 2, hetero=True, reroute_cap=0)),
}


@pytest.mark.parametrize("name", CASES)
def test_windows_against_the_oracle(name):
    import torch
    from paper_2508_21613_amd import binding as B
    vectors, sc = CASES[name]
    o, g = O.Scenario(sc), B.Scenario(sc)
    f = g.family(2)
    size = f["n_part"] * f["n_reroute"]
    rng = np.random.default_rng(1)
    out = torch.empty(size + 1, dtype=torch.int64, device="cuda")
    for first, count in ((0, 1), (1, 2047), (5, 2048), (3, 2049), (7, 8191), (0, 8193), (size // 3, 20011), (max(0, size - 4099), 4099)):
        first, count = min(first, size - 1), min(count, size - min(first, size - 1))
        for shift in (0, 1):                                     # (an odd number of 8-byte words into the allocation)
            out.fill_(-7)
            got = g.score_plans(f["offset"] + first, count, out=out[shift:shift + count]).cpu().numpy()
            assert out[shift + count:].eq(-7).all() and out[:shift].eq(-7).all()
            if shift == 0:
                want = got
                at = np.unique(np.concatenate([[0, count - 1], rng.integers(0, count, 40)]))
                for i in at:
                    assert int(o.score(f["offset"] + first + int(i), 1)[0]) == got[i], (first, count, i)
                if count <= 2500:
                    assert (o.score(f["offset"] + first, count) == got).all()
            else:
                assert (got == want).all()
    g.close()


def test_large_window_is_its_small_ones():
    from paper_2508_21613_amd import binding as B
    g = B.Scenario(_case(34, 6, 4, 16, 2, hetero=True))
    f = g.family(2)
    first, count = f["offset"] + 100003, (1 << 21) + 777            # (the larger tiles)
    whole = g.score_plans(first, count).cpu().numpy()
    step = (1 << 20) + 13
    parts = [g.score_plans(first + i, min(step, count - i)).cpu().numpy() for i in range(0, count, step)]
    assert (np.concatenate(parts) == whole).all() and (whole[:-1] != whole[1:]).any()
    g.close()
