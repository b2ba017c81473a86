"""Costs of windows of rerouting plan indices where one stage lost nodes: tiles that begin and end inside a partition, the fewest
vectors a tile's table takes and one fewer, the nearest counts there are on either side of the most it takes (32 KB) and of those that
take the room of the partitions (8 KB), rows of four and eight entries, odd starts and counts, an output that is not 16-byte aligned,
every rule of the tile's size, few and many stages.  Against the oracle; whole numbers, compared exactly."""
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
    "496 vectors, 31 stages": (496, _case(34, 31, 4, 30, 9)),
    "528 vectors, 32 stages": (528, _case(35, 32, 4, 31, 30, hetero=True)),
    "2016 vectors": (2016, _case(18, 5, 4, 62, 2, hetero=True)),
    "2016 vectors, 24 stages": (2016, _case(27, 24, 4, 62, 7)),
    "2080 vectors": (2080, _case(18, 5, 4, 63, 2)),
    "five peers, 210 vectors": (210, _case(20, 9, 6, 6, 2)),
    "five peers, 330 vectors, 8 stages": (330, _case(20, 8, 6, 7, 2, hetero=True)),
    "five peers, 1001 vectors, 32 stages": (1001, _case(35, 32, 6, 10, 7, hetero=True)),
    "five peers, 1365 vectors": (1365, _case(16, 4, 6, 11, 2)),
    "five peers, eight orphans each": (495, _case(18, 4, 6, 8, 2, hetero=True, reroute_cap=0)),
}


@pytest.mark.parametrize("name", CASES)
def test_windows_against_the_oracle(name):
    import torch
    from paper_2508_21613_amd import binding as B
    vectors, sc = CASES[name]
    o, g = O.Scenario(sc), B.Scenario(sc)
    f = g.family(2)
    assert f["n_reroute"] == vectors
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


# windows that take the larger tiles, and how many of their plan indices do not
LARGE = {
    "153 vectors": (_case(34, 6, 4, 16, 2, hetero=True), (1 << 21) + 777, (1 << 20) + 13),
    "16 vectors": (_case(28, 8, 3, 15, 1), 256 * 3584 + 1001, 400009),
    "17 vectors, 20 stages": (_case(27, 20, 3, 16, 1, hetero=True), 256 * 4096 + 3, 400009),
    "31 vectors": (_case(34, 6, 3, 30, 1), 256 * 7680 + 4097, 1000003),
    "63 vectors, 12 stages": (_case(21, 12, 3, 62, 1), (1 << 21) + 511, 1000003),
    "64 vectors, 9 stages": (_case(26, 9, 3, 63, 1, hetero=True), (1 << 21) + 513, 1000003),
    "2016 vectors": (_case(34, 6, 4, 62, 2), 768 * 2048 * 9 + 12345, 1000003),
    "five peers, 1001 vectors, 24 stages": (_case(30, 24, 6, 10, 3), 768 * 2048 * 5 + 2047, 1000003),
}


@pytest.mark.parametrize("name", LARGE)
def test_large_window_is_its_small_ones(name):
    from paper_2508_21613_amd import binding as B
    sc, count, step = LARGE[name]
    g = B.Scenario(sc)
    f = g.family(2)
    first = f["offset"] + 100003
    assert 100003 + count <= f["n_part"] * f["n_reroute"]
    whole = g.score_plans(first, count).cpu().numpy()
    parts = [g.score_plans(first + i, min(step, count - i)).cpu().numpy() for i in range(0, count, step)]
    assert (np.concatenate(parts) == whole).all() and (whole[:-1] != whole[1:]).any()
    g.close()
