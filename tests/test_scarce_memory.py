"""Large searches when the tables they would lay out cannot be allocated (they run on the kernels that need none and return
the same plans), and after a search whose wait failed (its tables count as laid out only once their search has been waited
for).  tests/c_client/scarce.c brings both about from the host."""
import os
import subprocess

import pytest

from oracle import oracle as O
from paper_2508_21613_amd import synth

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_search_without_memory_for_its_tables(tmp_path):
    from paper_2508_21613_amd import binding as B
    L, PP, DP = 32, 8, 2
    fwd, bwd, mem = synth.layer_tables(77, L)
    sc = synth.scenario(L, PP, DP, 9, fwd, bwd, mem, [3], 150, 8000)
    assert B.halves_selection(sc, 0)[0] and B.halves_selection(sc, 2)[0]
    exe = tmp_path / "scarce"
    lib_dir = os.path.join(ROOT, "paper_2508_21613_amd")
    subprocess.run(["gcc", "-std=c99", "-O1", "-Wall", "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "c_client", "scarce.c"),
                    "-o", str(exe), "-rdynamic", "-L", lib_dir, "-lchm", "-ldl", "-Wl,-rpath," + lib_dir], check=True)
    out = subprocess.run([str(exe)] + [str(int(x)) for a in (fwd, bwd, mem) for x in a], check=True, capture_output=True, text=True,
                         timeout=120).stdout.splitlines()
    scarce, plenty = [x[7:] for x in out if x.startswith("scarce ")], [x[7:] for x in out if x.startswith("plenty ")]
    assert len(scarce) == 4 and scarce == plenty and all(x.startswith("rc=0 ") for x in scarce), out
    assert int([x for x in out if x.startswith("refused")][0].split()[1]) > 0      # (the tables were asked for)
    # failed wait, next search, search on finished tables: kernels launched
    (failed, rc_f), (again, rc_a), (settled, rc_s) = [(int(x.split()[1]), x.split()[2]) for x in out if x.startswith("launches")]
    tables = sum(B.halves_selection(sc, k)[0] > 0 for k in range(3))
    assert (rc_f, rc_a, rc_s) == ("rc=-6", "rc=0", "rc=0"), out
    assert (again, settled) == (failed + 1, failed - tables), out        # (+ 1: the search's words are filled afresh, too)
    assert [x[6:] for x in out if x.startswith("after ")] == [plenty[3]] * 2
    g, o = B.Scenario(sc), O.Scenario(sc)
    for line, mask in zip(scarce, (1, 2, 4, 7)):
        rc, b = g.search_best(mask)
        assert line == "rc=%d index=%d cost=%d strategy=%d t_step=%d t_trans=%d" % (rc, b["index"], b["cost"], b["strategy"], b["t_step_us"], b["t_trans_us"])
        assert int(o.score(b["index"], 1)[0]) == b["cost"]
    g.close()
