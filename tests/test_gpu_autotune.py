"""Tuning again replaces what the table held, also where the fastest Thomas
kernel is an automatic choice without a number."""
import pytest

import workloads as W
from gpu_util import say

pytestmark = pytest.mark.gpu


def test_tuning_again_drops_a_slower_entry(tmp_path):
    import paper_2603_09528_amd as T
    # 131 072 lines of 150 planes: segments of 20, a configuration without a
    # number, against one lane a line
    p = W.make_problem((512, 256, 150), (0.0, 0.0, 1.0), (W.PP, W.PP, W.DD))
    table = tmp_path / "table.txt"
    table.write_text("0 2 131072 150 0 1\n")
    T.autotune_load(str(table))
    say("autotune", p.n)
    T.autotune([T.Plan.from_problem(p)])
    T.autotune_save(str(table))
    rows = [ln.split() for ln in table.read_text().splitlines() if ln.startswith("0 2 131072 150 ")]
    assert all(r[5] != "1" for r in rows), rows
