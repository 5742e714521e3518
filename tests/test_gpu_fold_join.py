"""Batches of small problems whose transform stages hold mirror-symmetric
directions and others: both kinds of tiles in one launch.  Every result is
bitwise that of the problem's own solve, and within 1e-12 of the oracle; sizes
at the edges of the tiles (16 slots, 64 and 128 lines, 8 and 16 columns a
step), one problem of either kind, and many."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import cuda, host, parity_error, say

pytestmark = pytest.mark.gpu

ND = ("N", "D")
M, D = (W.NN, W.DD), (ND, W.DD)   # x mirror-symmetric, x not
SETS = [
    [((16, 17, 9), M), ((17, 16, 9), D)],
    [((32, 33, 20), M), ((64, 31, 20), D), ((33, 32, 7), M)],
    [((31 + 7 * k, 96 - 5 * k, 30 + k), M if k % 2 else D) for k in range(8)],
    [((63, 64, 65), M), ((65, 63, 64), D), ((128, 20, 16), D), ((20, 128, 16), M)],
]


@pytest.mark.parametrize("probs", SETS, ids=lambda s: f"{len(s)}x{s[0][0][0]}")
@pytest.mark.parametrize("ymirror", [True, False])
def test_joined_stages_match_single_solves(probs, ymirror):
    import torch
    import paper_2603_09528_amd as T
    ps = [W.make_problem(n, (1.0, 1.2, 0.8), (bx, by if ymirror else ND, W.DD)) for n, (bx, by) in probs]
    plans = [T.Plan.from_problem(p) for p in ps]
    rhs = [W.rhs(p, 5 + i) for i, p in enumerate(ps)]
    dev = [cuda(f) for f in rhs]
    outs = [torch.empty_like(f) for f in dev]
    say("fold join", [p.n for p in ps], ymirror)
    T.Batch(plans).solve(dev, outs)
    torch.cuda.synchronize()
    for p, plan, f, d, o in zip(ps, plans, rhs, dev, outs):
        one = host(plan.solve(d))
        assert np.array_equal(host(o), one), p.n
        assert parity_error(p, one, O.solve(p, f)) <= 1e-12, p.n
