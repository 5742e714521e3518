"""FP32 batches whose transform stages hold mirror-symmetric directions and
others: both kinds of tiles in one launch, with the accumulating epilogue and
its norm partials in the corrections.  Bitwise the single solves; sizes at the
edges of the tiles, few tiles (16 x 64) and many (32 x 128)."""
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
    [((127, 128, 65), M), ((130, 63, 64), D), ((128, 96, 60), D), ((64, 129, 70), M)],
]


@pytest.mark.parametrize("probs", SETS, ids=lambda s: f"{len(s)}x{s[0][0][0]}")
@pytest.mark.parametrize("ymirror", [True, False])
def test_joined_stages_match_single_solves(probs, ymirror):
    import torch
    import paper_2603_09528_amd as T
    ps = [W.make_problem(n, (1.0, 1.2, 0.8), (bx, by if ymirror else ND, W.DD)) for n, (bx, by) in probs]
    plans = [T.Plan.from_problem(p, precision="fp32", fixed_refine=2) for p in ps]
    rhs = [W.rhs(p, 5 + i) for i, p in enumerate(ps)]
    dev = [cuda(f) for f in rhs]
    outs = [torch.empty_like(f) for f in dev]
    say("fold join fp32", [p.n for p in ps], ymirror)
    b = T.Batch(plans)
    b.solve(dev, outs)
    torch.cuda.synchronize()
    for i, (p, plan, f, d, o) in enumerate(zip(ps, plans, rhs, dev, outs)):
        one = host(plan.solve(d))
        assert np.array_equal(host(o), one), p.n
        assert parity_error(p, one, O.solve(p, f)) <= 1e-10, p.n
        # the sums behind the ratio in another order: 2^-53 times their count's logarithm
        assert abs(b.info(i).rel_correction / plan.info().rel_correction - 1.0) <= 1e-13, p.n
