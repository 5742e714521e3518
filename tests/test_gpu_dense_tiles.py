"""The persistent 128 x 128 tiles of the whole-basis products.  A direction with
one condition at both walls of a symmetric grid runs half-size products, so
these problems have an open boundary (different conditions) in x and in y: no
mirror image, the whole basis."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import cuda, host, parity_error, say

pytestmark = pytest.mark.gpu

ND, DN = ("N", "D"), ("D", "N")


def _T():
    import paper_2603_09528_amd as T
    return T


# whole tiles; every extent ragged (edge tiles, and the K tail in the last step)
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [(128, 128, 11), (140, 124, 12)], ids=str)
def test_persistent_tiles_match_oracle(tmp_path, n, prec):
    """Four 64 x 64 waves and eight 64 x 32 waves, forced through the tuning
    table; FP32 also runs the accumulating epilogue with its norm partials."""
    T = _T()
    p = W.make_problem(n, (1.5, 2.0, 1.0), (ND, DN, W.NN))
    f = W.rhs(p, 14)
    ref = O.solve(p, f)
    gp = {"fp64": 0, "fp32": 1}[prec]
    nx, ny = n[0], n[1]
    table = tmp_path / "tiles.txt"
    try:
        for v in (6, 7):
            say("persistent tile", n, prec, v)
            table.write_text(f"{gp} 0 0 {nx} {nx} {v}\n{gp} 1 {ny} {nx} {ny} {v}\n")
            T.autotune_load(str(table))
            kw = {} if prec == "fp64" else {"precision": prec, "rtol": 1e-13, "max_refine": 12}
            plan = T.Plan.from_problem(p, **kw)
            assert plan.transforms == ("gemm", "gemm")
            err = parity_error(p, host(plan.solve(cuda(f))), ref)
            assert err <= (1e-12 if prec == "fp64" else 1e-10), (v, err)
            if prec == "fp32":
                info = plan.info()
                assert info.iters > 0 and 0.0 < info.rel_correction < 1e-10
    finally:
        # back to the persistent four-wave tile
        table.write_text(f"{gp} 0 0 {nx} {nx} 6\n{gp} 1 {ny} {nx} {ny} 6\n")
        T.autotune_load(str(table))


@pytest.mark.parametrize("prec,fixed", [("fp64", -1), ("fp32", 2)])
def test_small_batch_runs_one_persistent_launch_a_problem(prec, fixed):
    """Up to four problems whose GEMMs take a persistent tile run one launch per
    problem instead of one work list; bitwise those of the single solves."""
    import torch
    T = _T()
    probs = [(W.make_problem((128, 128, 12), (1.5, 2.0, 1.0), (ND, DN, W.NN)), 41),
             (W.make_problem((128, 256, 10), (2.0, 1.0, 1.5), (DN, ND, W.DD), kind="helmholtz", alpha=1e-3), 42),
             (W.make_problem((256, 128, 9), (1.0, 1.5, 2.0), (ND, ND, W.NN)), 43)]
    plans = [T.Plan.from_problem(p, precision=prec, fixed_refine=fixed) for p, _ in probs]
    rhs = [cuda(W.rhs(p, s)) for p, s in probs]
    singles = [host(pl.solve(r)) for pl, r in zip(plans, rhs)]
    b = T.Batch(plans)
    outs = [torch.empty_like(r) for r in rhs]
    for use_graph in (False, True, True):
        b.solve(rhs, outs, use_graph=use_graph)
        torch.cuda.synchronize()
        for i in range(len(probs)):
            assert np.array_equal(host(outs[i]), singles[i]), (i, use_graph)
    for i, (p, s) in enumerate(probs):
        err = parity_error(p, singles[i], O.solve(p, W.rhs(p, s)))
        assert err <= (1e-12 if prec == "fp64" else 1e-10), (i, err)
