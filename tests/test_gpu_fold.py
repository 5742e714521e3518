"""Transforms of mirror-symmetric directions by two half-size products: sizes
around the edges of the tiles (modes of 16, 32 and 64 per parity, lines of 64
and 128, K steps of 8 and 16), odd and even lengths, every boundary condition
that is symmetric, against the oracle; larger grids, where the larger tiles
run, against the fast transforms of the same uniform directions."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import cuda, host, parity_error, say

pytestmark = pytest.mark.gpu


def _T():
    import paper_2603_09528_amd as T
    return T


TOL = {"fp64": 1e-12, "fp32": 1e-10, "bf16x3": 1e-10}

EDGE = [
    ((16, 17, 6), (1.5, 1.0, 1.0), (W.NN, W.DD, W.DD), "CCC"),
    ((31, 16, 5), (0.0, 2.0, 1.0), (W.PP, W.NN, W.NN), "CCC"),
    ((18, 33, 9), (0.0, 1.2, 0.5), (W.PP, W.DD, W.DD), "FFC"),
    ((63, 34, 7), (2.0, 0.0, 1.0), (W.DD, W.PP, W.NN), "CCC"),
    ((65, 66, 4), (1.0, 2.0, 1.0), (W.NN, W.NN, W.NN), "CCC"),
    ((129, 40, 6), (2.2, 1.0, 1.0), (W.DD, ("N", "D"), W.NN), "CCC"),
    ((20, 131, 5), (0.0, 2.5, 1.0), (("D", "N"), W.DD, W.DD), "CFC"),
    ((130, 127, 3), (0.0, 1.7, 1.0), (W.PP, W.NN, W.DD), "CCC"),
]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("case", EDGE, ids=lambda c: "x".join(map(str, c[0])))
def test_edges_match_oracle(case, prec):
    n, beta, bc, loc = case
    p = W.make_problem(n, beta, bc, loc=tuple(loc))
    f = W.rhs(p, 7)
    say(n, bc, loc, prec)
    kw = {} if prec == "fp64" else dict(precision=prec, rtol=1e-13, max_refine=12)
    plan = _T().Plan.from_problem(p, **kw)
    got = host(plan.solve(cuda(f)))
    err = parity_error(p, got, O.solve(p, f))
    assert err <= TOL[prec], err


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("n,bc", [((128, 256, 256), (W.NN, W.DD, W.NN)), ((256, 64, 520), (W.DD, W.NN, W.DD)),
                                  ((64, 128, 130), (W.PP, W.PP, W.DD))], ids=str)
def test_large_tiles_match_fast_transforms(n, bc, prec):
    """The same uniform problem with its dense bases (halved products) and by
    fast transforms, several right-hand sides: equal to the rounding of both
    (1e-12 relative; a mixed solve to its refinement target)."""
    p = W.make_problem(n, (0.0, 0.0, 1.5), bc)
    f = np.stack([W.rhs(p, 3 + i) for i in range(2)])
    kw = dict(nrhs=2) if prec == "fp64" else dict(nrhs=2, precision=prec, fixed_refine=4)
    T = _T()
    say(n, bc, prec)
    fast = T.Plan.from_problem(p, **kw)
    dense = T.Plan.from_problem(p, dense_x=True, dense_y=True, **kw)
    assert "gemm" not in fast.transforms and dense.transforms == ("gemm", "gemm")
    a, b = host(fast.solve(cuda(f))), host(dense.solve(cuda(f)))
    for i in range(2):
        err = parity_error(p, b[i], a[i])
        assert err <= TOL[prec], err


def test_nearly_symmetric_faces_take_whole_bases():
    """Faces symmetric only to 1e-9: no mirror direction, the whole basis."""
    p = W.make_problem((48, 36, 10), (1.5, 1.5, 1.0), (W.NN, W.DD, W.NN))
    for d in (0, 1):
        p.faces[d][3] *= 1 + 1e-9
    f = W.rhs(p, 9)
    got = host(_T().Plan.from_problem(p).solve(cuda(f)))
    assert parity_error(p, got, O.solve(p, f)) <= 1e-12
