"""FP64 half-size products of bases with remainders don't depend on the size of
the field: f scaled by a power of two has the scaled solution.

Every FP64 rounding scales exactly; what may differ is the remainders' part,
2^-54.5 of a line's values in each of the four passes at most, and with it the
rounding of the sum it is added to, 2^-53.  Cells differ by 13 in size, so the
norm in which a pass keeps lengths and the plain one by at most 3.6:
4 * (2^-53 + 2^-54.5) * 3.6 = 2.2e-15 of f, which here is at most twice u."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import cuda, host, parity_error, say

pytestmark = pytest.mark.gpu


def _T():
    import paper_2603_09528_amd as T
    return T


# one per tile (16 x 64, 64 x 64, 32 x 128); faces away from the origin, whose
# rounding leaves large remainders; odd lengths, face-located y
GRIDS = [((97, 76, 20), "CFC", 30.0), ((256, 200, 64), "CCC", 8.0), ((448, 384, 16), "CFC", 0.0)]


def _problem(n, loc, lower=0.0):
    p = W.make_problem(n, (2.0, 2.0, 1.0), (W.NN, W.DD, W.DD), loc=tuple(loc), kind="helmholtz", alpha=1e-6)
    for d in (0, 1):
        p.faces[d][:] = p.faces[d] + lower
    return p


@pytest.mark.parametrize("n,loc,lower", GRIDS, ids=str)
def test_scaled_fields_have_scaled_solutions(n, loc, lower):
    p = _problem(n, loc, lower)
    f = W.rhs(p, 21)
    plan = _T().Plan.from_problem(p)
    one = host(plan.solve(cuda(f)))
    assert np.linalg.norm(f) <= 2 * np.linalg.norm(one)
    if n[0] < 256:
        assert parity_error(p, one, O.solve(p, f)) <= 1e-12
    for k in (-400, -200, -90, 90, 200, 400):
        say(n, loc, "2^%d" % k)
        got = np.ldexp(host(plan.solve(cuda(np.ldexp(f, k)))), -k)
        err = np.linalg.norm(got - one) / np.linalg.norm(one)
        assert err <= 4.4e-15, (k, err)


def test_lines_of_every_size_agree_between_tiles():
    """Planes of very different size in one field: the same bits from a batch,
    whose tiles are other ones, as from single solves."""
    import torch
    T = _T()
    probs = [_problem(n, loc) for n, loc in (((192, 160, 24), "CFC"), ((48, 37, 20), "CCC"), ((40, 300, 12), "CCC"))]
    plans = [T.Plan.from_problem(p) for p in probs]
    rhs = []
    for i, p in enumerate(probs):
        f = W.rhs(p, 31 + i)
        for z in range(f.shape[0]):
            f[z] = np.ldexp(f[z], (0, -300, 150, -70, 0, 300)[z % 6])
        rhs.append(cuda(f))
    singles = [host(pl.solve(r)) for pl, r in zip(plans, rhs)]
    assert all(np.isfinite(s).all() for s in singles)
    outs = [torch.empty_like(r) for r in rhs]
    T.Batch(plans).solve(rhs, outs, use_graph=False)
    torch.cuda.synchronize()
    for o, s in zip(outs, singles):
        assert np.array_equal(host(o), s)


def test_infinite_and_nan_lines_stay_where_they_are():
    """y lines alone (implicit y and z on one plane): a line that holds an
    infinity or a NaN has no finite result, and no other line changes."""
    T = _T()
    p = W.make_problem((96, 72, 2), (1.0, 2.0, 1.0), (W.PP, W.NN, W.DD), kind="helmholtz", alpha=1e-6)
    f = W.rhs(p, 41)
    plan = T.Plan.from_problem(p, implicit="yz")
    one = host(plan.solve(cuda(f)))
    bad = f.copy()
    bad[1, 5, 3], bad[0, 70, 40], bad[1, 36, 64] = np.inf, np.nan, -np.inf
    got = host(plan.solve(cuda(bad)))
    lines = np.zeros(p.n[0], bool)
    lines[[3, 40, 64]] = True
    assert not np.isfinite(got[:, :, lines]).all(axis=(0, 1)).any()
    assert np.array_equal(got[:, :, ~lines], one[:, :, ~lines])
