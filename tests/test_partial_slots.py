"""The partial sums of an accumulating x inverse fit the workspace a plan asks
for, whatever tile runs: few long x lines make more tiles than any other grid
of their size.  CPU: the area behind the transform buffers against the tile
counts.  GPU: a solve in a workspace of exactly that size, with a guard behind
it, alone and as the last problem of a batch."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import cuda, host, parity_error, say


def _T():
    import paper_2603_09528_amd as T
    return T


# slots x lines of the tiles of half-size products: (modes of one parity, lines)
TILES = {"fp32": [(64, 128), (32, 128), (16, 64)], "bf16x3": [(64, 128), (32, 64)]}


def _al(x):
    return (x + 255) // 256 * 256


@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
@pytest.mark.parametrize("nx", [16, 250, 1600, 2000, 4000])
def test_workspace_holds_the_partials_of_every_tile(nx, prec):
    for ny, nz in ((1, 1), (2, 1), (1, 3), (2, 2), (5, 1), (2, 3), (7, 1), (2, 4)):
        # one unknown between Dirichlet walls: a face-located direction of two cells
        loc = ("C", "F" if ny == 1 else "C", "F" if nz == 1 else "C")
        p = W.make_problem((nx, max(ny, 2), max(nz, 2)), (0.0, 0.0, 0.0), (W.DD, W.DD, W.DD), loc=loc)
        plan = _T().Plan.from_problem(p, precision=prec, fixed_refine=2, host_only=True)
        lines = ny * nz
        assert plan.nxyz == (nx, ny, nz)
        n = nx * lines
        buffers = _al(8 * 2 * nx * ny * ((nz + 15) // 16)) + 3 * _al(4 * n)
        h = (nx + 1) // 2
        pairs = max(-(-h // s) * -(-lines // d) for s, d in TILES[prec])
        assert plan.workspace_bytes() - buffers >= 16 * pairs, (ny, nz, pairs)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
def test_few_long_lines_stay_in_the_workspace(prec):
    import torch
    T = _T()
    p = W.make_problem((2000, 2, 2), (0.0, 0.0, 0.0), (W.DD, W.NN, W.DD))
    q = W.make_problem((40, 24, 10), (1.0, 1.0, 1.0), (W.NN, W.DD, W.NN))
    fp, fq = W.rhs(p, 5), W.rhs(q, 6)
    kw = dict(precision=prec, fixed_refine=3)
    plan = T.Plan.from_problem(p, **kw)
    say("few long lines", prec)

    def guarded(nbytes):
        t = torch.full((nbytes + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        return t, t[:nbytes], t[nbytes:]

    whole, ws, guard = guarded(plan.workspace_bytes())
    one = host(plan.solve(cuda(fp), workspace=ws))
    assert bool((guard == 0xA5).all())
    assert parity_error(p, one, O.solve(p, fp)) <= 1e-10
    b = T.Batch([T.Plan.from_problem(q, **kw), T.Plan.from_problem(p, **kw)])
    whole, ws, guard = guarded(b.workspace_bytes())
    outs = [torch.empty(f.shape, dtype=torch.float64, device="cuda") for f in (fq, fp)]
    b.solve([cuda(fq), cuda(fp)], outs, use_graph=False, workspace=ws)
    torch.cuda.synchronize()
    assert bool((guard == 0xA5).all())
    assert np.array_equal(host(outs[1]), one)
    assert parity_error(q, host(outs[0]), O.solve(q, fq)) <= 1e-10
    assert b.info(0).rel_correction < 1e-4 and b.info(1).rel_correction < 1e-4
