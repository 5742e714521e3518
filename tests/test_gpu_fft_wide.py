"""Fast transforms along y in wide blocks (512 threads; from two blocks for
every compute unit on) against the narrow ones: the same lines solved as a
problem of five right-hand sides (wide, with a partial last block) and of one
(too few lines for wide blocks).  Every block shape does the same arithmetic on
a line: bitwise equal."""
import numpy as np
import pytest

import workloads as W
from gpu_util import cuda, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("bcy", ["PP", "NN", "DD"])
@pytest.mark.parametrize("ny,nx,nz", [(512, 43, 41), (1024, 27, 31), (2048, 19, 23)])
def test_wide_blocks_match_narrow(ny, nx, nz, bcy, prec):
    import paper_2603_09528_amd as T
    kw = dict(kind="helmholtz", alpha=1e-3, implicit="yz")
    if prec != "fp64":
        kw = dict(kind="helmholtz", alpha=1e-3, precision=prec, fixed_refine=0)
    say("fft wide", ny, nx, nz, bcy, prec)
    p = W.make_problem((nx, ny, nz), (0.0, 0.0, 1.0), (W.PP, getattr(W, bcy), W.DD))
    f = W.rhs(p, 3)
    many = host(T.Plan(p.n, p.faces, p.bc, nrhs=5, **kw).solve(cuda(np.stack([f] * 5))))
    one = host(T.Plan(p.n, p.faces, p.bc, nrhs=1, **kw).solve(cuda(f)))
    assert all(np.array_equal(many[r], one) for r in range(5))
