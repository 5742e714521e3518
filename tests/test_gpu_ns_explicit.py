"""The explicit-terms kernel of the Navier--Stokes substep at the edges of its
tiles: rows shorter than a wave, as long, one longer (x neighbours come from
the lanes beside), walls and wrapped rows at every place of a wave, chunks of
z planes that do not divide the planes, two cells a direction.  The explicit
terms E^k and the velocity of each substep against the oracle, with the bound
1e-11 max|ref| of the other substep tests (the pressure of such flat grids is
conditioned worse than that and is not this kernel's)."""
import numpy as np
import pytest

import workloads as W
from oracle import navier_stokes as NS
from gpu_util import cuda, host, say
from test_gpu_navier_stokes import TOL, _state

pytestmark = pytest.mark.gpu

P, N = W.PP, W.NN


@pytest.mark.parametrize("implicit", ["none", "yz"])
@pytest.mark.parametrize("n,bc", [
    ((2, 2, 2), (N, N, N)), ((3, 2, 9), (P, N, N)), ((63, 5, 4), (P, P, N)), ((64, 4, 5), (P, N, P)),
    ((64, 7, 33), (N, P, N)), ((65, 3, 34), (P, N, N)), ((65, 6, 3), (N, N, P)), ((129, 3, 2), (P, P, N)),
    ((257, 2, 13), (N, N, N)), ((96, 97, 65), (N, P, P)),
], ids=str)
def test_tile_edges(n, bc, implicit):
    import torch
    import paper_2603_09528_amd as T
    nu, dt = 0.02, 1e-3
    p = W.make_problem(n, tuple(0.0 if b == P else 1.0 for b in bc), bc)
    ns = T.NavierStokes(T.Plan.from_problem(p), nu, dt, implicit)
    vel, pr = _state(p, 21)
    dvel, dpr = [cuda(a) for a in vel], cuda(pr)
    de = tuple(torch.zeros_like(a) for a in dvel)
    e = (None, None, None)
    for k in (1, 2, 3):
        say("ns explicit", n, bc, implicit, "k", k)
        ns.substep(k, *dvel, de, dpr)
        torch.cuda.synchronize()
        vel, e, pr, _ = NS.rk3_substep(p, k, dt, nu, implicit, *vel, e, pr)
        for name, got, ref in zip(("u", "v", "w", "eu", "ev", "ew"), (*dvel, *de), (*vel, *e)):
            err = np.abs(host(got) - ref).max()
            assert err <= TOL * np.abs(ref).max(), (k, name, err / np.abs(ref).max())
