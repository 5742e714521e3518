"""The automatic Thomas configuration at the ends of each configuration's line
lengths (one row over the one below, full, one short of it): plain and cyclic
lines, FP64 against the oracle's lines (1e-12, as the explicit variants), the
pinned line in place and many lines against the sequential kernel; FP32
storage through refined solves against the oracle (1e-10)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import cuda, host, parity_error, say

pytestmark = pytest.mark.gpu

EDGES = [65, 95, 96, 97, 129, 159, 160, 161, 191, 192, 193, 257, 319, 320, 321, 383, 384, 385, 513, 639, 640, 641, 767,
         768, 769]


def _lines(nx, ny, nz, nsys, seed, periodic):
    rng = np.random.default_rng(seed)
    faces = np.cumsum(np.concatenate([[0.0], rng.uniform(0.5, 1.5, nz)]))
    ops = O.operator_1d(faces, W.PP if periodic else W.DD, "C")[:3]
    return ops, -rng.uniform(0.1, 50.0, nx), -rng.uniform(0.1, 50.0, ny), rng.standard_normal((nsys, nz, ny, nx))


def _solve(ops, lamx, lamy, f, sigma=0.0, tau=1.0, pin=-1, periodic=False, variant=-1, in_place=False):
    import torch
    import paper_2603_09528_amd as T
    nsys, nz, ny, nx = f.shape
    df = cuda(f)
    x = df if in_place else torch.empty_like(df)
    scratch = torch.empty(4 * nx * ny * nsys * ((nz + 15) // 16), dtype=torch.float64, device="cuda")
    T.thomas(nx, ny, nz, nsys, cuda(lamx), cuda(lamy), *(cuda(a) for a in ops), sigma, tau, pin, df, x, scratch,
             periodic_z=periodic, variant=variant)
    torch.cuda.synchronize()
    return host(x)


@pytest.mark.parametrize("nz", EDGES)
@pytest.mark.parametrize("periodic", [False, True])
def test_lengths_match_oracle(nz, periodic):
    ops, lamx, lamy, f = _lines(11, 5, nz, 2, nz, periodic)
    lam = lamy[:, None] + lamx[None, :]
    say("thomas length", nz, periodic)
    for sigma, tau in ((0.0, 1.0), (1.0, -3e-3)):
        if periodic:
            ref = np.stack([O.solver.cyclic_lines(*ops, lam, sigma, tau, q) for q in f])
        else:
            ref = np.stack([O.thomas_lines(*ops, lam, sigma, tau, q)[0] for q in f])
        got = _solve(ops, lamx, lamy, f, sigma, tau, periodic=periodic)
        assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("nz", [90, 96, 150, 180, 310, 320, 384, 600, 700])
def test_pinned_line_in_place(nz):
    nx, ny = 9, 4
    faces = np.cumsum(np.concatenate([[0.0], np.random.default_rng(nz).uniform(0.5, 1.5, nz)]))
    ops = O.operator_1d(faces, W.NN, "C")[:3]
    _, lamx, lamy, f = _lines(nx, ny, nz, 1, nz + 1, False)
    lamx[3] = lamy[2] = 0.0
    pin = 3 + nx * 2
    say("thomas pinned", nz)
    ref = _solve(ops, lamx, lamy, f, pin=pin, variant=0)
    got = _solve(ops, lamx, lamy, f, pin=pin, in_place=True)
    assert got[0, -1, 2, 3] == 0.0
    # the pinned line's condition number is about nz^2
    assert np.abs(got - ref).max() <= max(1e-12, 1e-15 * nz * nz) * np.abs(ref).max()


@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("nz,lines", [(200, (320, 320)), (250, (1024, 257)), (300, (320, 320)), (300, (1024, 257)),
                                      (370, (1024, 257)), (450, (1024, 257)), (600, (320, 320))], ids=str)
def test_many_lines_match_sequential(nz, lines, periodic):
    ops, lamx, lamy, f = _lines(lines[0], lines[1], nz, 1, nz + 2, periodic)
    say("thomas many", nz, lines, periodic)
    ref = _solve(ops, lamx, lamy, f, periodic=periodic, variant=0)
    got = _solve(ops, lamx, lamy, f, periodic=periodic)
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("nz", [90, 160, 185, 250, 320, 380, 500, 630])
@pytest.mark.parametrize("bcz", ["DD", "PP"])
def test_fp32_storage(nz, bcz):
    import paper_2603_09528_amd as T
    p = W.make_problem((20, 24, nz), (1.0, 1.0, 1.0 if bcz == "DD" else 0.0), (W.NN, W.DD, getattr(W, bcz)))
    f = W.rhs(p, nz)
    say("thomas fp32", nz, bcz)
    got = host(T.Plan.from_problem(p, precision="fp32", fixed_refine=3).solve(cuda(f)))
    assert parity_error(p, got, O.solve(p, f)) <= 1e-10
