"""Partitioned cyclic Thomas lines (periodic z, the automatic choice from 16
planes on): line lengths at the edges of every configuration and where the
rows do not divide evenly among the segments, against the oracle's dense
per-line solve; the pinned line; the configurations of many lines against
the sequential kernel."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import cuda, host, say

pytestmark = pytest.mark.gpu


def _run(nx, ny, nz, f, lamx, lamy, ops, sigma=0.0, tau=1.0, pin=-1, variant=-1, in_place=False):
    import torch
    import paper_2603_09528_amd as T
    df = cuda(f)
    x = df if in_place else torch.empty_like(df)
    scratch = torch.empty(4 * nx * ny * f.shape[0] * ((nz + 15) // 16), dtype=torch.float64, device="cuda")
    T.thomas(nx, ny, nz, f.shape[0], cuda(lamx), cuda(lamy), *(cuda(a) for a in ops), sigma, tau, pin, df, x,
             scratch, periodic_z=True, variant=variant)
    torch.cuda.synchronize()
    return host(x)


def _operator(nz, seed):
    faces = np.cumsum(np.concatenate([[0.0], np.random.default_rng(seed).uniform(0.5, 1.5, nz)]))
    return O.operator_1d(faces, W.PP, "C")[:3]


@pytest.mark.parametrize("nz", [16, 17, 31, 32, 33, 50, 64, 65, 127, 128, 129, 200, 256, 257, 511, 513, 1000])
@pytest.mark.parametrize("sigma,tau", [(0.0, 1.0), (1.0, -3e-3)])
def test_matches_oracle(nz, sigma, tau):
    nx, ny, nsys = 13, 3, 2
    say("cyclic part", nz, sigma, tau)
    rng = np.random.default_rng(nz)
    ops = _operator(nz, nz)
    lamx, lamy = -rng.uniform(0.0, 50.0, nx), -rng.uniform(0.1, 50.0, ny)
    f = rng.standard_normal((nsys, nz, ny, nx))
    lam = lamy[:, None] + lamx[None, :]
    ref = np.stack([O.solver.cyclic_lines(*ops, lam, sigma, tau, q) for q in f])
    got = _run(nx, ny, nz, f, lamx, lamy, ops, sigma, tau)
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("nz", [16, 33, 100, 250, 300])
def test_pinned_line_in_place_matches_sequential(nz):
    nx, ny = 9, 4
    rng = np.random.default_rng(nz + 1)
    ops = _operator(nz, nz + 1)
    lamx, lamy = -rng.uniform(1.0, 20.0, nx), -rng.uniform(1.0, 20.0, ny)
    lamx[3] = lamy[2] = 0.0
    f = rng.standard_normal((1, nz, ny, nx))
    pin = 3 + nx * 2
    say("cyclic part pinned", nz)
    ref = _run(nx, ny, nz, f, lamx, lamy, ops, pin=pin, variant=0)
    got = _run(nx, ny, nz, f, lamx, lamy, ops, pin=pin, in_place=True)
    assert got[0, -1, 2, 3] == 0.0
    # the pinned line's condition number is about nz^2: 1e-13 nz^2 of its size
    assert np.abs(got - ref).max() <= max(1e-12, 1e-15 * nz * nz) * np.abs(ref).max()


@pytest.mark.parametrize("nz", [131, 260])
def test_many_lines_match_sequential(nz):
    nx, ny = 1024, 260
    rng = np.random.default_rng(nz + 2)
    ops = _operator(nz, nz + 2)
    lamx, lamy = -rng.uniform(0.0, 50.0, nx), -rng.uniform(0.1, 50.0, ny)
    f = rng.standard_normal((1, nz, ny, nx))
    say("cyclic part many", nz)
    ref = _run(nx, ny, nz, f, lamx, lamy, ops, variant=0)
    got = _run(nx, ny, nz, f, lamx, lamy, ops)
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()
