"""Smooth cyclic lines on uniform z: close to singular, with every row alike, so
that roundings of the diagonal add up.  The partitioned kernel carries row sums,
which stay exact: its result is off by the rounding of each elimination step, at
most 64 of 2^-53, relative to |A^-1| |f|, which for white noise is at most
sqrt(nz) times the solution."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import cuda, host, say

pytestmark = pytest.mark.gpu


def _lines(a, b, c, lam, f):
    """Cyclic lines (T + lam) x = f in long double: elimination of the line
    without its corner couplings, and the corner by a rank-one update."""
    L = np.longdouble
    a, b, c, f = (np.asarray(v, dtype=L) for v in (a, b, c, f))
    n = len(a)
    d = b[:, None] + np.asarray(lam, dtype=L)[None, :]
    g = -d[0]
    d[0] = d[0] - g
    d[n - 1] = d[n - 1] - c[n - 1] * a[0] / g

    def solve(r):
        p, x = np.zeros_like(d), r.copy()
        p[0], x[0] = c[0] / d[0], x[0] / d[0]
        for k in range(1, n):
            m = 1 / (d[k] - a[k] * p[k - 1])
            p[k], x[k] = c[k] * m, (x[k] - a[k] * x[k - 1]) * m
        for k in range(n - 2, -1, -1):
            x[k] -= p[k] * x[k + 1]
        return x

    u = np.zeros_like(d)
    u[0], u[n - 1] = g, c[n - 1]
    x, z = solve(f), solve(u)
    return x - (x[0] + a[0] * x[n - 1] / g) / (1 + z[0] + a[0] * z[n - 1] / g) * z


@pytest.mark.parametrize("stretched", [False, True])
@pytest.mark.parametrize("nz", [100, 256, 600, 1000])
def test_smooth_lines_keep_their_accuracy(nz, stretched):
    import torch
    import paper_2603_09528_amd as T
    rng = np.random.default_rng(nz)
    w = rng.uniform(0.5, 1.5, nz) if stretched else np.ones(nz)
    faces = np.concatenate([[0.0], np.cumsum(w)]) / w.sum()
    ops = O.operator_1d(faces, W.PP, "C")[:3]
    lamx = -np.repeat([1.0, 10.0, 1000.0], 32)
    f = rng.standard_normal((1, nz, 1, len(lamx)))
    say("cyclic sums", nz, stretched)
    x = torch.empty(f.shape, dtype=torch.float64, device="cuda")
    scratch = torch.empty(4 * len(lamx) * ((nz + 15) // 16), dtype=torch.float64, device="cuda")
    T.thomas(len(lamx), 1, nz, 1, cuda(lamx), cuda(np.zeros(1)), *(cuda(q) for q in ops), 0.0, 1.0, -1, cuda(f), x, scratch,
             periodic_z=True)
    ref = _lines(*ops, lamx, f[0, :, 0, :])
    diff = (host(x)[0, :, 0, :] - ref).astype(float).reshape(nz, 3, 32)
    size = ref.astype(float).reshape(nz, 3, 32)
    err = np.sqrt((diff ** 2).sum(axis=(0, 2)) / (size ** 2).sum(axis=(0, 2)))
    assert (err <= 64 * 2.0 ** -53 * np.sqrt(nz)).all(), err
