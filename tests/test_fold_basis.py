"""The basis that the FP64 half-size products hold is the eigenbasis to the
rounding of a double (host only).

Bound of the 2-norm of a held vector less the eigenvector: the rounding of the
pair's main parts, each 2^-53 of its norm, weighted by |c| + |s| <= 1.42; that of
the rotation's (c, s), 2^-53; the two BF16 terms of remainders of at most 5e-12,
2^-18 of them, 0.17 of 2^-53 on each of the pair.  In all 2.75 x 2^-53."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_09528_amd", "csrc")
BOUND = 2.75


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("fold") / "fold_basis_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", CSRC, os.path.join(ROOT, "tests", "fold_basis_check.cpp"),
                           os.path.join(CSRC, "host_ops.cpp"), "-o", exe])

    def run(*grid):
        out = subprocess.run([exe] + [str(v) for v in grid], check=True, capture_output=True, text=True).stdout.split()
        return None if out == ["whole"] else (float(out[0]), out[1] == "1")
    return run


# cells, stretching, lower end, length, condition (1 Neumann, 2 Dirichlet), location (0 centre, 1 face)
STRETCHED = [(64, 1.5, 0, 1, 1, 0), (256, 2.0, 0, 1, 1, 0), (448, 2.0, 0, 1, 1, 0), (384, 2.0, 0, 1, 2, 1), (256, 2.0, -1, 2, 2, 0),
             (256, 2.0, 10, 1, 1, 0), (512, 2.0, 8, 1, 1, 0), (96, 2.0, 30, 1, 1, 0), (97, 2.0, 30, 1, 2, 0)]


@pytest.mark.parametrize("grid", STRETCHED, ids=str)
def test_stretched_directions_keep_their_eigenvectors(check, grid):
    err, _ = check(*grid)
    assert err <= BOUND, err


# (no power of two: the faces i / n, and so the volumes, are equal to rounding only)
UNIFORM = [(383, 0, 0, 1, 2, 0), (383, 0, 3, 1, 2, 0), (96, 0, 0, 3.7, 1, 0), (333, 0, 2, 1, 0, 0), (300, 0, 0, 2, 2, 1), (90, 0, 0, 1, 0, 1)]


@pytest.mark.parametrize("grid", UNIFORM, ids=str)
def test_uniform_directions_keep_their_volumes(check, grid):
    err, corrected = check(*grid)
    assert err <= BOUND, err
    assert corrected


def test_symmetric_faces_need_no_remainders(check):
    assert check(256, 0, 0, 1, 2, 0)[1] is False
    assert check(96, 0, -48, 96, 1, 0)[1] is False


def test_larger_remainders_take_the_whole_basis(check):
    """Remainders past what the two terms hold to a double's rounding."""
    assert check(512, 2.0, 60, 1, 1, 0) is None
