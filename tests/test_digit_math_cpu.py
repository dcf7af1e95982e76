"""The digit arithmetic of the int8 products (i8_digits.hpp), compiled with g++
from the header that the kernels include: the digits are those of the rounded
values, int32 holds the sums (both asserted by the program), and the Gram
matrix of a panel is accurate enough for the pivot floor of the factorisation,
also where one row dominates the columns of the panel.  No GPU."""
import math
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = tmp_path_factory.mktemp("digits") / "digit_check"
    subprocess.run(["g++", "-std=c++17", "-O3", "-Wall", "-Wextra", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2512_13728_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "digit_check.cpp"), "-o", str(out)], check=True)
    return str(out)


def digit_gram(exe, P, kchunk, top=0):
    """P^T P by K slices of kchunk rows; top: the largest weight kept (0: the
    kernels' own)."""
    head = np.array([P.shape[0], P.shape[1], kchunk, top], np.int32).tobytes()
    out = subprocess.run([exe], input=head + np.ascontiguousarray(P).tobytes(), capture_output=True, check=True).stdout
    W = np.frombuffer(out).reshape(P.shape[1], P.shape[1])
    return np.triu(W) + np.triu(W, 1).T


def smallest_pivot(W):
    """The smallest Cholesky pivot over the floor 1e-13 max W_ii, rows of
    floored pivots dropped (as the factorisation does)."""
    A, fl, least = W.copy(), 1e-13 * W.diagonal().max(), np.inf
    for p in range(len(A)):
        d = A[p, p]
        least = min(least, d / fl)
        if d > fl:
            row = A[p, p + 1:] / np.sqrt(d)
            A[p + 1:, p + 1:] -= np.outer(row, row)
    return least


def panel(m, n, r, f, seed):
    """P~ = B Q of a buffer with one row f times the others."""
    g = np.random.default_rng(seed)
    B = 4 * g.standard_normal((m, 48)) @ g.standard_normal((48, n)) + 0.4 * g.standard_normal((m, n))
    B[7] *= f
    Q = np.linalg.qr(g.standard_normal((n, r)))[0]
    return B.astype(np.float32).astype(np.float64) @ Q.astype(np.float32).astype(np.float64)


# A column's largest value is within 2^-47 of its scale, so W is the Gram
# matrix of a panel whose column j is off by up to 2^-47 sqrt(K) max_j, which
# moves a pivot of at least sigma_min^2 by at most 2^-46 sqrt(K) kappa of itself
# (3e-5 here; the weights dropped add as much)
@pytest.mark.parametrize("m,n,r,kchunk,f", [
    (2048, 512, 256, 256, 1e5), (2048, 512, 256, 2048, 1e5), (1024, 1024, 96, 256, 2e5), (4096, 256, 128, 4096, 6e4),
])
def test_dominant_row_floors_no_pivot(exe, m, n, r, kchunk, f):
    P = panel(m, n, r, f, seed=r + kchunk)
    W = P.T @ P
    want = smallest_pivot(W)
    assert want > 2        # no pivot of the panel is near the floor
    got = smallest_pivot(digit_gram(exe, P, kchunk))
    bound = (2.0 ** -44 * np.sqrt(m) * np.linalg.cond(P) + 1e-3) * want   # 1e-3: the reference's own fp64 sums
    assert abs(got - want) <= bound, (got, want, bound)
    # without the squares of digit 3 the pivot is lost (below the floor but for the first)
    assert abs(smallest_pivot(digit_gram(exe, P, kchunk, 5)) - want) > 10 * bound


# On a Gaussian panel the diagonal has no bias: a column's rounding averages to
# 2^-46 max / (sqrt(K) rms) of W_jj, the weight dropped next to 2^-54 (max/rms)^2
def test_gaussian_diagonal_is_unbiased(exe):
    P = np.random.default_rng(3).standard_normal((4096, 64))
    W = np.array([math.fsum(c * c) for c in P.T])
    rel = (digit_gram(exe, P, 4096).diagonal() - W) / W
    assert np.abs(rel).max() < 3e-15 and abs(rel.mean()) < 1e-15, (np.abs(rel).max(), rel.mean())
    low = (digit_gram(exe, P, 4096, 5).diagonal() - W) / W
    assert low.mean() < -3e-14
