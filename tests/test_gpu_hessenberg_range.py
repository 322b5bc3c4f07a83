"""Hessenberg reduction of finite inputs whose columns lie far from the rest of the
matrix: a first column far below max |A| (its reflector has entries of ordinary size
all the same), and first columns whose tail is subnormal, beside an ordinary subdiagonal
entry and beside a zero one.  Orders on both sides of 4096, where the column kernels
and the matrix-vector product change their tiles.  A Householder reduction is backward
stable column by column whatever the columns' sizes, so the bounds are the ones of the
other Hessenberg tests: backward error and orthogonality within 50 n eps.  (Entries at
1e-310 carry 5e-14 relative; that is below 50 n eps from n = 5 on.)"""
import numpy as np
import pytest
import torch

from gpu_util import gpu_backward_error, gpu_orthogonality
from paper_2002_05024_amd import binding as neig

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52
ORDERS = [60, 130, 1030, 4100]


def normal(n, seed):
    g = np.random.default_rng(seed)
    return g.standard_normal((n, n)) / np.sqrt(n)


def reduce(A):
    """H and Q1 on the GPU, and whether both are finite."""
    Ad = neig.colmajor(A, "cuda:0")
    Q = neig.hessenberg(Ad)
    return Ad, Q, bool(torch.isfinite(Ad).all()) and bool(torch.isfinite(Q).all())


@pytest.mark.parametrize("n", ORDERS)
@pytest.mark.parametrize("big,small", [(66, -997), (664, -392), (664, -498), (900, -300), (0, -1010)])
def test_column_far_below_the_matrix(n, big, small):
    """max |A| about 2^big, the first column about 2^small."""
    A = np.ldexp(normal(n, n), big)
    A[:, 0] = np.ldexp(normal(n, n)[:, 0], small)
    H, Q, finite = reduce(A)
    assert finite
    down = [neig.colmajor(np.ldexp(M, -big), "cuda:0") for M in (A, H.cpu().numpy())]
    assert gpu_backward_error(*down, Q) <= 50 * n * EPS
    assert gpu_orthogonality(Q) <= 50 * n * EPS


@pytest.mark.parametrize("n", ORDERS)
@pytest.mark.parametrize("alpha", [1.0, 0.0, 3e-310])
def test_subnormal_tail(n, alpha):
    A = normal(n, n + 1)
    A[1, 0] = alpha
    A[2:, 0] *= np.sqrt(n) * 1e-310
    H, Q, finite = reduce(A)
    assert finite
    assert gpu_backward_error(neig.colmajor(A, "cuda:0"), H, Q) <= 50 * n * EPS
    assert gpu_orthogonality(Q) <= 50 * n * EPS


def test_subnormal_tails_of_a_hessenberg_matrix():
    """A Hessenberg matrix with entries of 1e-309 below the subdiagonal, in every column:
    rapidly decaying kernels underflow to these."""
    n = 130
    A = np.triu(normal(n, 5), -1) + np.tril(np.full((n, n), 1e-309), -2)
    H, Q, finite = reduce(A)
    assert finite
    assert gpu_backward_error(neig.colmajor(A, "cuda:0"), H, Q) <= 50 * n * EPS
    assert gpu_orthogonality(Q) <= 50 * n * EPS
