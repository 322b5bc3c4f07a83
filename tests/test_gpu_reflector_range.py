"""Bulge reflectors whose generating vector is far smaller than other entries of the
same rows: a matrix of entries around 2^316 with one entry of 2^714 far right of the
diagonal, through each path that chases bulges (the in-LDS QR, deflation windows, the
sweep's windows, the batched solver).  The products of a reflector's vector with such
an entry must not leave the range.  One entry dominates the norm, so backward error and
orthogonality within 50 n eps are the bounds (eigenvalues so far below eps times the
norm need not converge, and are not asked to)."""
import numpy as np
import pytest
import torch

from checks import EPS, backward_error, orthogonality
from gpu_util import to_dev, to_host
from paper_2002_05024_amd import binding as neig

pytestmark = pytest.mark.gpu
LOW, HIGH = 316, 714


def matrix(n, r, c, sign=1):
    """Entries about 2^(+-LOW), and 2^HIGH (or its reverse) at (r, c)."""
    H = np.triu(np.random.default_rng(n).standard_normal((n, n)), -1)
    H = np.ldexp(H, sign * LOW)
    H[r, c] = np.ldexp(1.0, HIGH)
    return H


def check(H, S, Z):
    n = H.shape[0]
    assert np.isfinite(S).all() and np.isfinite(Z).all()
    down = np.ldexp(1.0, -HIGH)
    assert backward_error(H * down, S * down, Z) <= 50 * n * EPS
    assert orthogonality(Z) <= 50 * n * EPS


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("n", [20, 40, 64, 65, 96])
def test_small_block(n, sign):
    H = matrix(n, 0, n - 1, sign)
    Hd = to_dev(H)
    r = neig.small_schur(Hd)
    check(H, to_host(Hd), to_host(r.Z))


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("n,r,c", [(300, 0, 80), (300, 120, 190)])
def test_sweep(n, r, c, sign):
    H = matrix(n, r, c, sign)
    Hd, Zd = to_dev(H), to_dev(np.eye(n))
    s = np.ldexp(np.linspace(-1.0, 1.0, 16), sign * LOW)
    assert neig.sweep(Hd, Zd, 0, n - 1, s, np.zeros(16)) == 0
    check(H, to_host(Hd), to_host(Zd))


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("nw", [48, 90])
def test_deflation_window(nw, sign):
    n = 200
    H = matrix(n, n - nw, n - 1, sign)
    Hd, Zd = to_dev(H), to_dev(np.eye(n))
    neig.aed(Hd, Zd, 0, n - 1, nw)
    check(H, to_host(Hd), to_host(Zd))


@pytest.mark.parametrize("sign", [1, -1])
def test_batched(sign):
    Hs = [matrix(n, 0, n - 1, sign) for n in (40, 96, 150, 260)]
    out = neig.schur_batched([to_dev(H) for H in Hs])
    torch.cuda.synchronize()
    for H, s, z in zip(Hs, out.Hs, out.Zs):
        check(H, to_host(s), to_host(z))


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("n", [30, 250])
def test_whole_reduction(n, sign):
    H = matrix(n, 0, n - 1, sign)
    Hd = to_dev(H)
    r = neig.schur(Hd)
    check(H, to_host(Hd), to_host(r.Z))


@pytest.mark.parametrize("n", [40, 96])
def test_shifts_out_of_range(n):
    """Entries around 2^1005: the determinant of a shift pair overflows, and the block
    does not converge.  It stays a similarity, however many sweeps were tried."""
    H = np.ldexp(np.triu(np.random.default_rng(1000 * n).standard_normal((n, n)), -1), 1005)
    Hd = to_dev(H)
    r = neig.small_schur(Hd)
    S, Z = to_host(Hd), to_host(r.Z)
    down = np.ldexp(1.0, -1005)
    assert backward_error(H * down, S * down, Z) <= 50 * n * EPS
    assert orthogonality(Z) <= 50 * n * EPS
