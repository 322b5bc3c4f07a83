"""The in-LDS double-shift QR at the orders where its layout changes: one vector
per lane up to order 64 and two above, batches of 15 reflectors handed to the
waves that accumulate the factor, active blocks of three rows; and entries so
large or small that a generating vector's squares leave the range of the fast
reflector.  Bounds as elsewhere: 50 n eps for the backward error and the
orthogonality, 1e-10 ||H|| cond for eigenvalues that the oracle pins."""
import numpy as np
import pytest

import oracle
from checks import EPS, backward_error, orthogonality, structure_violations
from gpu_util import to_dev, to_host
from paper_2002_05024_amd import binding as neig
from paper_2002_05024_amd import inputs

pytestmark = pytest.mark.gpu


def check_schur(H, S, Z, wr, wi):
    n = H.shape[0]
    assert backward_error(H, S, Z) <= 50 * n * EPS
    assert orthogonality(Z) <= 50 * n * EPS
    assert structure_violations(S, wr, wi) == []


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 15, 16, 17, 18, 31, 32, 33, 62, 63, 64, 65, 66, 67, 80, 95, 96])
def test_small_schur_orders(n):
    H = inputs.random_hessenberg(n, inputs.rng(inputs.PLAIN, 9000 + n))
    Hd = to_dev(H)
    r = neig.small_schur(Hd)
    assert r.info == 0
    check_schur(H, to_host(Hd), to_host(r.Z), r.wr.cpu().numpy(), r.wi.cpu().numpy())
    S0, _, wr0, wi0, info0 = oracle.schur(H)
    assert info0 == 0
    cond = oracle.cond(S0)
    lam, lam0 = r.wr.cpu().numpy() + 1j * r.wi.cpu().numpy(), wr0 + 1j * wi0
    used = np.zeros(n, dtype=bool)
    for k in np.argsort(cond):
        if cond[k] >= 1e10:
            continue
        d = np.abs(lam - lam0[k])
        d[used] = np.inf
        j = int(np.argmin(d))
        used[j] = True
        assert d[j] <= 1e-10 * np.linalg.norm(H) * cond[k], (n, k, d[j], cond[k])


@pytest.mark.parametrize("n", [7, 40, 70])
@pytest.mark.parametrize("exponent", [-500, -340, 340, 500])
def test_small_schur_scaled(n, exponent):
    H = inputs.random_hessenberg(n, inputs.rng(inputs.PLAIN, 9200 + n))
    Hd = to_dev(np.ldexp(H, exponent))
    r = neig.small_schur(Hd)
    assert r.info == 0
    S = np.ldexp(to_host(Hd), -exponent)
    check_schur(H, S, to_host(r.Z), np.ldexp(r.wr.cpu().numpy(), -exponent), np.ldexp(r.wi.cpu().numpy(), -exponent))


@pytest.mark.parametrize("n", [5, 33, 66])
def test_small_schur_zero_vectors(n):
    """A block whose bulge vectors vanish: the cyclic shift (its first sweep has
    zero shifts) and a matrix with one exactly zero superdiagonal part."""
    C = inputs.cyclic_shift(n)
    Hd = to_dev(C)
    r = neig.small_schur(Hd)
    assert r.info == 0
    S, Z = to_host(Hd), to_host(r.Z)
    assert np.linalg.norm(C - Z @ S @ Z.T) <= 50 * n * EPS * np.linalg.norm(C)
    lam = np.sort_complex(np.round(r.wr.cpu().numpy() + 1j * r.wi.cpu().numpy(), 8))
    ref = np.sort_complex(np.round(np.exp(2j * np.pi * np.arange(n) / n), 8))
    assert np.allclose(lam, ref, atol=1e-7)
