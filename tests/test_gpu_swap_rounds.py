"""Rounds of concurrent block swaps: more pairs than one round takes (every second
row of a triangular form selected), all pairs of one type, mixed types, and the
window's edges, against the oracle's one-by-one swaps.  The eigenvalues are
separated by at least 0.01, so the order and the values are pinned: eigenvalues
within 1e-10 ||S||, backward error and orthogonality within 50 n eps."""
import numpy as np
import pytest

import oracle
from checks import EPS, backward_error, eigs, orthogonality, structure_violations
from gpu_util import to_dev, to_host
from paper_2002_05024_amd import binding as neig

pytestmark = pytest.mark.gpu


def form(sizes, seed):
    """A standardised Schur form with the given block sizes, eigenvalues apart."""
    g = np.random.default_rng(seed)
    n = int(np.sum(sizes))
    S = np.triu(g.standard_normal((n, n)) * 0.1 / np.sqrt(n), 1)
    place = g.permutation(len(sizes))
    j = 0
    for k, b in zip(place, sizes):
        re = -1.0 + 2.0 * (k + 0.5) / len(sizes)
        if b == 1:
            S[j, j] = re
        else:
            S[j, j] = S[j + 1, j + 1] = re
            S[j, j + 1], S[j + 1, j] = 0.5, -0.5
        j += b
    return np.asfortranarray(S)


@pytest.mark.parametrize("kind", ["ones", "twos", "mixed"])
@pytest.mark.parametrize("n", [2, 3, 5, 32, 64, 95, 96, 97, 130])
@pytest.mark.parametrize("select", ["alternate", "last", "random"])
def test_rounds(kind, n, select):
    g = np.random.default_rng(n)
    if kind == "ones":
        sizes = [1] * n
    elif kind == "twos":
        sizes = [2] * (n // 2) + [1] * (n % 2)
    else:
        sizes = []
        while sum(sizes) < n:
            sizes.append(min(int(g.integers(1, 3)), n - sum(sizes)))
    S = form(sizes, n + len(kind))
    at = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(int)
    sel = np.zeros(n, np.int32)
    if select == "alternate":
        sel[at[1::2]] = 1
    elif select == "last":
        sel[at[-1]] = 1
    else:
        sel[at[g.random(len(at)) < 0.5]] = 1
    Sd, Zd = to_dev(S), to_dev(np.eye(n))
    wr, wi, m, info = neig.reorder(Sd, Zd, sel)
    S0, Z0, wr0, wi0, m0, info0 = oracle.reorder(S, np.eye(n), sel)
    assert info == 0 and info0 == 0 and m == m0
    S1, Z1, wr, wi = to_host(Sd), to_host(Zd), wr.cpu().numpy(), wi.cpu().numpy()
    assert backward_error(S, S1, Z1) <= 50 * n * EPS
    assert orthogonality(Z1) <= 50 * n * EPS
    assert structure_violations(S1, wr, wi) == []
    assert np.max(np.abs(eigs(wr, wi) - eigs(wr0, wi0))) <= 1e-10 * np.linalg.norm(S)
