"""The Hessenberg reduction where its tiles change: 64- and 128-row workgroups of
the column kernels, chunk widths of the matrix-vector product (trailing blocks of
1024, 2048, 4096 rows), and inputs whose squares leave the range.  Bounds as in
the other Hessenberg tests: against the oracle H within 10 n eps ||A||_F and Q1
within 50 n eps; at sizes where the oracle takes too long, backward error and
orthogonality within 50 n eps."""
import numpy as np
import pytest
import torch

import oracle
from checks import EPS, backward_error, orthogonality
from gpu_util import gpu_backward_error, gpu_orthogonality, to_dev, to_host
from paper_2002_05024_amd import binding as neig
from paper_2002_05024_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [6, 63, 68, 127, 128, 130, 257, 1026])
def test_against_oracle(n):
    A = inputs.rng(90, n).standard_normal((n, n))
    H0, Q0 = oracle.hessenberg(A)
    Ad = to_dev(A)
    Q1 = to_host(neig.hessenberg(Ad))
    assert np.abs(to_host(Ad) - H0).max() <= 10 * n * EPS * np.linalg.norm(A)
    assert np.abs(Q1 - Q0).max() <= 50 * n * EPS


@pytest.mark.parametrize("n", [1025, 2049, 2051, 4097, 4099, 4225])
def test_sizes(n):
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    A = torch.empty(n, n + 3, dtype=torch.float64, device="cuda")[:, :n].t()  # padded leading dimension
    A.copy_(torch.randn(n, n, dtype=torch.float64, device="cuda", generator=g))
    A0 = A.clone()
    Q = neig.hessenberg(A)
    assert float(torch.tril(A, -2).abs().max()) == 0.0
    assert gpu_backward_error(A0, A, Q) <= 50 * n * EPS
    assert gpu_orthogonality(Q) <= 50 * n * EPS


@pytest.mark.parametrize("exponent", [-900, -500, 500, 900])
def test_scaled(exponent):
    """Scaling by a power of two changes nothing but the scale."""
    n = 150
    A = inputs.rng(89, n).standard_normal((n, n))
    H0, Q0 = oracle.hessenberg(A)
    Ad = to_dev(np.ldexp(A, exponent))
    Q1 = to_host(neig.hessenberg(Ad))
    assert np.abs(np.ldexp(to_host(Ad), -exponent) - H0).max() <= 10 * n * EPS * np.linalg.norm(A)
    assert np.abs(Q1 - Q0).max() <= 50 * n * EPS


def test_graded_columns():
    """Columns scaled over 240 decades: every reflector has its own range.  The
    form is not unique to rounding here (its later columns come from the noise of
    the first), so it is checked by its backward error and orthogonality."""
    n = 120
    A = inputs.rng(88, n).standard_normal((n, n)) * 10.0 ** np.linspace(0, -240, n)[None, :]
    Ad = to_dev(A)
    Q1 = to_host(neig.hessenberg(Ad))
    H1 = to_host(Ad)
    assert backward_error(A, H1, Q1) <= 50 * n * EPS
    assert orthogonality(Q1) <= 50 * n * EPS
