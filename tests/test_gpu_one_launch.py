"""Matrices that are a small block from the start (one launch for the whole reduction)
at the edges of its layout: orders 1 to 96, leading dimensions larger than the order, a
given Z, blocks that are decoupled from the beginning, non-finite entries, and the first
order that takes the general path.  Bounds as for the batch: backward error and
orthogonality within 50 n eps, eigenvalues against the oracle."""
import numpy as np
import pytest

import test_gpu_batched as batched
from gpu_util import to_host
from paper_2002_05024_amd import binding as neig
from paper_2002_05024_amd import inputs

pytestmark = pytest.mark.gpu


def padded(M, pad):
    import torch

    n = M.shape[0]
    buf = torch.full((n, n + pad), 7.0, dtype=torch.float64, device="cuda")
    V = buf[:, :n].t()
    V.copy_(torch.from_numpy(np.ascontiguousarray(M)))
    return buf, V


@pytest.mark.parametrize("n,pad,cut", [
    (1, 0, 0), (2, 3, 0), (3, 0, 0), (15, 1, 0), (16, 0, 7), (17, 5, 0), (33, 0, 32), (64, 0, 0), (65, 2, 1),
    (80, 0, 40), (95, 7, 0), (96, 0, 48), (97, 1, 0),
])
def test_orders(n, pad, cut):
    neig.load_library()
    g = inputs.rng(inputs.NORMAL, 8800 + n)
    H = inputs.random_hessenberg(n, g)
    if cut:
        H[cut, cut - 1] = 0.0
    Q, _ = np.linalg.qr(g.standard_normal((n, n)))
    hbuf, Hd = padded(H, pad)
    zbuf, Zd = padded(Q, pad)
    r = neig.schur(Hd, Zd)
    st = neig.get_stats()
    assert r.info == 0
    S, Z = to_host(Hd), to_host(Zd)
    batched.check_problem(H, S, Q.T @ Z, r.wr.cpu().numpy(), r.wi.cpu().numpy(), None, f"n={n}")
    assert bool((hbuf[:, n:] == 7.0).all()) and bool((zbuf[:, n:] == 7.0).all())
    if 1 < n <= 96:
        assert 1 <= st["small_solves"] <= n and st["aeds"] == 0 and st["alg_flops"] > st["small_flops"] > 0


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_nonfinite(bad):
    neig.load_library()
    H = inputs.random_hessenberg(40, inputs.rng(inputs.NORMAL, 8700))
    H[3, 20] = bad
    _, Hd = padded(H, 0)
    with pytest.raises(neig.NeigError):
        neig.schur(Hd)
