"""The batched kernel at the edges of its layout: factors of 2 to 96 rows (every
number of row tiles, with and without a remainder), windows barely wider than a
chain, one bulge, a full chain, and one bulge more than a chain holds; orders that
leave remainders of the groups of sixteen vectors, and leading dimensions larger
than the order.  Same checks and bounds as the mixed-size batch (backward error,
orthogonality and structure within 50 n eps, eigenvalues against the oracle or the
prescribed spectrum)."""
import numpy as np
import pytest

import test_gpu_batched as batched
from gpu_util import to_host
from paper_2002_05024_amd import binding as neig

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nw,ns,nmin,chase_w,sizes", [
    (2, 2, 2, 5, [3, 4, 17, 40]),
    (15, 2, 9, 16, [10, 31, 33, 64]),
    (16, 4, 16, 17, [17, 48, 65, 112]),
    (17, 16, 17, 26, [18, 49, 95, 130]),
    (31, 16, 30, 48, [47, 81, 160]),
    (33, 18, 32, 49, [49, 97, 209]),
    (47, 32, 47, 64, [63, 127, 240]),
    (64, 32, 64, 80, [65, 128, 255]),
    (80, 24, 65, 81, [145, 161, 289]),
    (81, 30, 80, 95, [177, 257]),
    (95, 32, 95, 96, [96, 193, 300]),
    (96, 32, 96, 96, [97, 192, 321]),
])
def test_factor_and_window_sizes(nw, ns, nmin, chase_w, sizes):
    import torch

    neig.load_library()
    old = neig.get_batched_tune()
    Hs, spectra = batched.make_batch(sizes, 50 + nw)
    dev = []
    for i, H in enumerate(Hs):  # column-major with a padded leading dimension
        n = H.shape[0]
        buf = torch.zeros((n, n + i), dtype=torch.float64, device="cuda")
        M = buf[:, :n].t()
        M.copy_(torch.from_numpy(H))
        dev.append(M)
    try:
        neig.set_batched_tune([1 << 30], [nw], [ns], [nmin], [chase_w])
        c = neig.schur_batched(dev)
        torch.cuda.synchronize()
    finally:
        neig.set_batched_tune(old["n_hi"], old["nw"], old["ns"], old["nmin"], old["chase_w"])
    assert np.all(c.info.cpu().numpy() == 0)
    for i, H in enumerate(Hs):
        batched.check_problem(H, to_host(c.Hs[i]), to_host(c.Zs[i]), c.wrs[i].cpu().numpy(), c.wis[i].cpu().numpy(),
                              spectra[i], f"problem {i} n={H.shape[0]}")
