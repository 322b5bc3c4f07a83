"""Which sweeps overlap their far updates by themselves (overlap 0): from order 8192 on,
and only while a step's updates are not much longer than its chase launch.  The sweep is
the same similarity either way: backward error and orthogonality within 50 n eps."""
import numpy as np
import pytest
import torch

from gpu_util import gpu_backward_error, gpu_orthogonality
from paper_2002_05024_amd import binding as neig

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


# 9000 x chains x window per chase step: 5.8e4, 2.3e5; 4.8e4, 1.9e5
@pytest.mark.parametrize("n,shifts,chase_w,overlaps", [(8191, 64, 64, False), (9000, 64, 64, True),
                                                       (9000, 256, 64, False), (9000, 64, 96, True),
                                                       (9000, 256, 96, False)])
def test_automatic_overlap(n, shifts, chase_w, overlaps):
    neig.load_library()
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    H0 = torch.randn(n, n, dtype=torch.float64, device="cuda", generator=g).t()
    H0.triu_(-1)
    H = H0.t().clone().t()
    Z = torch.eye(n, dtype=torch.float64, device="cuda").t().contiguous().t()
    old = neig.get_params()
    try:
        neig.set_params(chain=0, chase_w=chase_w, overlap=0)
        neig.sweep(H, Z, 0, n - 1, np.linspace(-30.0, 30.0, shifts), np.zeros(shifts))
    finally:
        neig.set_params(**old)
    assert (neig.get_stats()["gemm_flops_far"] > 0) == overlaps
    assert gpu_backward_error(H0, H, Z) <= 50 * n * EPS
    assert gpu_orthogonality(Z) <= 50 * n * EPS
