"""The chase windows at the edges of their layout: one to eight bulges per chain,
windows barely wider than a chain, of 63 to 96 rows (one or two columns per lane),
sweeps shorter than a batch of six steps, more bulges than one chain holds, blocks
that start at row 0, 1 or later and end before the last row.  Same checks and
bounds as the sweep test they call: backward error and orthogonality within
50 n eps, and the oracle's sequence of double steps by the implicit-Q theorem."""
import pytest

import test_gpu_parity as parity
from paper_2002_05024_amd import binding as neig

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,ktop,kbot,nbul,chain,chase_w", [
    (5, 0, 4, 1, 1, 8),
    (9, 0, 8, 1, 1, 8),
    (12, 1, 10, 2, 2, 8),
    (20, 0, 19, 1, 1, 8),
    (34, 2, 31, 5, 5, 17),
    (40, 0, 39, 3, 3, 12),
    (90, 0, 89, 8, 8, 26),
    (90, 5, 80, 8, 8, 27),
    (97, 0, 96, 6, 8, 63),
    (97, 1, 96, 8, 8, 64),
    (97, 1, 95, 8, 8, 65),
    (130, 3, 127, 7, 7, 66),
    (130, 0, 129, 8, 8, 95),
    (131, 2, 128, 8, 8, 96),
    (150, 0, 149, 12, 16, 96),
    (150, 4, 140, 11, 32, 64),
])
def test_sweep_windows(n, ktop, kbot, nbul, chain, chase_w):
    parity.test_sweep_implicit_q(neig, n, ktop, kbot, nbul, chain, chase_w)
