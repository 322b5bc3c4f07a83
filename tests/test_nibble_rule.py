"""What nibble 0 stands for on either side of the rule's edges, in the single-matrix and
in the batched solver (both call the function asked here), and that the tuner starts
from it.  No GPU needed."""
import ctypes
import os

import pytest

from paper_2002_05024_amd import autotune_single, binding

pytestmark = pytest.mark.skipif(not os.path.exists(binding.library_path()), reason="libneig.so not built")


@pytest.mark.parametrize("m,single,batched", [(97, 45, 45), (256, 45, 45), (257, 45, 20), (512, 45, 20),
                                              (513, 20, 20), (3000, 20, 20), (3001, 14, 20), (20000, 14, 20)])
def test_share_by_order(m, single, batched):
    lib = ctypes.CDLL(binding.library_path())
    assert lib.neig_default_nibble(m, 0) == single
    assert lib.neig_default_nibble(m, 1) == batched


def test_tuner_starts_from_the_default():
    for key, v in autotune_single.DEFAULT.items():
        assert v in autotune_single.GRID[key]
    assert autotune_single.DEFAULT["nibble"] == 0
