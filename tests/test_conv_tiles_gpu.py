"""Convolutions with eight channel tiles to a workgroup (65 to 128 output channels) whose
input halo is staged whole: against the oracle, at the tolerances of test_nn_gpu."""
import pytest

import test_nn_gpu as T
from paper_1812_03358_amd import nn as NN

pytestmark = pytest.mark.gpu

# D, H, W, c0, c1, cout, ks, up: from 256 blocks of 16 x 4 x TZ voxels on for 32 and 64
# channels; edges of tiles and a last channel tile that is not full or is missing
CASES = [
    (9, 10, 19, 16, 0, 128, 3, 0),
    (6, 8, 34, 8, 8, 72, 3, 0),
    (32, 34, 49, 32, 0, 128, 3, 0),
    (32, 32, 64, 16, 16, 96, 3, 1),
    (32, 32, 33, 64, 0, 112, 3, 0),
]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_eight_channel_tiles(case):
    T.test_conv_forward_dgrad_wgrad(NN, case)
