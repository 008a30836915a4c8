"""Weight gradients by filter rows of 32 x 32 channels: ragged channels, segments of fewer than 8 pixels, volumes, pixel ranges of one K tile, of a
round of records and of several; layers of a network that share a launch with larger ones."""
import pytest

import test_gpu_contractions as contractions
from harness import stage_backward_isolated
from test_gpu_conv import G, G3
from test_gpu_fused import C, chain

pytestmark = pytest.mark.gpu

SHAPES = [
    G(1, 20, 15, 32, 32, 3, 1, 1),        # the last segment 7 wide
    G(1, 3, 8, 8, 24, 3, 1, 1),           # less than one K tile
    G(2, 20, 21, 24, 32, 3, 1, 1),        # ... 5 wide: three of them
    G(2, 18, 16, 32, 16, 3, 1, 0),        # no padding: output rows of 14
    G3(2, 3, 6, 8, 32, 32, 3, 1, 1),      # volume
    G(3, 33, 40, 16, 32, 3, 1, 1),        # several ranges
    G(24, 128, 120, 32, 32, 3, 1, 1),     # ranges of 34 K tiles: three rounds of records
]


@pytest.fixture(scope="module")
def lpm():
    import torch
    assert torch.cuda.is_available()
    import paper_2207_11019_amd as lpm
    return lpm


@pytest.mark.parametrize("g", SHAPES, ids=lambda g: contractions._id(("", g)))
def test_weight_gradients_of_32_channels(lpm, g):
    contractions.test_contractions(lpm, ("bf16", g))


def test_launch_shared_with_larger_tiles(lpm):
    """Bias gradients and scales of 32-channel layers beside 64-channel and 1x1 ones, one launch."""
    layers = chain(C(16, 32, 3, 3, 16, 16, p=1, scale=True), C(32, 32, 3, 3, 16, 16, p=1), C(32, 72, 3, 3, 16, 16, p=1, scale=True), C(72, 32, 1, 1, 16, 16),
                   C(32, 24, 3, 3, 16, 16, p=1, scale=True))
    stage_backward_isolated(lpm, layers, [0, 5], 6, 6, 1, seed=59, dx_wanted=True, check_forward=True, grad_std=1.0)
