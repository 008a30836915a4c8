"""Contractions of a group of lanes per output: filters that cover their input, reductions of less than a turn of the lanes, of whole eights of turns
and not, strides; and max-pooling of channels that are no whole 16-byte chunks."""
import pytest

import test_gpu_contractions as contractions
from harness import stage_backward_isolated
from test_gpu_conv import G, G3
from test_gpu_fused import C, P, chain

pytestmark = pytest.mark.gpu

SHAPES = [
    G(3, 4, 4, 16, 10, 4),                # covers its input: one tap of 256 channels
    G(2, 3, 3, 20, 7, 3),                 # ... channels that are no whole turn of the lanes
    G3(2, 2, 3, 2, 16, 9, 2),             # ... a volume's corner
    G(2, 1, 1, 517, 9, 1),                # a turn more than eight, and five
    G(2, 1, 1, 9, 517, 1),
    G(1, 14, 15, 20, 5, 13, 1, 6),        # thirteen taps an axis
    G(1, 16, 15, 5, 20, 13, 3, 6),        # ... strided
]


@pytest.fixture(scope="module")
def lpm():
    import torch
    assert torch.cuda.is_available()
    import paper_2207_11019_amd as lpm
    return lpm


@pytest.mark.parametrize("g", SHAPES, ids=lambda g: contractions._id(("", g)))
@pytest.mark.parametrize("name", ["bf16", "f32"])
def test_contractions_of_few_outputs(lpm, name, g):
    contractions.test_contractions(lpm, (name, g))


@pytest.mark.parametrize("c", [3, 20], ids=lambda v: str(v))
@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "bf16"])
def test_pooling_of_ragged_channels(lpm, c, dtype):
    layers = chain(C(4, c, 3, 3, 10, 6, p=1, scale=True), P(c, 10, 6), C(c, 8, 5, 3, 5, 3))
    stage_backward_isolated(lpm, layers, [0, 3], 3, 3, dtype, seed=53, dx_wanted=True, check_forward=True, grad_std=1.0)


# lanes of a group: 1 (up to 3 channels), 4 (up to 11), 16 (up to 47), 64; turns: one to nine, 16 and 17, the last one whole and not
@pytest.mark.parametrize("cin", [2, 3, 5, 8, 11, 13, 33, 47, 64, 65, 128, 150, 193, 256, 300, 384, 420, 449, 512, 513, 1024, 1025])
def test_turns_of_one_tap(lpm, cin):
    contractions.test_contractions(lpm, ("f32", G(2, 2, 3, cin, 5, 1)))


# strides up to more than the filter, whose residue classes some taps and some pixels are in none of; a volume's
@pytest.mark.parametrize("g", [G(2, 9, 7, 5, 9, 2, 4), G(1, 11, 12, 3, 20, 5, 5, 2), G(2, 1, 4, 7, 6, 3, 2, 1), G(1, 13, 13, 6, 70, 1, 6),
                               G3(1, 7, 6, 5, 5, 9, 3, 3, 1), G3(2, 1, 4, 3, 6, 7, 3, 2, 1)], ids=lambda g: contractions._id(("", g)))
@pytest.mark.parametrize("name", ["bf16", "f32"])
def test_strides(lpm, name, g):
    contractions.test_contractions(lpm, (name, g))
