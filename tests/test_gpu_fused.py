"""What a stage's backward pass fuses into its contraction kernels, from a forward state prepared by the oracle: pooling backward in
the data gradient, and (see NETS) the epilogues of residual blocks at every tile size, scales applied on the way, weight gradients
beside other streams.  Each network is one or two stages with the gradient of the input wanted."""
import numpy as np
import pytest

from harness import stage_backward_isolated

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lpm():
    import torch
    assert torch.cuda.is_available()
    import paper_2207_11019_amd as lpm
    return lpm


def C(cin, cout, kh, kw, h, w, s=1, p=0, relu=True, bias=True, scale=False, src=None, add=None):
    return dict(kind="conv", cin=cin, cout=cout, kh=kh, kw=kw, stride=s, pad=p, h_in=h, w_in=w, relu=relu, bias=bias, scale=scale,
                src=src, add_src=add, cut_after=True)


def P(c, h, w):
    return dict(kind="maxpool2", cin=c, cout=c, kh=2, kw=2, stride=2, pad=0, h_in=h, w_in=w, relu=False, bias=False, scale=False,
                src=None, add_src=None, cut_after=False)


def chain(*layers):
    for i, l in enumerate(layers):
        if l["src"] is None:
            l["src"] = i - 1
    return list(layers)


# pooling between convolutions whose channel counts are no whole 16-byte chunks, or are
POOLED = [(6, 16, 5, 0), (12, 24, 3, 1), (20, 64, 3, 1), (16, 40, 5, 2)]


@pytest.mark.parametrize("c1,c2,k,p", POOLED, ids=lambda v: str(v))
@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "bf16"])
def test_pooling_backward_before_a_convolution(lpm, c1, c2, k, p, dtype):
    layers = chain(C(4, c1, 3, 3, 16, 16, p=1), P(c1, 16, 16), C(c1, c2, k, k, 8, 8, p=p, scale=True))
    print("channels", c1, c2, "filter", k, "dtype", dtype, flush=True)
    stage_backward_isolated(lpm, layers, [0, 3], 3, 3, dtype, seed=21, dx_wanted=True, check_forward=True, grad_std=1.0)
