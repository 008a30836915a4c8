"""Contractions by filter rows in pieces of 32 or 48 channels (filters three wide whose channels are no whole K tiles): every tile, both
pieces, ragged last pieces, images of one and two pixels a row, volumes, filters of other heights, pooling in front and behind."""
import pytest

import test_gpu_contractions as contractions
from harness import stage_backward_isolated
from test_gpu_conv import G, G3
from test_gpu_fused import C, P, chain

pytestmark = pytest.mark.gpu

SHAPES = [
    G(2, 13, 6, 32, 96, 3, 1, 1),         # 128x32, pieces of 32 channels: one and three of them
    G(1, 11, 12, 160, 224, 3, 1, 1),      # ... five and seven, one row of tiles and a ragged one
    G(2, 9, 9, 48, 144, 3, 1, 1),         # ... pieces of 48
    G(1, 12, 11, 80, 136, 3, 1, 1),       # ... the last one ragged
    G(2, 7, 9, 16, 24, 3, 1, 1),          # ... the only one
    G(1, 8, 17, 56, 104, 3, 1, 1),        # ... ragged pieces of 32
    G(3, 5, 1, 40, 32, 3, 1, 1),          # both outer taps beside the image everywhere
    G(2, 1, 9, 96, 72, 3, 1, 1),          # one image row
    G(2, 7, 2, 32, 160, 3, 1, 1),         # two pixels a row
    G(1, 1, 1, 32, 48, 3, 1, 1),          # one pixel
    G3(2, 3, 5, 6, 32, 48, 3, 1, 1),      # volume
    G3(1, 2, 4, 3, 96, 32, 3, 1, 1),
    dict(G(2, 6, 7, 32, 72, 3, 1, 1), kh=2),
    dict(G(1, 6, 7, 160, 48, 3, 1, 1), kh=5),
    G(2, 9, 11, 32, 48, 5, 1, 2),         # five taps wide: pieces of 32, of 48
    G(2, 9, 11, 48, 80, 5, 1, 2),
    G(1, 12, 13, 104, 72, 5, 1, 2),       # ... ragged
    G(3, 5, 1, 40, 32, 5, 1, 2),          # ... one, two and three pixels a row
    G(3, 5, 2, 32, 40, 5, 1, 2),
    G(2, 4, 3, 16, 24, 5, 1, 2),
    dict(G(2, 7, 8, 96, 32, 5, 1, 2), kh=4),
    G3(1, 4, 5, 6, 24, 32, 5, 1, 2),
    G(2, 100, 98, 32, 104, 5, 1, 2),      # ... 256x64, eight wavefronts
    G(3, 120, 122, 32, 104, 5, 1, 2),     # ... four
    G(3, 113, 114, 48, 96, 5, 1, 2),      # ... 128x96
    G(2, 230, 231, 24, 32, 5, 1, 2),      # ... 256x32
    G(2, 20, 20, 128, 24, 3, 1, 1),       # whole K tiles, half a tile of outputs
    G(1, 9, 9, 352, 416, 3, 1, 1),        # too long for the few tiles: as before
    G(2, 115, 114, 160, 160, 3, 1, 1),    # 256x32
    G(2, 230, 231, 24, 32, 3, 1, 1),      # ... one column
    G(2, 100, 98, 32, 104, 3, 1, 1),      # 256x64, eight wavefronts
    G(2, 100, 98, 104, 40, 3, 1, 1),      # ... of the data gradient
    G(3, 120, 122, 32, 104, 3, 1, 1),     # 256x64, four
    G(3, 120, 122, 104, 32, 3, 1, 1),
    G(3, 113, 114, 32, 96, 3, 1, 1),      # 128x96
    G(3, 113, 114, 96, 88, 3, 1, 1),      # ... ragged N; of the data gradient, pieces of 48
    G(3, 113, 114, 48, 96, 3, 1, 1),      # ... pieces of 48
]


@pytest.fixture(scope="module")
def lpm():
    import torch
    assert torch.cuda.is_available()
    import paper_2207_11019_amd as lpm
    return lpm


@pytest.mark.parametrize("g", SHAPES, ids=lambda g: contractions._id(("bf16", g)) + ("_r%d" % g["kh"] if g["kh"] != g["kw"] else ""))
def test_contractions_by_rows_in_pieces(lpm, g):
    contractions.test_contractions(lpm, ("bf16", g))


def test_pooling_between_rows_in_pieces(lpm):
    """Images of 32, 16 and 8 pixels a row, pooled by the kernels that make them; gradients routed back."""
    layers = chain(C(40, 48, 3, 3, 32, 32, p=1), P(48, 32, 32), C(48, 96, 3, 3, 16, 16, p=1), P(96, 16, 16), C(96, 32, 3, 3, 8, 8, p=1, scale=True))
    stage_backward_isolated(lpm, layers, [0, 5], 2, 2, 1, seed=41, dx_wanted=True, check_forward=True, grad_std=1.0)


# images in a micro-batch, channels: tiles of 256x64 (eight wavefronts, four), 128x96 (pieces of 32 and 48) and 256x32
LARGE = [(20, 32, 104), (43, 32, 104), (38, 32, 96), (38, 48, 96), (101, 24, 32)]


@pytest.mark.parametrize("m,ci,c", LARGE, ids=lambda v: str(v))
def test_pooling_of_32_wide_images_in_pieces(lpm, m, ci, c):
    layers = chain(C(ci, c, 3, 3, 32, 32, p=1), P(c, 32, 32), C(c, 16, 1, 1, 16, 16, scale=True))
    print("m", m, "channels", ci, c, flush=True)
    stage_backward_isolated(lpm, layers, [0, 3], m, m, 1, seed=43, dx_wanted=True, check_forward=True, grad_std=1.0)


@pytest.mark.parametrize("m,ci,c", LARGE, ids=lambda v: str(v))
def test_pooling_backward_of_rows_in_pieces(lpm, m, ci, c):
    layers = chain(C(8, c, 1, 1, 64, 64), P(c, 64, 64), C(c, ci, 3, 3, 32, 32, p=1, scale=True))
    print("m", m, "channels", c, ci, flush=True)
    stage_backward_isolated(lpm, layers, [0, 3], m, m, 1, seed=47, dx_wanted=True, check_forward=True, grad_std=1.0)


# residue classes of images of fewer pixels than strides, of whole strides and one more, of a volume's slices
@pytest.mark.parametrize("g", [G(2, 1, 3, 32, 64, 3, 2, 1), G(1, 3, 2, 32, 40, 5, 4, 2), G(2, 9, 10, 64, 32, 3, 3, 1), G(1, 8, 13, 40, 24, 7, 4, 3),
                               G3(1, 1, 2, 3, 32, 64, 3, 2, 1), G3(2, 4, 5, 2, 32, 24, 3, 2, 1)], ids=lambda g: contractions._id(("", g)))
@pytest.mark.parametrize("name", ["bf16", "f32"])
def test_strided_data_gradients_of_small_images(lpm, name, g):
    contractions.test_contractions(lpm, (name, g))


def as_in_a_stage(lpm, g, seed):
    """One layer as a stage of its own and alone on the same operands, which are of many magnitudes, so that another order of sums shows:
    (geometry, x, weights, transposed, dz, scratch), the stage's y and dx."""
    import torch
    gen = torch.Generator().manual_seed(seed)
    layer = chain(C(g["cin"], g["cout"], g["kh"], g["kw"], g["h"], g["w"], p=g["pad"], relu=False, bias=False))
    if g.get("d", 1) > 1:
        layer[0].update(d_in=g["d"], kd=g["kd"], pad_d=g["pad_d"])
    st = lpm.Stage(layer, 0, 1, g["m"], lpm.BF16)
    buf = lambda n: torch.zeros(max(n, 256), dtype=torch.uint8, device="cuda")
    rnd = lambda n: (torch.randn(n, generator=gen) * 2.0 ** torch.randint(-7, 8, (n,), generator=gen)).to(torch.bfloat16).cuda()
    params, lowp, grads, stash, fws, bws = [buf(n) for n in (st.param_bytes, st.lowp_bytes, st.grad_bytes, st.stash_bytes, st.fwd_ws_bytes, st.bwd_ws_bytes)]
    w = rnd(g["cout"] * g.get("kd", 1) * g["kh"] * g["kw"] * g["cin"])
    params.view(torch.float32)[:w.numel()].copy_(w.float())
    st.sync_lowp(params, lowp)
    x, dz = rnd(st.in_bytes // 2), rnd(st.out_bytes // 2)
    y, dx = torch.empty_like(dz), torch.empty_like(x)
    st.forward(x, y, None, None, params, lowp, stash, fws, 1.0)
    st.backward(x, y, dz, dx, params, lowp, stash, grads, False, bws)
    wt = w.view(g["cout"], -1, g["cin"]).permute(2, 1, 0).contiguous().view(-1)
    return (x, w, wt, dz, buf(max(lpm.lpm_conv_ws_bytes(g, lpm.BF16)))), y, dx


# ragged channels, both ways; half a tile of outputs; shared reductions; a volume
TIMED = [G(2, 9, 9, 160, 96, 3, 1, 1), G(1, 13, 12, 96, 200, 3, 1, 1), G(1, 12, 12, 128, 24, 3, 1, 1), G(1, 16, 31, 96, 232, 3, 1, 1),
         G(1, 9, 10, 104, 72, 5, 1, 2), G(2, 9, 9, 48, 32, 3, 1, 1)]


@pytest.mark.parametrize("g", TIMED, ids=lambda g: contractions._id(("", g)))
def test_timed_contractions_are_those_of_a_stage(lpm, g):
    """lpm_conv_time measures what a stage of the same layer runs: the same bits."""
    import torch
    (x, w, wt, dz, ws), y, dx = as_in_a_stage(lpm, g, 61)
    ty, tx = torch.empty_like(y), torch.empty_like(dx)
    lpm.lpm_conv_time(0, g, lpm.BF16, x, w, wt, ty, torch.zeros(w.numel(), device="cuda"), ws, warmup=0, iters=1)
    lpm.lpm_conv_time(1, g, lpm.BF16, tx, w, wt, dz, torch.zeros(w.numel(), device="cuda"), ws, warmup=0, iters=1)
    torch.cuda.synchronize()
    assert torch.equal(ty, y.clamp(min=0)) and torch.equal(tx, dx)


# reductions shared by blocks, by the wavefronts of 32x32 and of 32x64 tiles; data gradients of them
SHARED = [G(2, 8, 8, 200, 232, 3, 1, 1), G(2, 8, 8, 96, 160, 5, 1, 2), G(1, 16, 31, 96, 232, 3, 1, 1), G(1, 16, 31, 200, 232, 3, 1, 1), G(1, 10, 101, 200, 264, 3, 1, 1),
          G(1, 10, 101, 264, 200, 3, 1, 1)]


@pytest.mark.parametrize("g", SHARED, ids=lambda g: contractions._id(("", g)))
def test_shared_reductions_keep_their_short_sums(lpm, g):
    """A call of its own whose reduction blocks or wavefronts share adds it up as a stage does.  (In one walk through all of K a tenth more of the results
    were not the rounded exact ones.)"""
    import torch
    (x, w, wt, dz, ws), y, dx = as_in_a_stage(lpm, g, 67)
    ly, lx = torch.empty_like(y), torch.empty_like(dx)
    lpm.lpm_conv_forward(g, lpm.BF16, x, w, None, None, None, False, ly, ws)
    lpm.lpm_conv_dgrad(g, lpm.BF16, dz, w, wt, lx, False, ws)
    torch.cuda.synchronize()
    assert torch.equal(ly, y) and torch.equal(lx, dx)


# several pieces of a tap's channels, whole and ragged, where one block has all of K
@pytest.mark.parametrize("g", [G(3, 19, 150, 104, 136, 5, 1, 2), G(3, 17, 90, 224, 160, 3, 1, 1), dict(G(3, 18, 90, 160, 176, 3, 1, 1), kh=5), G(3, 16, 90, 80, 224, 3, 1, 1)],
                         ids=lambda g: contractions._id(("bf16", g)))
def test_pieces_of_long_reductions(lpm, g):
    contractions.test_contractions(lpm, ("bf16", g))


# ---- five taps: pooling in front and behind, as above
def test_pooling_between_five_taps(lpm):
    layers = chain(C(32, 48, 5, 5, 32, 32, p=2), P(48, 32, 32), C(48, 32, 5, 5, 16, 16, p=2), P(32, 16, 16), C(32, 16, 5, 5, 8, 8, p=2, scale=True))
    stage_backward_isolated(lpm, layers, [0, 5], 2, 2, 1, seed=71, dx_wanted=True, check_forward=True, grad_std=1.0)


@pytest.mark.parametrize("m,ci,c", LARGE, ids=lambda v: str(v))
def test_five_taps_of_32_wide_images_pooled(lpm, m, ci, c):
    ci = max(ci, 32) if c != 32 else 16        # (a layer of a stage: 16, 32 or 48 channels)
    layers = chain(C(ci, c, 5, 5, 32, 32, p=2), P(c, 32, 32), C(c, 16, 1, 1, 16, 16, scale=True))
    print("m", m, "channels", ci, c, flush=True)
    stage_backward_isolated(lpm, layers, [0, 3], m, m, 1, seed=73, dx_wanted=False, check_forward=True, grad_std=1.0)


@pytest.mark.parametrize("m,ci,c", LARGE, ids=lambda v: str(v))
def test_pooling_backward_of_five_taps(lpm, m, ci, c):
    ci = max(ci, 32) if c != 32 else 16
    layers = chain(C(8, c, 1, 1, 64, 64), P(c, 64, 64), C(c, ci, 5, 5, 32, 32, p=2, scale=True))
    print("m", m, "channels", c, ci, flush=True)
    stage_backward_isolated(lpm, layers, [0, 3], m, m, 1, seed=79, dx_wanted=True, check_forward=True, grad_std=1.0)


def test_pooling_of_32_wide_images_on_256x32(lpm):
    """Three taps, 16 channels: the only tiles of LARGE that its 24 channels, in chunks across taps in a stage, do not reach."""
    layers = chain(C(16, 32, 3, 3, 32, 32, p=1), P(32, 32, 32), C(32, 16, 1, 1, 16, 16, scale=True))
    stage_backward_isolated(lpm, layers, [0, 3], 101, 101, 1, seed=83, dx_wanted=False, check_forward=True, grad_std=1.0)
    layers = chain(C(8, 32, 1, 1, 64, 64), P(32, 64, 64), C(32, 16, 3, 3, 32, 32, p=1, scale=True))
    stage_backward_isolated(lpm, layers, [0, 3], 101, 101, 1, seed=89, dx_wanted=True, check_forward=True, grad_std=1.0)
