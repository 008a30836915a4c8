"""The contraction kernels at the edges of their tiles and dispatch rules, through the C ABI, against PyTorch's convolutions
in double precision on the CPU: every tile variant, channel counts that are whole 16-byte chunks but no whole K tiles, channel
counts that are not (gathered operands), strides, volumes, split reductions called twice on the same scratch."""
import numpy as np
import pytest

from test_gpu_conv import G, G3
from harness import rel_err

pytestmark = pytest.mark.gpu

BOTH = [
    G(2, 9, 7, 24, 40, 3, 1, 1),          # no whole K tile per tap; ragged M and N
    G(1, 10, 9, 40, 72, 5, 2, 2),         # stride 2, every residue class, N over one tile
    G(1, 11, 11, 8, 16, 3, 3, 1),         # stride 3: one chunk per tap (float: two)
    G(3, 4, 4, 64, 72, 4, 1, 0),          # the filter covers its input: seen as 1x1
    G(2, 4, 4, 512, 64, 3, 1, 1),         # split reduction, one row tile
    G3(1, 4, 5, 6, 16, 24, 3, 1, 1),      # volume
    G3(1, 5, 5, 4, 16, 32, 3, 2, 1),      # volume, stride 2
    G(2, 17, 15, 3, 64, 3, 1, 1),         # gathered: two channel tiles
    G(1, 95, 97, 3, 65, 3, 2, 1),         # gathered: a channel past two tiles, stride 2
    G(2, 70, 70, 6, 16, 5, 1, 0),         # gathered: more than one block's row tiles, five K steps and more
    G(2, 14, 14, 6, 16, 5, 1, 0),         # gathered: the reduction shared by a block's wavefronts
    G(1, 33, 31, 3, 33, 7, 2, 3),         # gathered: 147 terms
    G3(1, 9, 8, 7, 1, 32, 3, 1, 1),       # gathered: a volume of one channel
    G(2, 8, 8, 5, 7, 3, 1, 1),            # fewer than 256 rows
    G(3, 1, 1, 84, 10, 1, 1, 0),          # head
]
BF16 = [
    G(1, 152, 152, 8, 128, 1, 1, 0),      # 181 tiles of 128x128: three stages
    G(3, 128, 128, 8, 128, 1, 1, 0),      # 384 of them: two
    G(2, 107, 109, 32, 200, 3, 1, 1),     # ragged M and N, by filter rows in pieces (the 366 tiles of 128x128: STAGE)
    G(2, 107, 109, 200, 32, 3, 1, 1),     # ... of the data gradient
    G(2, 107, 109, 256, 256, 1, 1, 0),    # ... of both, whole K tiles
    G(2, 151, 153, 256, 64, 3, 2, 1),     # 730 of a strided data gradient
    G(2, 107, 109, 88, 200, 3, 1, 1),     # the same with a dozen K tiles (184 tiles of 256x128 in chunks across taps: STAGE)
    G(2, 107, 109, 200, 88, 3, 1, 1),
    G(2, 107, 109, 768, 256, 1, 1, 0),    # ... whole K tiles, the fewest
    G(2, 107, 109, 256, 768, 1, 1, 0),
    G(2, 151, 153, 256, 192, 3, 2, 1),    # ... strided
    G(3, 128, 128, 8, 64, 3, 1, 1),       # 384 tiles of 128x64
    G(3, 127, 128, 64, 72, 1, 1, 0),      # N over half a tile, ragged M
    G(1, 128, 128, 128, 8, 1, 1, 0),      # the same sizes for the data gradient
    G(3, 128, 128, 128, 8, 1, 1, 0),
    G(3, 128, 128, 256, 256, 1, 1, 0),    # 128x128 weight-gradient tiles
    G(1, 20, 15, 64, 64, 3, 1, 1),        # filter rows over segments of 8 pixels, the last one 7 wide
    G(1, 20, 13, 72, 40, 3, 1, 1),        # ... 5 wide: single taps
    G3(1, 3, 6, 8, 64, 64, 3, 1, 1),      # ... volume
    G(3, 5, 1, 64, 40, 3, 1, 1),          # contractions by filter rows: both outer taps beside the image everywhere
    G(2, 1, 9, 128, 72, 3, 1, 1),         # ... one image row, two K tiles a tap
    G(2, 7, 2, 64, 128, 3, 1, 1),         # ... two pixels a row
    G(1, 6, 7, 512, 512, 3, 1, 1),        # ... a reduction whose parts begin in the middle of a filter row's channels
    G3(2, 3, 5, 6, 128, 64, 3, 1, 1),     # ... volume
    dict(G(2, 6, 7, 64, 72, 3, 1, 1), kh=2),                # ... filters of two and of five rows: images a row taller, or two shorter
    dict(G(1, 6, 7, 128, 64, 3, 1, 1), kh=5),
    G(1, 147, 148, 64, 64, 3, 1, 1),      # ... 340 tiles of 64x64: three stages
    G(3, 127, 128, 64, 64, 3, 1, 1),      # ... 128x64
    G(2, 107, 109, 64, 200, 3, 1, 1),     # ... 128x128, three stages: forward
    G(2, 107, 109, 200, 64, 3, 1, 1),     # ... and data gradient
    G(3, 128, 128, 64, 128, 3, 1, 1),     # (two stages: tap by tap)
    G(2, 38, 41, 256, 256, 3, 1, 1),      # ... 64x64, four K tiles a tap, unsplit
    G(1, 16, 31, 192, 232, 3, 1, 1),      # a block's wavefronts share the reduction: tiles of 32x32, forward, data gradient,
    G(1, 16, 31, 232, 192, 3, 1, 1),
    G(1, 16, 31, 200, 232, 3, 1, 1),      # ... chunks across taps
    G(1, 16, 31, 1600, 232, 1, 1, 0),     # ... one tap
    G(1, 16, 31, 96, 232, 3, 1, 1),       # ... that would not be split either
    G(1, 32, 62, 192, 232, 3, 2, 1),      # ... stride 2
    G(1, 10, 101, 192, 264, 3, 1, 1),     # ... of 32x64
    G(1, 10, 101, 264, 192, 3, 1, 1),
    G(1, 10, 101, 200, 264, 3, 1, 1),
    G(1, 10, 101, 264, 200, 3, 1, 1),
    G(2, 80, 80, 64, 64, 5, 1, 2),        # single taps, ranges of 20 K tiles: the pixel records in several rounds
    G(5, 64, 64, 256, 256, 3, 1, 1),      # filter rows, ranges of 64 K tiles: records in several rounds, four stages
]
F32 = [                                   # data gradients of one, three and (strided, by residue class) one to four K tiles
    G(1, 16, 31, 64, 232, 3, 1, 1),       # a block's wavefronts share the reduction: tiles of 32x32
    G(1, 16, 31, 232, 64, 3, 1, 1),
    G(1, 16, 31, 36, 232, 5, 1, 2),
    G(1, 16, 31, 232, 36, 5, 1, 2),
    G(1, 10, 101, 64, 264, 3, 1, 1),      # ... of 32x64
    G(1, 10, 101, 264, 64, 3, 1, 1),
    G(1, 10, 101, 36, 264, 5, 1, 2),
    G(2, 105, 107, 40, 32, 1, 1, 0),      # more blocks than the card has CUs: three stages
    G(2, 105, 107, 36, 96, 1, 1, 0),
    G(2, 105, 107, 64, 32, 3, 2, 1),
    G(2, 40, 41, 40, 32, 1, 1, 0),        # fewer: four
    G(2, 20, 21, 36, 96, 1, 1, 0),
    G(2, 20, 21, 64, 32, 3, 2, 1),
]


@pytest.fixture(scope="module")
def lpm():
    import torch
    assert torch.cuda.is_available()
    import paper_2207_11019_amd as lpm
    return lpm


def _id(c):
    g = c[1]
    return "%s_m%d_%s%dx%d_%d_%d_k%d_s%d" % (c[0], g["m"], "d%d_" % g["d"] if "d" in g else "", g["h"], g["w"], g["cin"], g["cout"], g["kh"], g["stride"])


@pytest.mark.parametrize("case", [(t, g) for g in BOTH for t in ("bf16", "f32")] + [("bf16", g) for g in BF16] + [("f32", g) for g in F32], ids=_id)
def test_contractions(lpm, case):
    import torch
    import torch.nn.grad as tg
    name, g = case
    print("geometry", name, g, flush=True)
    bf = name == "bf16"
    dt, td = (lpm.BF16, torch.bfloat16) if bf else (lpm.F32, torch.float32)
    gen = torch.Generator().manual_seed(7)
    D, KD, s = g.get("d", 1), g.get("kd", 1), g["stride"]
    pad = (g.get("pad_d", 0), g["pad"], g["pad"])
    st = (s if D > 1 else 1, s, s)
    # channels last as the kernels take them; double precision, [N][C][D][H][W], for the reference
    x = torch.randn(g["m"], D, g["h"], g["w"], g["cin"], generator=gen).to(td)
    w = (torch.randn(g["cout"], KD, g["kh"], g["kw"], g["cin"], generator=gen) / (g["cin"] * KD * g["kh"] * g["kw"]) ** 0.5).to(td)
    nchw = lambda t: t.double().permute(0, 4, 1, 2, 3).contiguous()
    nhwc = lambda t: t.permute(0, 2, 3, 4, 1).contiguous()
    xr, wr = nchw(x), nchw(w)
    z = torch.nn.functional.conv3d(xr, wr, stride=st, padding=pad)
    dz = torch.randn(nhwc(z).shape, generator=gen).to(td)
    add = torch.randn(dz.shape, generator=gen).to(td)
    sc, bi = torch.rand(g["cout"], generator=gen) + 0.5, torch.randn(g["cout"], generator=gen)
    dx_ref = nhwc(tg.conv3d_input(xr.shape, wr, nchw(dz), stride=st, padding=pad))
    dw_ref = nhwc(tg.conv3d_weight(xr, wr.shape, nchw(dz), stride=st, padding=pad))

    dev = lambda t: t.reshape(-1).cuda()
    xd, wd, dzd, addd, scd, bid = dev(x), dev(w), dev(dz), dev(add), dev(sc), dev(bi)
    wt = dev(w.permute(4, 1, 2, 3, 0).contiguous()) if bf else None
    ws = torch.full((max(max(lpm.lpm_conv_ws_bytes(g, dt)), 256),), 0x55, dtype=torch.uint8, device="cuda")
    err = lambda got, ref: rel_err(got.float().cpu().numpy().astype(np.float64), ref.reshape(-1).numpy())
    tol = 2e-2 if bf else 2e-5

    y = [torch.empty(dz.numel(), dtype=td, device="cuda") for _ in range(2)]
    for k in range(2):                    # the second call meets the first one's scratch
        lpm.lpm_conv_forward(g, dt, xd, wd, scd, bid, addd, True, y[k], ws)
    dx = [torch.full((x.numel(),), 0.5, dtype=td, device="cuda") for _ in range(2)]
    for k in range(2):
        lpm.lpm_conv_dgrad(g, dt, dzd, wd, wt, dx[k], k == 1, ws)
    dw = [torch.full((w.numel(),), 0.5, dtype=torch.float32, device="cuda") for _ in range(2)]
    for k in range(2):
        lpm.lpm_conv_wgrad(g, dt, xd, dzd, dw[k], k == 1, ws)
    torch.cuda.synchronize()
    assert err(y[0], (nhwc(z) * sc + bi + add.double()).clamp(min=0)) <= tol
    assert torch.equal(y[0], y[1])
    assert err(dx[0], dx_ref) <= tol and err(dx[1], dx_ref + 0.5) <= tol
    assert err(dw[0], dw_ref) <= (1e-3 if bf else 2e-5) and err(dw[1], dw_ref + 0.5) <= (1e-3 if bf else 2e-5)


# In the order of sums that a stage keeps, which lone calls of these need not: chunks across the taps of a filter, whose channels are no whole K tiles
STAGE = [
    G(2, 107, 109, 40, 200, 3, 1, 1),     # 128x128, three stages: forward, data gradient
    G(2, 107, 109, 200, 40, 3, 1, 1),
    G(3, 128, 128, 40, 128, 3, 1, 1),     # ... two
    G(2, 107, 109, 88, 200, 3, 1, 1),     # 256x128
    G(2, 107, 109, 200, 88, 3, 1, 1),
    G(3, 127, 128, 40, 72, 3, 1, 1),      # 128x64: of the data gradient
    G(1, 16, 31, 200, 232, 3, 1, 1),      # a block's wavefronts share the reduction: tiles of 32x32
    G(1, 16, 31, 96, 232, 3, 1, 1),       # ... that would not be split either
    G(1, 10, 101, 200, 264, 3, 1, 1),     # ... of 32x64
    G(1, 10, 101, 264, 200, 3, 1, 1),
    G(1, 16, 31, 40, 24, 5, 1, 2),        # 64x64, 5x5
    G(1, 12, 11, 224, 160, 3, 1, 1),      # ... in parts
]


@pytest.mark.parametrize("g", STAGE, ids=lambda g: _id(("bf16", g)))
def test_contractions_in_a_stages_order(lpm, g):
    """The bf16 forward pass and data gradient that lpm_conv_time runs, against double precision."""
    import torch
    import torch.nn.grad as tg
    print("geometry", g, flush=True)
    gen = torch.Generator().manual_seed(7)
    x = torch.randn(g["m"], g["h"], g["w"], g["cin"], generator=gen).to(torch.bfloat16)
    w = (torch.randn(g["cout"], g["kh"], g["kw"], g["cin"], generator=gen) / (g["cin"] * g["kh"] * g["kw"]) ** 0.5).to(torch.bfloat16)
    nchw = lambda t: t.double().permute(0, 3, 1, 2).contiguous()
    nhwc = lambda t: t.permute(0, 2, 3, 1).contiguous()
    z = torch.nn.functional.conv2d(nchw(x), nchw(w), padding=g["pad"])
    dz = torch.randn(nhwc(z).shape, generator=gen).to(torch.bfloat16)
    dx_ref = nhwc(tg.conv2d_input(nchw(x).shape, nchw(w), nchw(dz), padding=g["pad"]))
    dev = lambda t: t.reshape(-1).cuda()
    xd, wd, dzd, wt = dev(x), dev(w), dev(dz), dev(w.permute(3, 1, 2, 0).contiguous())
    ws = torch.full((max(max(lpm.lpm_conv_ws_bytes(g, lpm.BF16)), 256),), 0x55, dtype=torch.uint8, device="cuda")
    y, dx, dw = torch.empty_like(dzd), torch.empty_like(xd), torch.zeros(w.numel(), device="cuda")
    err = lambda got, ref: rel_err(got.float().cpu().numpy().astype(np.float64), ref.reshape(-1).numpy())
    lpm.lpm_conv_time(0, g, lpm.BF16, xd, wd, wt, y, dw, ws, warmup=0, iters=1)
    lpm.lpm_conv_time(1, g, lpm.BF16, dx, wd, wt, dzd, dw, ws, warmup=0, iters=1)
    torch.cuda.synchronize()
    assert err(y, nhwc(z).clamp(min=0)) <= 2e-2 and err(dx, dx_ref) <= 2e-2


@pytest.mark.parametrize("m,h,w,C", [(2, 1, 1, 8), (1, 3, 11, 24), (2, 8, 8, 40), (1, 5, 4, 264), (3, 4, 4, 96), (1, 23, 23, 128), (1, 31, 31, 32)],
                         ids=lambda v: str(v))
def test_attention_bf16(lpm, m, h, w, C):
    """One attention layer as a stage of its own: one position, positions and channels that fill no tile, more channel groups
    than wavefronts, several row blocks, the longest rows."""
    import torch
    from oracle import lpm_oracle as orc
    layers = [dict(kind="attn", cin=3 * C, cout=C, kh=1, kw=1, stride=1, pad=0, h_in=h, w_in=w, relu=False, bias=False, scale=False,
                   src=-1, add_src=None, cut_after=False)]
    gen = np.random.default_rng(5)
    bf = lambda a: torch.from_numpy(a).to(torch.bfloat16).double().numpy()
    x, dy = bf(gen.standard_normal((m, 3 * C, h, w))), bf(gen.standard_normal((m, C, h, w)))
    net = lpm.Net(layers, [0, 1], m, 1, lpm.BF16, dx_wanted=True)
    net.step(lpm.pack_act(x, lpm.BF16), None, lpm.pack_act(dy, lpm.BF16), 0.0, 0.0, lpm.LOCKED)
    torch.cuda.synchronize()
    y = net.read_act_out(0, 0)
    assert rel_err(y, orc.attn_fwd(x)) <= 6e-3                     # (one rounding to bf16 of the result)
    assert rel_err(net.read_grad_in(0, 0), orc.attn_bwd(x, dy)) <= 6e-3
