"""What a stage's backward pass fuses into its contraction kernels, from a forward state prepared by the oracle: pooling backward in
the data gradient, and (see NETS) the epilogues of residual blocks at every tile size, scales applied on the way, weight gradients
beside other streams.  Each network is one or two stages with the gradient of the input wanted."""
import numpy as np
import pytest

from harness import compare, gpu_step, oracle_step, stage_backward_isolated

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


# ... on the larger tiles of the data gradient: 128x64, 128x128, 256x128 (pooled images and channels of the middle tensor)
@pytest.mark.parametrize("m,c,h", [(45, 40, 22), (23, 128, 32), (90, 200, 16)], ids=["tile128x64", "tile128", "tile256"])
def test_pooling_backward_on_larger_tiles(lpm, m, c, h):
    layers = chain(C(8, c, 1, 1, 2 * h, 2 * h), P(c, 2 * h, 2 * h), C(c, 768, 1, 1, h, h, scale=True))
    print("m", m, "channels", c, "height", h, flush=True)
    stage_backward_isolated(lpm, layers, [0, 3], m, m, 1, seed=31, dx_wanted=True, check_forward=True, grad_std=1.0)


# pooling behind and in front of a contraction on 32-row tiles, whose wavefronts share the reduction
@pytest.mark.parametrize("m,layers", [(4, (C(192, 128, 3, 3, 16, 16, p=1, scale=True), P(128, 16, 16), C(128, 16, 1, 1, 8, 8))),
                                      (2, (C(8, 256, 1, 1, 32, 32), P(256, 32, 32), C(256, 192, 3, 3, 16, 16, p=1, scale=True)))], ids=["forward", "backward"])
def test_pooling_on_tiles_of_32_rows(lpm, m, layers):
    layers = chain(*[dict(l) for l in layers])
    print("m", m, "layers", [(l["cin"], l["cout"]) for l in layers], flush=True)
    stage_backward_isolated(lpm, layers, [0, 3], m, m, 1, seed=33, dx_wanted=True, check_forward=True, grad_std=1.0)


# forward pooling of images 32 wide, whose windows span two pieces of a tile: on every tile, split, in ragged channels, one row of windows
@pytest.mark.parametrize("m,cin,c,h", [(2, 16, 24, 32), (1, 256, 64, 32), (3, 64, 72, 2), (24, 16, 64, 32), (24, 16, 128, 32), (24, 32, 256, 32), (24, 96, 256, 32)],
                         ids=["ragged", "split", "one_row", "tile128x64", "tile128", "large", "tile256"])
def test_pooling_forward_of_rows_of_32(lpm, m, cin, c, h):
    layers = chain(C(cin, c, 3, 3, h, 32, p=1, scale=True), P(c, h, 32), C(c, 16, 1, 1, h // 2, 16))
    print("m", m, "channels", cin, c, "height", h, flush=True)
    stage_backward_isolated(lpm, layers, [0, 3], m, m, 1, seed=27, dx_wanted=True, check_forward=True, grad_std=1.0)


# ... and of the kernel that gathers element by element, whose tiles go by pooling window: few and many rows, channels in chunks and ragged,
# more than one tile of them, a tile that ends inside an image
@pytest.mark.parametrize("m,cin,c,k,p,h,w,dtype", [(8, 1, 6, 5, 0, 28, 28, 0), (3, 6, 16, 5, 0, 22, 16, 0), (12, 3, 20, 3, 1, 28, 30, 0), (3, 6, 40, 3, 1, 10, 14, 0),
                                                   (5, 3, 16, 3, 1, 18, 22, 1), (12, 3, 70, 3, 1, 28, 30, 1), (3, 6, 12, 5, 2, 10, 14, 1)],
                         ids=["lenet", "f32_chunks", "f32_many", "f32_two_tiles", "bf16_chunks", "bf16_many", "bf16_split"])
def test_pooling_forward_of_gathered_layers(lpm, m, cin, c, k, p, h, w, dtype):
    ho, wo = h + 2 * p - k + 1, w + 2 * p - k + 1
    layers = chain(C(cin, c, k, k, h, w, p=p, scale=True), dict(P(c, ho, ho), h_in=ho, w_in=wo), C(c, 16, 1, 1, ho // 2, wo // 2))
    print("m", m, "channels", cin, c, "dtype", dtype, flush=True)
    stage_backward_isolated(lpm, layers, [0, 3], m, m, dtype, seed=29, dx_wanted=False, check_forward=True, grad_std=1.0)


# average pooling and the layer over its channels in one kernel: channels that fill no block and several, one output and the most, positions that
# are no multiple of the threads' share; a layer of more outputs, which has kernels of its own; samples or weights that leave only the forward pass or
# only the data gradient in one
@pytest.mark.parametrize("m,c,n,h,w", [(3, 24, 10, 3, 5), (2, 512, 100, 4, 4), (2, 1032, 1, 2, 3), (1, 64, 128, 1, 1), (2, 64, 136, 4, 4), (257, 1024, 1, 1, 1),
                                       (2, 1032, 33, 2, 2)], ids=lambda v: str(v))
@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "bf16"])
def test_head(lpm, m, c, n, h, w, dtype):
    gap = dict(kind="gap", cin=c, cout=c, kh=h, kw=w, stride=1, pad=0, h_in=h, w_in=w, relu=False, bias=False, scale=False, src=None, add_src=None, cut_after=False)
    layers = chain(C(8, c, 1, 1, h, w, scale=True), gap, C(c, n, 1, 1, 1, 1, relu=False))
    print("m", m, "channels", c, "outputs", n, "image", h, w, "dtype", dtype, flush=True)
    stage_backward_isolated(lpm, layers, [0, 3], m, m, dtype, seed=35, dx_wanted=True, check_forward=True, grad_std=1.0)


# ... whose layer has no bias; with another reader of the pooling's input, whose gradient is there first; at the head of a stage, where it applies the
# ReLU mask of the stage before, alone and to the sum with that reader's
@pytest.mark.parametrize("starts", [(0, 1), (0,)], ids=["cut", "inside"])
@pytest.mark.parametrize("beside", [True, False], ids=["reader", "alone"])
@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "bf16"])
def test_head_adds_and_masks(lpm, dtype, beside, starts):
    m, c, n, h = 8, 24, 16, 4
    gap = dict(kind="gap", cin=c, cout=c, kh=h, kw=h, stride=1, pad=0, h_in=h, w_in=h, relu=False, bias=False, scale=False, src=None, add_src=None, cut_after=False)
    layers = [C(8, c, 1, 1, h, h), gap, C(c, n, 1, 1, 1, 1, relu=False, bias=False)]
    layers = chain(*layers, *([C(c, n, h, h, h, h, relu=False, src=0, add=2)] if beside else []))
    starts = list(starts) + [len(layers)]
    print("dtype", dtype, "layers", len(layers), "starts", starts, flush=True)
    if len(starts) == 2:
        stage_backward_isolated(lpm, layers, starts, m, m, dtype, seed=39, dx_wanted=True, check_forward=True, grad_std=1.0)
        return
    o = oracle_step(layers, starts, 2 * m, 2, dtype == 1, seed=39, lr=0.05, mu=0.9)
    for mode in (lpm.LOCKED, lpm.OVERLAPPED):
        net = gpu_step(lpm, layers, starts, 2 * m, 2, dtype, o, 0.05, 0.9, mode)
        compare(net, layers, starts, 2, dtype, o)


# ... and the gradient of the pooled tensor is there to be read, as that of any tensor inside a stage, also where the gradient of the
# pooling's input is not wanted.  A stored value is within half a unit of its last place of the sum, whose float error is below (n + 1) 2^-24 of the
# sum of magnitudes.
@pytest.mark.parametrize("dx_wanted", [True, False], ids=["dx", "no_dx"])
@pytest.mark.parametrize("m,c,n,h,w", [(3, 24, 10, 3, 5), (2, 1032, 1, 2, 3)], ids=lambda v: str(v))
@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "bf16"])
def test_gradient_of_the_pooled_tensor(lpm, m, c, n, h, w, dtype, dx_wanted):
    import torch
    gap = dict(kind="gap", cin=c, cout=c, kh=h, kw=w, stride=1, pad=0, h_in=h, w_in=w, relu=False, bias=False, scale=False, src=None, add_src=None, cut_after=False)
    st = lpm.Stage(chain(gap, C(c, n, 1, 1, 1, 1, relu=False)), 0, 2, m, dtype)
    print("m", m, "channels", c, "outputs", n, "dtype", dtype, flush=True)
    tdt, rng = (torch.bfloat16 if dtype else torch.float32), np.random.default_rng(37)
    buf = lambda k: torch.zeros(max(k, 256), dtype=torch.uint8, device="cuda")      # noqa: E731
    rnd = lambda k, s: torch.from_numpy(rng.normal(0, s, k).astype(np.float32)).to(tdt)      # noqa: E731
    params, lowp, grads, stash, fws, bws = [buf(k) for k in (st.param_bytes, st.lowp_bytes, st.grad_bytes, st.stash_bytes, st.fwd_ws_bytes, st.bwd_ws_bytes)]
    wt, dy, (off, _) = rnd(n * c, 0.1), rnd(m * n, 1.0), st.param_offset(1, 0)
    params.view(torch.float32)[off:off + n * c] = wt.float().cuda()
    lowp = lowp if dtype else None
    st.sync_lowp(params, lowp)
    x, y, dx = rnd(m * h * w * c, 1.0).cuda(), buf(st.out_bytes), buf(st.in_bytes)
    st.forward(x, y, None, None, params, lowp, stash, fws, 1.0)
    bws.fill_(0x7f)
    st.backward(x, y, dy.cuda(), dx if dx_wanted else None, params, lowp, stash, grads, False, bws)
    torch.cuda.synchronize()
    at, size = st.grad_offset(0)
    got = bws[at:at + size].view(tdt)[:m * c].double().cpu().numpy().reshape(m, c)
    a, b = dy.double().numpy().reshape(m, n), wt.double().numpy().reshape(n, c)
    sums = (n + 1) * 2.0 ** -24 * (np.abs(a) @ np.abs(b))
    assert (np.abs(got - a @ b) <= sums + 2.0 ** (-8 if dtype else -24) * (np.abs(a @ b) + sums)).all()
    if dx_wanted:
        d = dx.view(tdt)[:m * h * w * c].double().cpu().numpy().reshape(m, h * w, c)
        want = got[:, None, :] / (h * w)
        assert (np.abs(d - want) <= 2.0 ** (-8 if dtype else -23) * np.abs(want)).all()


# ... and float sums are no further from the exact ones than those of the layer's own kernels: forward 64 running sums of c / 64 products, folded in
# pairs, back 16 of n / 16, added in 64 bits.  A rounding is off by at most 2^-24 / sqrt(3) of its value (rms); a running sum of k terms of either sign gathers k / 2
# of them, relative to the squared result, and so do all running sums together; a level of folding and the rounding to float one each.
@pytest.mark.parametrize("c,n", [(1024, 32), (1000, 48), (512, 128)], ids=lambda v: str(v))
def test_float_sums_of_the_head(lpm, c, n):
    import torch
    m = 16
    gap = dict(kind="gap", cin=c, cout=c, kh=1, kw=1, stride=1, pad=0, h_in=1, w_in=1, relu=False, bias=False, scale=False, src=None, add_src=None, cut_after=False)
    st = lpm.Stage(chain(gap, C(c, n, 1, 1, 1, 1, relu=False, bias=False)), 0, 2, m, 0)
    print("channels", c, "outputs", n, flush=True)
    rng = np.random.default_rng(41)
    buf = lambda k: torch.zeros(max(k, 256), dtype=torch.uint8, device="cuda")      # noqa: E731
    rnd = lambda *k: rng.normal(0, 1, k).astype(np.float32)      # noqa: E731
    params, grads, stash, fws, bws, y, dx = [buf(k) for k in (st.param_bytes, st.grad_bytes, st.stash_bytes, st.fwd_ws_bytes, st.bwd_ws_bytes, st.out_bytes, st.in_bytes)]
    x, w, dy = rnd(m, c), rnd(n, c), rnd(m, n)
    off, _ = st.param_offset(1, 0)
    params.view(torch.float32)[off:off + n * c] = torch.from_numpy(w).cuda().view(-1)
    xd = torch.from_numpy(x).cuda()
    st.forward(xd, y, None, None, params, None, stash, fws, 1.0)
    st.backward(xd, y, torch.from_numpy(dy).cuda(), dx, params, None, stash, grads, False, bws)
    torch.cuda.synchronize()
    for got, a, b, bound in ((y, x, w.T, c / 128 + 7), (dx, dy, w, n / 32 + 1)):
        want = a.astype(np.float64) @ b.astype(np.float64)
        got = got.view(torch.float32)[:want.size].double().cpu().numpy().reshape(want.shape)
        assert np.linalg.norm(got - want) <= 2.0 ** -24 / 3 ** 0.5 * bound ** 0.5 * np.linalg.norm(want)


def bottlenecks(w, mid, h, m, shortcuts, first_scale=True):
    """Stem, then blocks 1x1 reduce - 1x1 expand + shortcut, then one more reduction that keeps the last block inside the stage.
    shortcuts: the tensor each block adds ('x': the block's input, 'in': the stage's)."""
    layers = [C(w, w, 1, 1, h, h, scale=first_scale)]
    for s in shortcuts:
        x = len(layers) - 1
        layers.append(C(w, mid, 1, 1, h, h, scale=True, src=x))
        layers.append(C(mid, w, 1, 1, h, h, scale=True, src=x + 1, add=x if s == "x" else -1))
    layers.append(C(w, mid, 1, 1, h, h, src=len(layers) - 1))
    return chain(*layers), m


def projected(cin, w, mid, h, m):
    """A block whose shortcut is a projection with a scale of its own."""
    return chain(C(cin, cin, 1, 1, h, h), C(cin, mid, 1, 1, h, h, scale=True, src=0), C(cin, w, 1, 1, h, h, relu=False, scale=True, src=0),
                 C(mid, w, 1, 1, h, h, scale=True, src=1, add=2), C(w, mid, 1, 1, h, h)), m


def down(c, w, h, m):
    """A basic block whose output two strided layers read."""
    g = (h - 1) // 2 + 1
    return chain(C(c, c, 1, 1, h, h, scale=True), C(c, c, 3, 3, h, h, p=1, scale=True), C(c, c, 3, 3, h, h, p=1, scale=True, src=1, add=0),
                 C(c, w, 3, 3, h, h, s=2, p=1, scale=True, src=2), C(c, w, 1, 1, h, h, s=2, relu=False, scale=True, src=2),
                 C(w, w, 3, 3, g, g, p=1, scale=True, src=3, add=4), C(w, c, 1, 1, g, g)), m


def read_thrice(c, h, m):
    """A tensor that two layers read and a third one adds."""
    return chain(C(c, c, 1, 1, h, h, scale=True), C(c, c, 1, 1, h, h, scale=True, src=0), C(c, c, 1, 1, h, h, relu=False, scale=True, src=0),
                 C(c, c, 3, 3, h, h, p=1, scale=True, src=1, add=2), C(c, c, 1, 1, h, h, scale=True, src=3, add=0), C(c, c, 1, 1, h, h)), m


def pooled_beside(c, h, m):
    """A tensor that a strided layer and a max-pooling read."""
    layers = chain(C(c, c, 1, 1, h, h, scale=True), C(c, c, 3, 3, h, h, s=2, p=1, scale=True, src=0), P(c, h, h),
                   C(c, c, 1, 1, h // 2, h // 2, scale=True, src=1, add=2))
    layers[2]["src"] = 0
    return layers, m


def branch(cin, c, mid, w, h, m, s=1, shared=False):
    """A block with a projection, both of stride s; shared: its last layer reads what the projection reads."""
    g = (h - 1) // s + 1
    if shared:
        return chain(C(cin, c, 1, 1, h, h), C(c, w, 1, 1, h, h, relu=False, scale=True, src=0), C(c, w, 3, 3, h, h, p=1, scale=True, src=0, add=1),
                     C(w, c, 1, 1, h, h)), m
    return chain(C(cin, c, 1, 1, h, h), C(c, mid, 3, 3, h, h, s=s, p=1, scale=True, src=0), C(c, w, 1, 1, h, h, s=s, relu=False, scale=True, src=0),
                 C(mid, w, 3, 3, g, g, p=1, scale=True, src=1, add=2), C(w, c, 1, 1, g, g)), m


def added_source(c, h, m):
    """A projection that reads the tensor which the layer beside it adds."""
    return chain(C(c, c, 1, 1, h, h, scale=True), C(c, c, 3, 3, h, h, p=1, scale=True, src=0, add=0), C(c, c, 1, 1, h, h, relu=False, scale=True, src=0),
                 C(c, c, 3, 3, h, h, p=1, scale=True, src=1, add=2), C(c, c, 1, 1, h, h)), m


def branches(c, h, m):
    """Three layers in a row that read the same tensor, two of them added further on."""
    return chain(C(c, c, 1, 1, h, h), C(c, c, 3, 3, h, h, p=1, scale=True, src=0), C(c, c, 1, 1, h, h, relu=False, scale=True, src=0),
                 C(c, c, 1, 1, h, h, relu=False, scale=True, src=0), C(c, c, 3, 3, h, h, p=1, scale=True, src=1, add=2),
                 C(c, c, 1, 1, h, h, scale=True, src=4, add=3), C(c, c, 1, 1, h, h)), m


def long_projection(cin, w, mid, h, wd, m):
    """The same with filters of 13 x 1."""
    return chain(C(cin, cin, 1, 1, h, wd), C(cin, mid, 13, 1, h, wd, scale=True, src=0), C(cin, w, 13, 1, h, wd, relu=False, bias=False, scale=True, src=0),
                 C(mid, w, 1, 1, h - 12, wd, scale=True, src=1, add=2), C(w, mid, 1, 1, h - 12, wd)), m


def mixed():
    return chain(C(16, 24, 3, 3, 14, 14, p=1), C(24, 40, 1, 1, 14, 14), C(40, 40, 3, 3, 14, 14, p=1, scale=True), C(40, 72, 3, 3, 14, 14, s=2, p=1),
                 C(72, 64, 5, 5, 7, 7, p=2), C(64, 6, 1, 1, 7, 7), C(6, 136, 3, 3, 7, 7, p=1), C(136, 128, 1, 1, 7, 7, scale=True), C(128, 64, 3, 3, 7, 7, p=1))


NETS = {
    # bf16: the masked sum of the contributions to a block's output, the gradient of its shortcut and, where two blocks share one, the
    # sum of both -- on every tile of the data gradient, in whole and in ragged row and channel tiles
    "tile64": (bottlenecks(64, 16, 12, 2, ["in", "x", "in"]), "bf16"),
    "tile64_ragged": (bottlenecks(72, 24, 11, 3, ["in", "in"]), "bf16"),
    "tile64_split": (bottlenecks(64, 2048, 4, 2, ["in", "in"]), "bf16"),
    "tile128x64": (bottlenecks(64, 16, 108, 2, ["in", "in"]), "bf16"),
    "tile128_8w": (bottlenecks(128, 16, 108, 2, ["in", "x", "in"]), "bf16"),
    "tile128_8w_ragged": (bottlenecks(120, 64, 109, 2, ["in", "in"]), "bf16"),
    "tile128": (bottlenecks(256, 16, 111, 2, ["in", "in"]), "bf16"),
    "tile256": ((chain(C(200, 200, 1, 1, 107, 109, scale=True), C(200, 88, 3, 3, 107, 109, p=1), C(88, 200, 1, 1, 107, 109, scale=True, add=0),
                       C(200, 88, 3, 3, 107, 109, p=1)), 2), "bf16"),
    # ... where the wavefronts of a block share the reduction
    "tile32": (down(192, 64, 16, 3), "bf16"),
    "tile32x64": (down(192, 64, 23, 3), "bf16"),
    "tile32_float": (down(64, 32, 27, 3), "f32"),
    "tile32x64_float": (down(64, 32, 38, 3), "f32"),
    "projected128": (projected(16, 128, 16, 108, 2), "bf16"),
    # the same in float, where a block's scale enters through the weights of its data gradient: channels in whole K tiles, in chunks of
    # 16 bytes, and gathered one by one
    "float_whole": (bottlenecks(32, 64, 40, 2, ["in", "x", "in"]), "f32"),
    "float_chunks": (bottlenecks(36, 20, 40, 2, ["in", "in"]), "f32"),
    "float_projected": (projected(20, 44, 36, 40, 2), "f32"),
    # tensors with several readers: the first one's data gradient adds what the others left, masks and hands on
    "down": (down(64, 128, 16, 3), "bf16"),
    "down_ragged": (down(40, 72, 13, 3), "bf16"),
    "down_float": (down(36, 44, 13, 3), "f32"),
    "read_thrice": (read_thrice(64, 14, 3), "bf16"),
    "read_thrice_float": (read_thrice(20, 14, 3), "f32"),
    "pooled_beside": (pooled_beside(64, 16, 3), "bf16"),
    "pooled_beside_float": (pooled_beside(20, 16, 3), "f32"),
    # contractions that share a launch: strided and not, in whole K tiles and in chunks, with one of them split, of more blocks than
    # the card has CUs; and those that cannot: both split, or reading or writing the same gradient
    "pair": (branch(16, 64, 64, 128, 9, 2), "bf16"),
    "pair_ragged": (branch(16, 40, 24, 72, 11, 2), "bf16"),
    "pair_split": (branch(16, 64, 512, 256, 8, 2, s=2), "bf16"),
    "pair_strided_ragged": (branch(16, 40, 24, 72, 17, 2, s=2), "bf16"),
    "pair_large": (branch(16, 64, 64, 128, 64, 8, s=2), "bf16"),
    "pair_float": (branch(8, 32, 64, 96, 17, 2), "f32"),
    "pair_float_large": (branch(8, 32, 64, 64, 64, 12, s=2), "f32"),
    "pair_float_ragged": (branch(8, 20, 44, 36, 65, 12, s=2), "f32"),
    "pair_both_split": (branch(16, 1536, 64, 64, 4, 2, s=2), "bf16"),
    "pair_three": (branches(64, 12, 2), "bf16"),
    "pair_three_float": (branches(20, 12, 2), "f32"),
    "pair_shared": (branch(16, 64, 0, 64, 12, 2, shared=True), "bf16"),
    "pair_added": (added_source(64, 12, 2), "bf16"),
    "pair_added_float": (added_source(32, 12, 2), "f32"),
    # layers whose dz carries their scale (their filter is too long for the weight gradients that multiply by it): the block's input, and
    # a projection
    "scaled_dz": ((chain(C(6, 16, 13, 1, 20, 12, bias=False, scale=True), C(16, 40, 3, 3, 8, 12, p=1, scale=True)), 2), "bf16"),
    "scaled_dz128": ((chain(C(6, 128, 13, 1, 120, 108, bias=False, scale=True), C(128, 16, 1, 1, 108, 108, scale=True)), 2), "bf16"),
    "scaled_dz_float": ((chain(C(6, 16, 13, 1, 20, 24, bias=False, scale=True), C(16, 40, 3, 3, 8, 24, p=1, scale=True)), 2), "f32"),
    "scaled_projection": (long_projection(6, 64, 16, 20, 12, 2), "bf16"),
    "scaled_projection128": (long_projection(6, 128, 16, 120, 108, 2), "bf16"),
    "scaled_projection_float": (long_projection(6, 64, 32, 32, 40, 2), "f32"),
    # data gradients gathered channel by channel, with scales on either side
    "gathered_bf16": ((chain(C(4, 6, 3, 3, 16, 16, p=1, scale=True), C(6, 10, 3, 3, 16, 16, p=1, scale=True), C(10, 7, 5, 5, 16, 16, scale=True)), 2), "bf16"),
    "gathered_float": ((chain(C(4, 6, 3, 3, 16, 16, p=1, scale=True), C(6, 10, 3, 3, 16, 16, p=1, scale=True), C(10, 7, 5, 5, 16, 16, scale=True)), 2), "f32"),
    # weight gradients of a backward pass cut into fewer pixel ranges than those of a lone call: filter rows, single taps, large tiles
    "ranges_rows": ((chain(C(64, 64, 3, 3, 64, 64, p=1, scale=True), C(64, 64, 1, 1, 64, 64, scale=True)), 9), "bf16"),
    "ranges_large": ((chain(C(256, 256, 1, 1, 128, 128, scale=True), C(256, 128, 1, 1, 128, 128)), 3), "bf16"),
    "ranges_float": ((chain(C(16, 32, 3, 3, 40, 40, p=1, scale=True), C(32, 16, 1, 1, 40, 40)), 9), "f32"),
    # weight gradients that share a launch: every kind of tile beside layers that have kernels of their own, in ragged channel counts
    # and pixel ranges, and 128-channel tiles
    "group_mixed": ((mixed(), 5), "bf16"),
    "group_mixed_float": ((mixed(), 5), "f32"),
    "group_large": ((chain(C(8, 16, 1, 1, 64, 64), C(16, 16, 1, 1, 64, 64), C(16, 256, 1, 1, 64, 64), C(256, 200, 1, 1, 64, 64, scale=True),
                           C(200, 256, 1, 1, 64, 64), C(256, 256, 1, 1, 64, 64)), 6), "bf16"),
}


@pytest.mark.parametrize("name", NETS)
def test_fused_backward(lpm, name):
    (layers, m), dtype = NETS[name]
    print("network", name, flush=True)
    stage_backward_isolated(lpm, layers, [0, len(layers)], m, m, 1 if dtype == "bf16" else 0, seed=23, dx_wanted=True, check_forward=True, grad_std=1.0)
