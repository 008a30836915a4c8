"""Performance cases of the training step, through the public entry points of the package.

Four kinds of work, each as a user's program does it:

  step    one mini-batch of a partitioned network: Net.step (every F_{z,j}, B_{z,j} and one update per stage)
  eval    forward pass of a whole network on one batch as a single stage: validation between epochs
  stage   one sub-module driven by hand, as a rank of a larger job drives it: forward, backward with the input
          gradient, Adam update
  layer   the three contractions of one convolution (forward, data gradient, weight gradient) on caller buffers

The networks are the layer lists of workloads.configs at the repository's own sizes, at batches from a few images to
what fills the card, at other image sizes and widths, in bfloat16 and float.
"""
import math

import torch

import paper_2207_11019_amd as lpm
from workloads import configs

LR, MU = 0.002, 0.9


# ---------------------------------------------------------------------------------------------- networks
def _network(c):
    """(layer list, number of stages, fixed plan or None) of a case."""
    net = c["net"]
    if net == "lenet":
        return configs.lenet(), 2, None
    if net == "vgg16_cifar":
        return configs.vgg16_cifar(), 4, None
    if net == "vgg16_224":
        return configs.vgg16_224(), 4, None
    if net == "resnet":          # basic blocks over four stages of the given first width
        w = c["width"]
        return configs.resnet18_cifar((w, 2 * w, 4 * w, 8 * w), c["blocks"], c["hw"], c["classes"]), 4, None
    if net == "bottleneck":      # one partition of bottleneck blocks, fed by the stage before and the stage after
        return configs.r50_conv4x(c["cin"], c["hw"], c["mid"], 4 * c["mid"], c["blocks"]), 1, None
    if net == "resattnet":       # volumetric residual network with self-attention
        w = c["width"]
        return configs.resattnet18_3d((w, 2 * w, 4 * w, 8 * w), 2, c["vol"]), 4, None
    raise ValueError(net)


def _in_elems(layers):
    ch, h, w = configs.in_shape(layers[0])
    return ch * h * w


def _dtype(c):
    return (lpm.BF16, torch.bfloat16) if c["dtype"] == "bf16" else (lpm.F32, torch.float32)


def _mac(l):
    """Multiply-adds of one sample in one direction."""
    if l["kind"] == "attn":
        p = l["h_in"] * l["w_in"]
        return 2 * p * p * l["cout"]
    if l["kind"] not in ("conv", "fc"):
        return 0
    if l["kind"] == "fc":
        return l["cout"] * l["cin"] * l.get("d_in", 1) * l["h_in"] * l["w_in"]
    d, h, w = configs.out_dhw(l)
    return d * h * w * l["cout"] * l["cin"] * l.get("kd", 1) * l["kh"] * l["kw"]


def _weights(layers):
    n = 0
    for l in layers:
        for k, s in configs.param_shapes(l).items():
            if k != "s":
                n += math.prod(s)
    return n


# ---------------------------------------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest step in use: a float LeNet on 28x28 digits, four micro-batches of eight
        dict(name="lenet_f32_b32", kind="step", net="lenet", dtype="f32", m=8, M=4, mode="overlapped"),
        # CIFAR training of a plain convolutional stack, batch 128
        dict(name="vgg16_cifar_b128", kind="step", net="vgg16_cifar", dtype="bf16", m=16, M=8, mode="overlapped"),
        # CIFAR training of a residual network, batch 256
        dict(name="resnet18_cifar_b256", kind="step", net="resnet", width=64, blocks=2, hw=32, classes=10, dtype="bf16", m=32, M=8,
             mode="overlapped"),
        # one partition of an ImageNet-size network, fed by its neighbours: the benchmark's headline
        dict(name="r50_conv4x_b64", kind="step", net="bottleneck", cin=512, hw=28, mid=256, blocks=6, dtype="bf16", m=16, M=4,
             mode="overlapped"),
        # the same partition with micro-batches sized for the card's memory
        dict(name="r50_conv4x_b512", kind="step", net="bottleneck", cin=512, hw=28, mid=256, blocks=6, dtype="bf16", m=128, M=4,
             mode="overlapped"),
        # the largest network: 224x224 images, 138 million weights
        dict(name="vgg16_224_b32", kind="step", net="vgg16_224", dtype="bf16", m=4, M=8, mode="overlapped"),
        # volumetric scans with self-attention, batch of six
        dict(name="resattnet18_3d_b6", kind="step", net="resattnet", width=32, vol=32, dtype="bf16", m=2, M=3, mode="overlapped"),
        # full-precision training of the same residual network (the precision the method was published with), run without overlap
        dict(name="resnet18_cifar_f32_b32", kind="step", net="resnet", width=64, blocks=2, hw=32, classes=10, dtype="f32", m=8, M=4,
             mode="locked"),
        # widths and images that are no power of two, micro-batches of odd size, 100 classes
        dict(name="resnet18_w48_hw48_b65", kind="step", net="resnet", width=48, blocks=2, hw=48, classes=100, dtype="bf16", m=13, M=5,
             mode="locked"),
        # validation: one image batch through the forward pass, small enough that launches count
        dict(name="eval_resnet18_b16", kind="eval", net="resnet", width=64, blocks=2, hw=32, classes=10, dtype="bf16", m=16),
        # one sub-module of a layer-wise partitioned job driven by its own loop, with Adam
        dict(name="stage_adam_hw14_b32", kind="stage", cin=256, cout=512, hw=14, dtype="bf16", m=32),
        # a single ragged layer: 27x27 images, 96 -> 160 channels, the contractions alone
        dict(name="layer_27x27_c96_k160", kind="layer", h=27, w=27, cin=96, cout=160, k=3, stride=1, dtype="bf16", m=24),
    ]


def _log(rng, lo, hi):
    """An integer between lo and hi, spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _fit(m, sample_bytes):
    """The nearest micro-batch whose inputs are whole 256-byte lines, as the library asks of micro-batch boundaries."""
    unit = 256 // math.gcd(256, sample_bytes)
    return max(1, round(m / unit)) * unit


def draw(rng):
    kind = rng.choices(("step", "eval", "stage", "layer"), (8, 1, 1, 2))[0]
    dtype = rng.choices(("bf16", "f32"), (5, 1))[0]
    es = 2 if dtype == "bf16" else 4
    if kind == "layer":
        k = rng.choice((1, 3, 3, 5))
        h, cin, cout = _log(rng, max(4, k), 112), 8 * _log(rng, 2, 96), 8 * _log(rng, 2, 96)
        stride = rng.choice((1, 1, 2))
        top = 2e10 if dtype == "bf16" else 2e9            # multiply-adds in one direction
        most = max(1, min(256, int(top / (h * h / stride ** 2 * cin * cout * k * k))))
        return dict(kind=kind, h=h, w=max(k, h + rng.randint(-2, 2)), cin=cin, cout=cout, k=k, stride=stride, dtype=dtype, m=_log(rng, 1, most))
    if kind == "stage":
        hw = rng.randint(7, 40)
        cin, cout = 32 * _log(rng, 1, 16), 32 * _log(rng, 1, 16)
        m = _log(rng, 1, 64 if dtype == "bf16" else 8)
        return dict(kind=kind, cin=cin, cout=cout, hw=hw, dtype=dtype, m=_fit(m, es * cin * hw * hw))
    if dtype == "f32" and kind == "step":                  # LeNet, or a residual network up to the listed one's work
        mode = rng.choice(("overlapped", "locked"))
        if rng.random() < 0.5:
            return dict(kind=kind, net="lenet", dtype=dtype, m=4 * _log(rng, 1, 32), M=rng.randint(1, 8), mode=mode)
        hw, width = rng.choice((16, 20, 24, 32)), rng.choice((32, 48, 64))
        m = _fit(_log(rng, 4, 16), es * 3 * hw * hw)
        return dict(kind=kind, net="resnet", width=width, blocks=rng.choice((1, 2)), hw=hw, classes=rng.choice((10, 100)), dtype=dtype, m=m,
                    M=rng.randint(1, max(1, 32 // m)), mode=mode)
    if kind == "eval":
        hw = rng.choice((16, 24, 32, 40, 48, 64))
        m = _fit(_log(rng, 1, 256 if dtype == "bf16" else 16), es * 3 * hw * hw)
        return dict(kind=kind, net="resnet", width=rng.choice((32, 48, 64, 96)), blocks=rng.choice((1, 2, 3)), hw=hw,
                    classes=rng.choice((10, 100, 1000)), dtype=dtype, m=m)
    mode = rng.choices(("overlapped", "locked"), (3, 1))[0]
    net = rng.choices(("vgg16_cifar", "vgg16_224", "resnet", "bottleneck", "resattnet"), (2, 1, 3, 3, 2))[0]
    if net == "vgg16_cifar":
        return dict(kind=kind, net=net, dtype=dtype, m=_log(rng, 2, 256), M=rng.randint(2, 8), mode=mode)
    if net == "vgg16_224":
        return dict(kind=kind, net=net, dtype=dtype, m=rng.randint(2, 8), M=rng.randint(1, 4), mode=mode)
    if net == "resnet":
        hw, width = rng.choice((24, 32, 40, 48, 56, 64)), rng.choice((32, 48, 64, 80, 96))
        unit = (width / 64 * hw / 32) ** 2 * (1 if width % 32 == 0 else 4)
        m = _fit(_log(rng, 4, max(4, min(256, 128 / unit))), es * 3 * hw * hw)
        return dict(kind=kind, net=net, width=width, blocks=rng.choice((1, 2, 3)), hw=hw, classes=rng.choice((10, 100)), dtype=dtype, m=m,
                    M=rng.randint(1, 8), mode=mode)
    if net == "bottleneck":
        hw, mid = 2 * rng.randint(7, 28), 32 * rng.randint(2, 8)
        m = _log(rng, 2, max(2, min(128, 128 * (28 / hw) ** 2)))
        return dict(kind=kind, net=net, cin=2 * mid, hw=hw, mid=mid, blocks=rng.randint(1, 6), dtype=dtype, m=m, M=rng.randint(1, 4), mode=mode)
    vol, width = rng.choice((16, 20, 24, 28, 32)), rng.choice((16, 32, 32, 64))
    if width == 64:
        vol = min(vol, 24)
    return dict(kind=kind, net=net, width=width, vol=vol, dtype=dtype, m=_fit(rng.randint(1, 4), es * vol ** 3), M=rng.randint(1, 4), mode=mode)


# ---------------------------------------------------------------------------------------------- inputs
def _normal(gen, n, std, tdt):
    return torch.randn(n, generator=gen, device="cuda", dtype=torch.float32).mul_(std).to(tdt)


def _gradient(gen, pixels, channels, tdt):
    """An upstream gradient: a mean of its own per channel, as pooling heads and biases hand down, and noise of that size."""
    return (_normal(gen, pixels * channels, 2e-4, torch.float32).view(pixels, channels) + _normal(gen, channels, 2e-4, torch.float32)).to(tdt).view(-1)


def _he(l):
    _, cin, kh, kw = configs.param_shapes(l)["W"]
    return math.sqrt(2.0 / (cin * kh * kw))


def _std(l):
    """Standard deviation of a layer's weights: He-normal, and a quarter of that for the last layer of a residual branch and for
    fully connected layers, which keeps activations, loss and gradients at the scale they have in a trained network."""
    return _he(l) * (0.25 if l["add_src"] is not None or l["kind"] == "fc" else l.get("w_gain", 1.0))


def _fill(gen, layers, stages, bufs, dtype):
    """Weights, biases and frozen scales (0.5..1.5) of every layer, and where the buffers hold it a momentum half the
    size of He-normal weights, an update of a thousandth of a weight per step: a run under way.  Drawn layer by layer."""
    for st, b in zip(stages, bufs):
        p = b["params"].view(torch.float32)
        v = b["momentum"].view(torch.float32) if "momentum" in b else None
        for i in range(st.first, st.last):
            l = layers[i]
            for which, k in enumerate(("W", "b", "s")):
                if k not in configs.param_shapes(l):
                    continue
                off, n = st.param_offset(i, which)
                if k == "s":
                    p[off:off + n] = torch.rand(n, generator=gen, device="cuda") + 0.5
                    continue
                w = _normal(gen, n, _std(l) if k == "W" else 0.05, torch.float32)
                p[off:off + n] = w.to(torch.bfloat16).float() if k == "W" and dtype == lpm.BF16 else w
                if v is not None:
                    v[off:off + n] = _normal(gen, n, 0.5 * _he(l), torch.float32)
        if dtype == lpm.BF16:
            st.sync_lowp(b["params"], b["lowp"])


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return {"step": _prepare_step, "eval": _prepare_eval, "stage": _prepare_stage, "layer": _prepare_layer}[case["kind"]](case, gen)


def _labels(gen, n, classes):
    """Classes of unequal frequency, as data sets have them."""
    return (torch.rand(n, generator=gen, device="cuda").square_() * classes).to(torch.int32).clamp_(max=classes - 1)


def _prepare_step(c, gen):
    layers, Z, fixed = _network(c)
    dtype, tdt = _dtype(c)
    cp = dict(lpm.MI355X_COST[c["dtype"]], link_byte_per_us=0, microbatch=c["m"], n_microbatch=c["M"])
    starts, _ = lpm.lpm_partition(layers, Z, cp, fixed)
    loss = layers[-1]["kind"] == "softmax_ce"
    net = lpm.Net(layers, starts, c["m"], c["M"], dtype, dx_wanted=not loss)
    s = dict(run="step", net=net, mode=lpm.LOCKED if c["mode"] == "locked" else lpm.OVERLAPPED, labels=None, dy=None, out={})
    _fill(gen, layers, net.stages, net.bufs, dtype)
    for z, st in enumerate(net.stages):
        b, n = net.bufs[z], st.grad_bytes // 4
        s["out"]["params%d" % z] = b["params"].view(torch.float32)[:n]
        s["out"]["momentum%d" % z] = b["momentum"].view(torch.float32)[:n]
    B = c["m"] * c["M"]
    s["x"] = _normal(gen, B * _in_elems(layers), 1.0, tdt)
    if loss:
        s["labels"] = _labels(gen, B, layers[-1]["cin"])
        s["out"]["loss"] = net.loss[:1]
    else:
        ch, h, w = configs.out_shape(layers[-1])
        s["dy"] = _gradient(gen, B * h * w, ch, tdt)
    return s


def _prepare_eval(c, gen):
    layers, _, _ = _network(c)
    dtype, tdt = _dtype(c)
    st = lpm.Stage(layers, 0, len(layers), c["m"], dtype)
    buf = lambda n: torch.zeros(max(n, 256), dtype=torch.uint8, device="cuda")      # noqa: E731
    params, lowp = buf(st.param_bytes), buf(st.lowp_bytes) if dtype == lpm.BF16 else None
    _fill(gen, layers, [st], [dict(params=params, lowp=lowp)], dtype)
    return dict(run="eval", st=st, params=params, lowp=lowp, x=_normal(gen, c["m"] * _in_elems(layers), 1.0, tdt),
                y=buf(st.out_bytes).view(tdt), labels=_labels(gen, c["m"], c["classes"]), loss=torch.zeros(1, device="cuda"),
                stash=buf(st.stash_bytes), ws=buf(st.fwd_ws_bytes), scale=1.0 / c["m"])


def _prepare_stage(c, gen):
    b = configs._Builder(c["cin"], c["hw"], c["hw"])
    b.conv(c["cout"], 3, stride=1, pad=1)
    b.conv(c["cout"], 3, stride=2, pad=1, scale=True)
    layers = b.finish()
    dtype, tdt = _dtype(c)
    st = lpm.Stage(layers, 0, len(layers), c["m"], dtype)
    buf = lambda n: torch.zeros(max(n, 256), dtype=torch.uint8, device="cuda")      # noqa: E731
    s = dict(run="stage", st=st, params=buf(st.param_bytes), lowp=buf(st.lowp_bytes) if dtype == lpm.BF16 else None, grads=buf(st.grad_bytes),
             m1=buf(st.grad_bytes), m2=buf(st.grad_bytes), stash=buf(st.stash_bytes), fws=buf(st.fwd_ws_bytes), bws=buf(st.bwd_ws_bytes),
             y=buf(st.out_bytes).view(tdt), dx=buf(st.in_bytes).view(tdt))
    _fill(gen, layers, [st], [s], dtype)
    n = st.grad_bytes // 4
    s["m1"].view(torch.float32)[:n] = _normal(gen, n, 1e-3, torch.float32)
    s["m2"].view(torch.float32)[:n] = _normal(gen, n, 1e-3, torch.float32).square_() + 1e-6
    s["x"] = _normal(gen, st.in_bytes // s["y"].element_size(), 1.0, tdt).relu_()
    s["dy"] = _gradient(gen, st.out_bytes // s["y"].element_size() // c["cout"], c["cout"], tdt)
    s["out"] = dict(y=s["y"], dx=s["dx"], grads=s["grads"].view(torch.float32), params=s["params"].view(torch.float32)[:n],
                    m1=s["m1"].view(torch.float32), m2=s["m2"].view(torch.float32))
    return s


def _geom(c):
    return dict(m=c["m"], h=c["h"], w=c["w"], cin=c["cin"], cout=c["cout"], kh=c["k"], kw=c["k"], stride=c["stride"], pad=c["k"] // 2)


def _out_hw(c):
    p = c["k"] // 2
    return (c["h"] + 2 * p - c["k"]) // c["stride"] + 1, (c["w"] + 2 * p - c["k"]) // c["stride"] + 1


def _prepare_layer(c, gen):
    g = _geom(c)
    dtype, tdt = _dtype(c)
    ho, wo = _out_hw(c)
    K = c["k"] * c["k"] * c["cin"]
    w = _normal(gen, c["cout"] * K, math.sqrt(2.0 / K), tdt)
    wt = w.view(c["cout"], c["k"] * c["k"], c["cin"]).permute(2, 1, 0).contiguous() if dtype == lpm.BF16 else None
    return dict(run="layer", g=g, dtype=dtype, w=w, wt=wt, x=_normal(gen, c["m"] * c["h"] * c["w"] * c["cin"], 1.0, tdt).relu_(),
                dz=_gradient(gen, c["m"] * ho * wo, c["cout"], tdt), y=torch.empty(c["m"] * ho * wo * c["cout"], dtype=tdt, device="cuda"),
                dx=torch.empty(c["m"] * c["h"] * c["w"] * c["cin"], dtype=tdt, device="cuda"), dw=torch.empty(c["cout"] * K, device="cuda"),
                bias=_normal(gen, c["cout"], 0.05, torch.float32),
                ws=torch.zeros(max(max(lpm.lpm_conv_ws_bytes(g, dtype)), 256), dtype=torch.uint8, device="cuda"))


# ---------------------------------------------------------------------------------------------- one pass
def run(s):
    kind = s["run"]
    if kind == "step":
        s["net"].step(s["x"], s["labels"], s["dy"], LR, MU, s["mode"])
        return s["out"]
    if kind == "eval":
        s["loss"].zero_()
        s["st"].forward(s["x"], s["y"], s["labels"], s["loss"], s["params"], s["lowp"], s["stash"], s["ws"], s["scale"],
                        torch.cuda.current_stream())
        return dict(logits=s["y"], loss=s["loss"])
    if kind == "stage":
        st, q = s["st"], torch.cuda.current_stream()
        st.forward(s["x"], s["y"], None, None, s["params"], s["lowp"], s["stash"], s["fws"], 1.0, q)
        st.backward(s["x"], s["y"], s["dy"], s["dx"], s["params"], s["lowp"], s["stash"], s["grads"], False, s["bws"], q)
        st.update_adam(s["params"], s["lowp"], s["grads"], s["m1"], s["m2"], 1e-4, 0.9, 0.999, 1e-8, 10, False, q)
        return s["out"]
    q = torch.cuda.current_stream()
    lpm.lpm_conv_forward(s["g"], s["dtype"], s["x"], s["w"], None, s["bias"], None, True, s["y"], s["ws"], q)
    lpm.lpm_conv_dgrad(s["g"], s["dtype"], s["dz"], s["w"], s["wt"], s["dx"], False, s["ws"], q)
    lpm.lpm_conv_wgrad(s["g"], s["dtype"], s["x"], s["dz"], s["dw"], False, s["ws"], q)
    return dict(y=s["y"], dx=s["dx"], dw=s["dw"])


# ---------------------------------------------------------------------------------------------- work and tolerance
def work(case):
    c = case
    es = 2 if c["dtype"] == "bf16" else 4
    if c["kind"] == "layer":
        ho, wo = _out_hw(c)
        x, y, w = c["m"] * c["h"] * c["w"] * c["cin"], c["m"] * ho * wo * c["cout"], c["cout"] * c["k"] ** 2 * c["cin"]
        return {"bytes": es * (2 * x + 2 * y + w) + 4 * w, "flops": 6 * y * c["k"] ** 2 * c["cin"]}
    if c["kind"] == "stage":
        o = (c["hw"] + 1) // 2
        w1, w2 = 9 * c["cin"] * c["cout"], 9 * c["cout"] ** 2
        x, y = c["m"] * c["hw"] ** 2 * c["cin"], c["m"] * o * o * c["cout"]
        # x and dy read, y and dx written; weights, two moments read and written, gradient written
        return {"bytes": es * 2 * (x + y) + 28 * (w1 + w2), "flops": 6 * c["m"] * (c["hw"] ** 2 * w1 + o * o * w2)}
    layers, _, _ = _network(c)
    mac, first = sum(_mac(l) for l in layers), _mac(layers[0])
    if c["kind"] == "eval":
        return {"bytes": c["m"] * es * (_in_elems(layers) + c["classes"]) + es * _weights(layers), "flops": 2 * c["m"] * mac}
    B, loss = c["m"] * c["M"], layers[-1]["kind"] == "softmax_ce"
    ends = B * es * (_in_elems(layers) + (0 if loss else _in_elems(layers) + math.prod(configs.out_shape(layers[-1]))))
    # weights and momentum read and written once
    return {"bytes": ends + 16 * _weights(layers), "flops": 2 * B * (3 * mac - (first if loss else 0))}


def tolerance(case):
    """bfloat16: a stored activation rounded the other way moves single layers by 2^-8, and the ReLU masks and pooling maxima it
    decides move the gradients of a deep network by a few per cent of their norm, single elements by more (two orders of
    summation of the forward pass: up to 1e-2 of the momentum after one step, 2e-2 after two).  float: the orders of
    summation alone, and in the networks the few masks that hinge on them."""
    if case["dtype"] == "bf16":
        return {"layer": {"rel": 4e-3, "max": 0.02}, "eval": {"rel": 0.015, "max": 0.06}}.get(case["kind"], {"rel": 0.03, "max": 0.9})
    return {"layer": {"rel": 2e-5, "max": 1e-3}, "eval": {"rel": 1e-4, "max": 1e-3}}.get(case["kind"], {"rel": 2e-3, "max": 0.5})
