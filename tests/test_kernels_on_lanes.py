"""The GPU tests' small cases on the CPU, kernels run lane by lane (tests/lanes): beside the results that those tests compare,
every access lies in the operand it means, in the LDS of its launch and in the filter's or image's extent, and nothing rests on
a wait or barrier that is not there."""
import ctypes
import os
import subprocess
import sys

import pytest

TESTS = os.path.dirname(os.path.abspath(__file__))
LANES = os.path.join(TESTS, "lanes")
sys.path.insert(0, LANES)
import lanes_build  # noqa: E402


@pytest.fixture(scope="session")
def lanes(tmp_path_factory):
    return lanes_build.build(str(tmp_path_factory.mktemp("lanes")))


RUNS = [
    # loads land late, and in descending order of wavefronts and blocks, or early and ascending; file; selection
    (0, "test_gpu_contractions.py", "not m5_64x64 and not m3_1 and not m2_80 and not m2_107 and not m2_151"),
    (1, "test_gpu_contractions.py", "bf16_m1 or f32_m1 or f32_m2 or 3_4x4 or m2_4x4"),
    (1, "test_gpu_conv.py", "not m4_64x64 and not 57x59 and not 60x60 and not 32x32x64 and not d6k3_16 and not 15x15x512"),
    (0, "test_gpu_update.py", ""),
    (0, "test_gpu_fused.py", "not ranges and not 128 and not 256 and not large"),
    (1, "test_gpu_contractions.py", "88_200 or 256_768 or 256_192"),          # 256x128 tiles
    (1, "test_gpu_fused.py", "256 or large or (rows and tile128)"),           # ... large ones, groups and pairs of them, pooling over two pieces
    (1, "test_gpu_small.py", ""),
    (1, "test_gpu_wgrad32.py", "not m24"),
    (1, "test_gpu_rows.py", "not m2_115 and not m2_230 and not m2_100 and not m3_1 and not 32_wide and not backward_of"),
    (0, "test_gpu_rows.py", "m2_100x98_32 or m3_113x114_32 or (32_wide and 20)"),
    (1, "test_gpu_parity.py", "small_networks and bf16 and not graph and not pipelined"),
]


@pytest.mark.parametrize("late,name,select", RUNS, ids=["%s-%s%s" % (r[1][9:-3], "late" if r[0] else "early", "-large" if "not" not in r[2] and "256" in r[2] else "") for r in RUNS])
def test_gpu_tests_on_lanes(lanes, late, name, select):
    env = dict(os.environ, LPM_LANES=lanes, LPM_LANES_LATE=str(late), PYTHONPATH=os.pathsep.join([LANES, os.environ.get("PYTHONPATH", "")]))
    cmd = [sys.executable, "-m", "pytest", "-p", "lanes_plugin", "-p", "no:cacheprovider", "-q", "-m", "gpu", os.path.join(TESTS, name)]
    r = subprocess.run(cmd + (["-k", select] if select else []), env=env, cwd=os.path.dirname(TESTS), capture_output=True, text=True, timeout=900)
    assert r.returncode == 0, r.stdout[-6000:] + r.stderr[-3000:]
    assert " passed" in r.stdout and " failed" not in r.stdout


OPERANDS = """
import ctypes, lanes_plugin, torch
from paper_2207_11019_amd import binding
E = lanes_plugin._E
E.lanes_owned.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
guarded = lambda t: E.lanes_owned(t.data_ptr(), t.numel() * t.element_size()) and not E.lanes_owned(t.data_ptr(), t.numel() * t.element_size() + 1)
a = torch.zeros(640).cuda()
for t in (a, a.to(torch.bfloat16), a.clone(), a + 1, a.view(20, 32).t().contiguous(), torch.empty(64, dtype=torch.uint8, device="cuda")):
    assert binding._ptr(t) == t.data_ptr() and guarded(t)
assert binding._ptr(a[64:]) == a.data_ptr() + 256
try:
    binding._ptr(torch.zeros(640))
except AssertionError:
    print("refused")
"""


def test_operands_lie_between_pages_without_access(lanes):
    """Whatever torch makes of device memory is device memory, each tensor between pages of its own; host memory is refused.  (Operands in
    the heap had no such pages, and what was said of one held for the next at its address: a range too short, or one too long.)"""
    env = dict(os.environ, LPM_LANES=lanes, PYTHONPATH=os.pathsep.join([LANES, os.path.dirname(TESTS), os.environ.get("PYTHONPATH", "")]))
    r = subprocess.run([sys.executable, "-c", OPERANDS], env=env, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("refused"), r.stdout + r.stderr


LOADS = """
import ctypes, lanes_plugin, torch
import paper_2207_11019_amd as lpm
from test_gpu_conv import G
E = lanes_plugin._E
E.lanes_element_loads.restype = ctypes.c_long
def loads(call):
    before = E.lanes_element_loads()
    call()
    return E.lanes_element_loads() - before
for h, cin, cout, k in [(3, 106, 8, 1), (3, 8, 106, 1), (2, 600, 5, 1), (4, 18, 5, 3), (4, 5, 18, 3), (3, 2, 9, 2), (3, 9, 2, 2), (1, 1100, 3, 1)]:
    g = G(1, h, h, cin, cout, k, 1, 0)
    ho = h - k + 1
    f32 = lambda n: torch.randn(n).cuda()
    x, w, dz = f32(h * h * cin), f32(cout * k * k * cin), f32(ho * ho * cout)
    ws = torch.zeros(max(max(lpm.lpm_conv_ws_bytes(g, lpm.F32)), 256), dtype=torch.uint8, device="cuda")
    y, dx = f32(dz.numel()), f32(x.numel())
    for n, out, call in ((cin, dz.numel(), lambda: lpm.lpm_conv_forward(g, lpm.F32, x, w, None, None, None, False, y, ws)),
                         (cout, x.numel(), lambda: lpm.lpm_conv_dgrad(g, lpm.F32, dz, w, None, dx, 0, ws))):
        lanes = 64 if n >= 48 else 16 if n >= 12 else 4 if n >= 4 else 1
        turns, groups = -(-n // lanes), -(-out * lanes // 256) * 256 // lanes
        got = loads(call)
        assert 0 < got <= 2 * groups * k * k * turns * lanes, (g, n, got)
print("no more")
"""


def test_groups_of_lanes_load_the_terms_that_there_are(lanes):
    """Two loads per term of the lanes' turns through the channels of a tap, and none of turns that do not exist.  (Eight turns at a time of 106 channels
    on 64 lanes, two turns: four times the loads, and the time.)"""
    env = dict(os.environ, LPM_LANES=lanes, PYTHONPATH=os.pathsep.join([LANES, TESTS, os.path.dirname(TESTS), os.environ.get("PYTHONPATH", "")]))
    r = subprocess.run([sys.executable, "-c", LOADS], env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("no more"), r.stdout + r.stderr


COVERING = """
import ctypes, lanes_plugin, sys
import paper_2207_11019_amd as lpm
E = lanes_plugin._E
E.lpm_conv_forward.argtypes = lpm.lib.lpm_conv_forward.argtypes
E.lanes_host_only(1)
p = 1 << 20
for w in (32767, 32768):
    for dtype in (lpm.F32, lpm.BF16):
        g = lpm.lpm_conv_geom(1, 32768, w, 2, 8, 32768, w, 1, 0, 1, 1, 0)
        assert E.lpm_conv_forward(ctypes.byref(g), dtype, p, p, None, None, None, 0, p, p, None) == 0
"""


def test_covering_filters_of_31_bits(lanes):
    """A filter that covers its input is one tap of all its values while their number has 31 bits, and taps otherwise: 2^31 bfloat16 values had been a tap of
    -2^31 channels to the matrix-core kernel, the floats no channels to the group of lanes."""
    env = dict(os.environ, LPM_LANES=lanes, LPM_LANES_TRACE="1", PYTHONPATH=os.pathsep.join([LANES, os.path.dirname(TESTS), os.environ.get("PYTHONPATH", "")]))
    r = subprocess.run([sys.executable, "-c", COVERING], env=env, capture_output=True, text=True, timeout=120)
    kernels = [l.split("LDS: ")[1].replace("void ", "").replace("lpm::", "") for l in r.stderr.splitlines() if l.startswith("lanes: ") and "LDS: " in l]
    assert r.returncode == 0, r.stderr
    assert kernels == ["conv_fwd_generic<%s, 1, %s>" % (t, deep) for deep in ("true", "false") for t in ("float", "bf16_t")], kernels


HELD = """
import ctypes, lanes_plugin, torch
import paper_2207_11019_amd as lpm
from workloads import configs
E = lanes_plugin._E
E.lanes_hold.argtypes = [ctypes.c_void_p] + [ctypes.c_int] * 3
assert E.lanes_hold_twice() != 0, "a second call took the place of one that waits"
b = configs._Builder(16, 9, 9)
b.conv(16, 3, pad=1); b.gap(); b.conv(24, 1); b.conv(16, 1)
layers = b.finish()
def step(hold):
    torch.manual_seed(3)
    st = lpm.Stage(layers, 0, len(layers), 2, lpm.BF16)
    for i, fwd, bwd in hold:
        E.lanes_hold(st.h, i, fwd, bwd)
    buf = lambda n: torch.zeros(max(n, 256), dtype=torch.uint8, device="cuda")
    rnd = lambda n: (torch.randn(n // 2) * 0.1).to(torch.bfloat16).cuda()
    params, lowp, grads, stash, fws, bws = [buf(n) for n in (st.param_bytes, st.lowp_bytes, st.grad_bytes, st.stash_bytes, st.fwd_ws_bytes, st.bwd_ws_bytes)]
    params.view(torch.float32).copy_(torch.randn(params.numel() // 4) * 0.1)
    st.sync_lowp(params, lowp)
    x, dy, y, dx = rnd(st.in_bytes), rnd(st.out_bytes), buf(st.out_bytes), buf(st.in_bytes)
    st.forward(x, y, None, None, params, lowp, stash, fws, 1.0)
    st.backward(x, y, dy, dx, params, lowp, stash, grads, False, bws)
    assert y.any() and dx.any() and grads.any()
    return y, dx, grads, stash
want = step([])
for hold in ([(0, 1, 0)], [(3, 1, 0)], [(2, 0, 1)], [(0, 0, 1)], [(0, 1, 1), (2, 0, 1), (3, 1, 0)]):
    assert all(torch.equal(a, b) for a, b in zip(want, step(hold))), hold
print("all ran")
"""


def test_no_held_call_is_lost(lanes):
    """A contraction that waits for the next layer's launch runs before anything else that is launched, and at the end of its pass:
    in front of an average pooling, as the last layer of a stage, and as the first one of it on the way back."""
    env = dict(os.environ, LPM_LANES=lanes, PYTHONPATH=os.pathsep.join([LANES, os.path.dirname(TESTS), os.environ.get("PYTHONPATH", "")]))
    r = subprocess.run([sys.executable, "-c", HELD], env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("all ran"), r.stdout + r.stderr


@pytest.mark.parametrize("dtype,m,hw,c,n", [(1, 32769, 1, 8, 1), (0, 65537, 1, 4, 1), (1, 3, 4, 1032, 10)], ids=["bf16", "float", "small"])
def test_stop_event_stands_behind_the_head(lanes, dtype, m, hw, c, n):
    """The event that other streams wait for comes with the last launch of the kernel it is given to, whatever the number of samples.  (In
    groups of 32768 samples it came with the first one.)"""
    lib = ctypes.CDLL(lanes)
    lib.lanes_behind_head.restype = ctypes.c_long
    lib.lanes_host_only(1)
    left = lib.lanes_behind_head(dtype, m, hw, c, n)
    lib.lanes_host_only(0)
    assert left == 0


ROUTES = """
import ctypes, lanes_plugin, sys
import paper_2207_11019_amd as lpm
E = lanes_plugin._E
E.lpm_conv_forward.argtypes, E.lpm_conv_dgrad.argtypes = lpm.lib.lpm_conv_forward.argtypes, lpm.lib.lpm_conv_dgrad.argtypes
E.lanes_host_only(1)
p = 1 << 20
for m, d, h, w, c, n, k in %s:
    for fwd in (1, 0):
        kd = 3 if d > 1 else 1
        g = lpm.lpm_conv_geom(m, h, w, c if fwd else n, n if fwd else c, k, k, 1, k // 2, d, kd, kd // 2)
        if fwd: rc = E.lpm_conv_forward(ctypes.byref(g), lpm.BF16, p, p, None, None, None, 0, p, p, None)
        else: rc = E.lpm_conv_dgrad(ctypes.byref(g), lpm.BF16, p, p, p, p, 0, p, None)
        assert rc == 0
"""


# images, slices, height, width, channels of the reduction, outputs, filter; by filter rows in pieces?
@pytest.mark.parametrize("g,rows", [
    ((26, 1, 32, 32, 16, 224, 3), False), ((20, 1, 32, 32, 16, 224, 3), True),           # 16 channels, 3x3: 384 tiles of 128x128
    ((8, 1, 40, 40, 16, 72, 5), False), ((8, 1, 40, 40, 16, 64, 5), True),                # ... 5x5: 64 outputs
    ((2, 4, 20, 20, 16, 32, 3), False), ((3, 16, 20, 20, 16, 32, 3), True),               # ... volumes: 128 tiles of 128x32
    ((3, 16, 20, 20, 16, 40, 3), False),                                                  # ... and half a tile of outputs
    ((38, 1, 37, 37, 360, 208, 3), False), ((38, 1, 37, 37, 360, 192, 3), True),          # pieces of 48 against large tiles; 128x96 tiles of them
    ((5, 1, 37, 37, 360, 208, 3), True),                                                  # ... fewer than 384
    ((11, 1, 50, 50, 48, 120, 3), False), ((11, 1, 50, 50, 48, 96, 3), True), ((14, 1, 50, 50, 48, 120, 3), True),      # ... a round of CUs four fifths full
    ((47, 1, 88, 88, 48, 120, 3), False), ((47, 1, 88, 88, 48, 64, 3), True),
], ids=lambda v: "_".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_which_calls_go_in_pieces(lanes, g, rows):
    """... those that are no slower for it: in the others pieces are half empty, or their small tiles stand against large ones."""
    env = dict(os.environ, LPM_LANES=lanes, LPM_LANES_TRACE="1", PYTHONPATH=os.pathsep.join([LANES, os.path.dirname(TESTS), os.environ.get("PYTHONPATH", "")]))
    r = subprocess.run([sys.executable, "-c", ROUTES % [g]], env=env, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    kernels = [l.split("LDS: ")[1].replace("void ", "").replace("lpm::", "").split("<")[0] for l in r.stderr.splitlines() if l.startswith("lanes: ") and "LDS: " in l]
    assert kernels == ["rows_kernel" if rows else "igemm_kernel"] * 2, kernels


ORDER = """
import ctypes, lanes_plugin, sys, torch
import paper_2207_11019_amd as lpm
from test_gpu_conv import G, G3
E = lanes_plugin._E
E.lanes_lone_and_paired.argtypes = [ctypes.c_int, ctypes.POINTER(lpm.lpm_conv_geom)] + [ctypes.c_void_p] * 6
gen = torch.Generator().manual_seed(9)
rnd = lambda n: (torch.randn(n, generator=gen) * 2.0 ** torch.randint(-7, 8, (n,), generator=gen)).to(torch.bfloat16).cuda()
ws = torch.zeros(1 << 20, dtype=torch.uint8, device="cuda")
for c in (16, 32, 48):
    for op in (0, 1):
        volume = G3(2, 16, 24, 24, c, 24, 3, 1, 1) if c == 16 else G3(1, 4, 5, 7, c, 40, 3, 1, 1)
        for q in [G(2, 9, 14, c, 40, 3, 1, 1), G(2, 9, 11, c, 56, 5, 1, 2), dict(G(2, 6, 9, c, 24, 3, 1, 1), kh=2), volume, G(2, 1, 9, c, 40, 3, 1, 1)]:
            if op:
                q = dict(q, cin=q["cout"], cout=q["cin"])
            d, kd, pd = q.get("d", 1), q.get("kd", 1), q.get("pad_d", 0)
            rows_in, rows_out = q["m"] * d * q["h"] * q["w"], q["m"] * (d + 2 * pd - kd + 1) * (q["h"] + 2 - q["kh"] + 2 * (q["pad"] - 1) + 1) * q["w"]
            g = lpm.lpm_conv_geom(q["m"], q["h"], q["w"], q["cin"], q["cout"], q["kh"], q["kw"], 1, q["pad"], d, kd, pd)
            a, w = rnd((rows_out if op else rows_in) * c), rnd(q["cin"] * q["cout"] * kd * q["kh"] * q["kw"])
            out = [torch.zeros((rows_in * q["cin"]) if op else (rows_out * q["cout"]), dtype=torch.bfloat16, device="cuda") for _ in range(3)]
            assert E.lanes_lone_and_paired(op, ctypes.byref(g), *[t.data_ptr() for t in (a, w, *out, ws)]) == 0, (op, q)
            assert out[0].any() and torch.equal(out[0], out[1]) and torch.equal(out[1], out[2]), (op, q)
print("the same")
"""


@pytest.mark.parametrize("late", [0, 1], ids=["early", "late"])
def test_pieces_of_a_stage_keep_the_order_of_sums(lanes, late):
    """Layers of 16, 32 and 48 channels, which a stage runs by filter rows in pieces, give the bits of the chunks across taps that they go in where two
    of them share a launch: another order in a stage would move masks and maxima of the networks."""
    env = dict(os.environ, LPM_LANES=lanes, LPM_LANES_LATE=str(late), LPM_LANES_TRACE="1", PYTHONPATH=os.pathsep.join([LANES, TESTS, os.path.dirname(TESTS), os.environ.get("PYTHONPATH", "")]))
    r = subprocess.run([sys.executable, "-c", ORDER], env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("the same"), r.stdout + r.stderr
    kernels = [l.split("LDS: ")[1].replace("void ", "").replace("lpm::", "").split("<")[0] for l in r.stderr.splitlines() if l.startswith("lanes: ") and "LDS: " in l]
    assert kernels == ["rows_kernel", "igemm_pair"] * 30, kernels


DONE = """
import ctypes, lanes_plugin
import paper_2207_11019_amd as lpm
from workloads import configs
E = lanes_plugin._E
E.lanes_forward_done.argtypes = [ctypes.c_void_p]
E.lanes_host_only(1)
def done(relu, m, *more):
    b = configs._Builder(16, 9, 9)
    b.conv(16, 3, pad=1); b.gap(); b.conv(24, 1, relu=relu)
    for c in more: b.conv(c, 1)
    layers = b.finish()
    st = lpm.Stage(layers, 0, len(layers), m, lpm.BF16)
    return E.lanes_forward_done(st.h)
print([done(False, 2), done(False, 2, 16), done(True, 2), done(False, 1025)])
"""


def test_end_of_a_forward_pass_comes_with_its_last_kernel(lanes):
    """... also where that is the head's, which runs under the pooling's turn; a layer behind it, a head of two kernels."""
    env = dict(os.environ, LPM_LANES=lanes, PYTHONPATH=os.pathsep.join([LANES, os.path.dirname(TESTS), os.environ.get("PYTHONPATH", "")]))
    r = subprocess.run([sys.executable, "-c", DONE], env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("[1, 1, 1, 1]"), r.stdout + r.stderr


@pytest.mark.parametrize("m,hw,c,n,fwd,bwd", [(8, 1, 64, 10, 1, 1), (32, 16, 512, 10, 1, 1), (512, 16, 512, 128, 1, 1), (513, 1, 512, 33, 0, 0), (192, 1, 1024, 33, 1, 1),
                                              (193, 1, 1024, 33, 0, 1), (256, 1, 1024, 32, 1, 1), (257, 1, 1024, 32, 1, 0), (1024, 1, 256, 128, 1, 1),
                                              (2049, 1, 8, 33, 0, 1), (341, 1, 768, 33, 1, 1), (1088, 1, 8, 32, 1, 1), (4097, 15, 64, 10, 0, 0),
                                              (4097, 16, 64, 10, 0, 1), (1 << 23, 16, 8, 10, 0, 0),
                                              (8, 1, 1032, 33, 0, 1), (8, 4, 2048, 100, 0, 1), (8, 16, 2048, 32, 1, 1)])
def test_heads_that_share_a_kernel(lanes, m, hw, c, n, fwd, bwd):
    """... are those whose one kernel takes no longer than the pooling's and the contraction's: not with many samples, nor where every sample's block
    would read hundreds of kilobytes of weights.  (Up to 2048 channels and 128 outputs all of them did: 9 times the data gradient's time with 2048 samples.)"""
    lib = ctypes.CDLL(lanes)
    for dtype in (0, 1):
        if hw * c * (2 if dtype else 4) <= 65536:
            assert (lib.lanes_head(dtype, m, hw, c, n, 1), lib.lanes_head(dtype, m, hw, c, n, 0)) == (fwd, bwd)


@pytest.mark.parametrize("m,c,n", [(1089, 8, 32), (4096, 64, 32), (1025, 8, 33), (2048, 128, 128)])
def test_heads_of_many_samples_share_a_kernel_in_float(lanes, m, c, n):
    lib = ctypes.CDLL(lanes)
    assert [lib.lanes_head(dtype, m, 1, c, n, 1) for dtype in (0, 1)] == [1, 0]


@pytest.mark.parametrize("op,h,taken", [(0, 16382, True), (0, 16383, False), (1, 16381, True), (1, 16382, False)],
                         ids=["forward-in", "forward-out", "dgrad-in", "dgrad-out"])
def test_buffers_near_4_gib(lanes, op, h, taken):
    """The gathered tensor's buffer begins a halo early -- one image row and a pixel for the forward pass of a padded 3x3 filter, two of
    each for its data gradient -- and both together have to stay below 4 GiB: h rows of 16384 pixels of 16 bytes."""
    import paper_2207_11019_amd as lpm
    w, halo = 16384, (1 if op == 0 else 2)
    assert (h * w * 16 + halo * (w + 1) * 16 < (1 << 32) - 1) == taken
    g = lpm.lpm_conv_geom(1, h, w, 8, 8, 3, 3, 1, 1, 1, 1, 0)
    assert bool(ctypes.CDLL(lanes).lanes_takes(op, lpm.BF16, ctypes.byref(g))) == taken


def test_lds_limits_are_set_per_device(lanes):
    """Kernels with more than 64 KB of LDS, each launched on a first and then on a second device of the process: a device takes
    such a launch only after the attribute was set with that device current."""
    import paper_2207_11019_amd as lpm
    lib = ctypes.CDLL(lanes)
    lib.lanes_complaints.restype = ctypes.c_long
    for name in ("lpm_conv_forward", "lpm_conv_dgrad", "lpm_conv_wgrad", "lpm_stage_create", "lpm_stage_forward", "lpm_stage_backward"):
        getattr(lib, name).argtypes = getattr(lpm.lib, name).argtypes
    p = 1 << 20                            # any address: the launches are not run
    geoms = [(2, 9, 7, 24, 40, 3, 1), (3, 128, 128, 8, 64, 3, 1), (1, 152, 152, 8, 128, 1, 0), (12, 128, 128, 128, 128, 1, 0), (12, 128, 128, 128, 128, 5, 2),
             (5, 64, 64, 256, 256, 3, 1), (2, 70, 70, 6, 16, 5, 0)]
    attn = lpm.layers_from_dicts([dict(kind="attn", cin=96, cout=32, kh=1, kw=1, stride=1, pad=0, h_in=31, w_in=31, src=-1)])
    lib.lanes_host_only(1)
    for dev in (0, 1, 0):
        lib.lanes_set_device(dev)
        before = lib.lanes_complaints()
        for m, h, w, cin, cout, k, pad in geoms:
            g = lpm.lpm_conv_geom(m, h, w, cin, cout, k, k, 1, pad, 1, 1, 0)
            for dt in (lpm.BF16, lpm.F32):
                assert lib.lpm_conv_forward(ctypes.byref(g), dt, p, p, None, None, None, 0, p, p, None) == 0
                assert lib.lpm_conv_dgrad(ctypes.byref(g), dt, p, p, p if dt == lpm.BF16 else None, p, 0, p, None) == 0
                assert lib.lpm_conv_wgrad(ctypes.byref(g), dt, p, p, p, 0, p, None) == 0
        st = ctypes.c_void_p()
        assert lib.lpm_stage_create(attn, 1, 0, 1, 2, lpm.BF16, ctypes.byref(st)) == 0
        assert lib.lpm_stage_forward(st, p, p, None, None, p, p, p, p, 1.0, None) == 0
        assert lib.lpm_stage_backward(st, p, p, p, p, p, p, p, p, 0, p, None) == 0
        lib.lpm_stage_destroy(st)
        assert lib.lanes_complaints() == before, "device %d" % dev
    lib.lanes_host_only(0)
