"""pytest plugin: the GPU tests with the library's kernels running lane by lane on the CPU (see lanes.cpp), device memory being host
memory between pages without access.  LPM_LANES names the library that lanes_build.build() made, LPM_LANES_LATE=1 asks for loads
that land late and the descending order of wavefronts and blocks, LPM_LANES_TRACE=1 for a line per launch on stderr."""
import ctypes
import os

import pytest
import torch
import torch.overrides

_CDLL = ctypes.CDLL
_E = _CDLL(os.environ["LPM_LANES"])
_E.lanes_alloc.restype, _E.lanes_alloc.argtypes = ctypes.c_void_p, [ctypes.c_size_t]
_E.lanes_owned.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
_E.lanes_complaints.restype = ctypes.c_long
_E.lanes_late(int(os.environ.get("LPM_LANES_LATE", "0")))


class _Library(_CDLL):
    def __init__(self, name, *a, **k):
        super().__init__(os.environ["LPM_LANES"] if str(name).endswith("liblpm.so") else name, *a, **k)


class _Stream:
    made = 0

    def __init__(self, *a, **k):
        _Stream.made += 1
        self.cuda_stream = _Stream.made

    def wait_stream(self, other):
        pass

    def synchronize(self):
        pass


def _on_gpu(device):
    return device is not None and "cuda" in str(device)


def _device_memory(t):
    return t.numel() > 0 and bool(_E.lanes_owned(t.data_ptr(), t.numel() * t.element_size()))


def _moved(t):
    """A copy in device memory of its own."""
    t = t.contiguous()
    n = t.numel() * t.element_size()
    if n == 0:
        return t
    r = torch.frombuffer((ctypes.c_ubyte * n).from_address(_E.lanes_alloc(n)), dtype=torch.uint8).view(t.dtype).view(t.shape)
    return r.copy_(t)


def _made(f):
    def g(*a, device=None, **k):
        t = f(*a, **k)
        return _moved(t) if _on_gpu(device) else t
    return g


_to = torch.Tensor.to


def _tensor_to(t, *a, device=None, **k):
    names = [x for x in a if isinstance(x, str)]
    a = [x for x in a if not isinstance(x, str)]
    r = _to(t, *a, **k) if (a or k) else t
    return _moved(r) if _on_gpu(device or (names[0] if names else None)) else r


class _StaysThere(torch.overrides.TorchFunctionMode):
    """What torch makes of a tensor in device memory is in device memory, too: operands of a call that lay in the heap would have no pages
    without access around them, and the next tensor there would stand for what was freed."""
    def __torch_function__(self, f, types, args=(), kwargs=None):
        r = f(*args, **(kwargs or {}))
        if isinstance(r, torch.Tensor) and not _device_memory(r) and any(isinstance(t, torch.Tensor) and _device_memory(t) for t in args):
            return _moved(r)
        return r


ctypes.CDLL = _Library
torch.cuda.is_available = lambda: True
torch.cuda.synchronize = lambda *a: None
torch.cuda.Stream = _Stream
_current = _Stream()
torch.cuda.current_stream = lambda *a: _current
torch.device = lambda *a: str(a[0])
for _n in ("zeros", "empty", "full", "rand", "randn"):
    setattr(torch, _n, _made(getattr(torch, _n)))
torch.Tensor.cuda = lambda t, *a, **k: _moved(t)
torch.Tensor.to = _tensor_to
_StaysThere().__enter__()

import paper_2207_11019_amd.binding as binding  # noqa: E402


def _ptr(t):
    if t is None or isinstance(t, int):
        return t
    assert t.numel() == 0 or _device_memory(t), "host memory handed to the library: a tensor of %s" % str(tuple(t.shape))
    return t.data_ptr()


binding._ptr = _ptr


@pytest.hookimpl(hookwrapper=True)
def pytest_runtest_call(item):
    before = _E.lanes_complaints()
    outcome = yield
    if not outcome.excinfo and _E.lanes_complaints() > before:
        outcome.force_exception(AssertionError("%d accesses or launches to complain about (see stderr)" % (_E.lanes_complaints() - before)))
