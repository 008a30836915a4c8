import faulthandler
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

# A GPU test that takes the process with it (the GPU runtime aborts from a thread of its own) leaves its name as the last line of the output
# and of this file, which also gets the stack of every Python thread -- in the output that dump would push the name out of sight.
LOG = os.environ.get("GPU_TEST_LOG", os.path.join(ROOT, "gpu_tests.log"))
_log = None


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def _started(nodeid):
    global _log
    if _log is None:
        try:
            _log = open(LOG, "wb", buffering=0)
            faulthandler.enable(file=_log)
        except OSError:
            _log = False
    if _log:
        _log.write((nodeid + "\n").encode())
    print(nodeid, flush=True)                  # (output is not captured between tests)


@pytest.hookimpl(hookwrapper=True)
def pytest_runtest_protocol(item, nextitem):
    if item.get_closest_marker("gpu"):
        _started(item.nodeid)
    yield
