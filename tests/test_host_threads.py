"""The schedules' enqueue threads under ThreadSanitizer, and the lifetime of their handles, events and threads under AddressSanitizer
(no GPU: the runtime of tests/lanes with launches not run)."""
import os
import subprocess
import sys

import pytest

TESTS = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(TESTS, "lanes"))
import lanes_build  # noqa: E402


@pytest.mark.parametrize("kind", ["thread", "address"])
def test_enqueue_threads_under_sanitizer(tmp_path, kind):
    exe = lanes_build.build(str(tmp_path), flags=["-fsanitize=" + kind], extra=[os.path.join(TESTS, "host_threads.cpp")], exe="host_threads", opt="-O1")
    # (a thread that comes late to a step it has no part in does so in two runs of three)
    for _ in range(4 if kind == "thread" else 1):
        r = subprocess.run([exe], capture_output=True, text=True, timeout=600, env=dict(os.environ, TSAN_OPTIONS="exitcode=66", ASAN_OPTIONS="detect_leaks=0"))
        assert "Sanitizer" not in r.stderr and r.returncode == 0, (r.returncode, r.stdout[-500:], r.stderr[:6000])
        assert r.stdout.strip().endswith("done, 0 complaints")
