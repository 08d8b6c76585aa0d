"""A device synchronisation, on any thread, fails while any stream is being captured, and
breaks that capture: what is then sent to a stream forked from it runs at once.  A context
that grows (a serving lane's, on the worker thread) and another that captures a batch's
graph take turns, so that neither call fails; a capture that somebody else's synchronisation
broke does not fail the batch, which is launched kernel by kernel, and none of its kernels
runs before that.

The library's host code runs here against a stand-in of the HIP runtime that keeps these
rules (tests/fake_hip); no kernel runs."""
import os
import subprocess
import sys

import pytest

from test_workspace_order import HERE, PROGRAM, fake  # noqa: F401  (the stand-in, built)

COMMON = PROGRAM[:PROGRAM.index("def run(what)")] + r"""
import threading
def batch(c, n=20):
    ts = [task(64) for _ in range(n)]
    return lib.recon_batch(c, (recon.recon_task * n)(*ts), n, stream)
fake.fake_capture_ms(20)
"""

GROWTH = COMMON + r"""
errors, stop = [], threading.Event()
def serve():
    side = 8192
    while not stop.is_set() and side < 30000:     # each request larger: its lane grows
        t, side = ctypes.c_uint64(), side + 512
        if lib.recon_submit(ctx, ctypes.byref(task(side)), ctypes.byref(t)) or lib.recon_wait(ctx, t, 10000000):
            errors.append(lib.recon_last_error())
th = threading.Thread(target=serve)
th.start()
for _ in range(10):                               # each context captures its first batch
    c = P()
    if lib.recon_create(ctypes.byref(c), 0, None) or batch(c):
        errors.append(lib.recon_last_error())
    ok(lib.recon_destroy(c))
stop.set()
th.join()
ok(lib.recon_destroy(ctx))
print("breaks", fake.fake_breaks(), "errors", errors)
"""

BROKEN = COMMON + r"""
def outside():                                    # another thread synchronises the device once
    while fake.hipDeviceSynchronize() == 0:
        pass
    fake.hipGetLastError()
th = threading.Thread(target=outside)
th.start()
n = fake.fake_launches()
ok(batch(ctx))
th.join()
direct = fake.fake_launches() - n
for _ in range(2):                                # (captured anew, then replayed)
    n = fake.fake_launches()
    ok(batch(ctx))
    assert fake.fake_launches() - n == 1, fake.fake_launches() - n
ok(lib.recon_destroy(ctx))
print("breaks", fake.fake_breaks(), "direct", direct > 3, "strays", fake.fake_strays())
"""


def run(program, fake):  # noqa: F811
    p = subprocess.run([sys.executable, "-c", program, fake], capture_output=True, text=True, timeout=120,
                       cwd=os.path.dirname(HERE))
    assert p.returncode == 0, p.stdout + p.stderr
    return p.stdout


def test_growth_waits_for_captures(fake):  # noqa: F811
    assert "breaks 0 errors []" in run(GROWTH, fake)


def test_broken_capture_is_launched_directly(fake):  # noqa: F811
    assert "breaks 1 direct True strays 0" in run(BROKEN, fake)
