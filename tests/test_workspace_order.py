"""A context's scheduler words are cleared when its workspace grows.  The clearing has to
come before the launch that follows on whatever stream that is: a memset on the null
stream, which returns before it has happened, is not waited for by the non-blocking streams
of the serving lanes, of the pipeline, of a batch's block heights or of the caller, and
would zero the words of a launch at work.

The library's host code runs here against a stand-in of the HIP runtime that keeps that order
(tests/fake_hip); no kernel runs."""
import os
import subprocess
import sys

import pytest

import kemu

HERE = os.path.dirname(os.path.abspath(__file__))
FAKE = os.path.join(HERE, "fake_hip")

PROGRAM = r"""
import ctypes, importlib.util, sys, types
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)   # (the name librecon.so asks for)
sys.modules["torch"] = types.ModuleType("torch")           # (its runtime must not be loaded beside)
import paper_1209_3332_amd as recon
lib = recon.load_library()
def ok(rc):
    assert rc == 0, lib.recon_last_error()
P = ctypes.c_void_p
ctx, stream = P(), P()
ok(lib.recon_create(ctypes.byref(ctx), 0, None))
fake.hipStreamCreateWithFlags(ctypes.byref(stream), 1)     # non-blocking
at = [1 << 20]
def image(h, w):
    at[0] += h * w
    return recon.recon_image(at[0] - h * w, h, w, w)
def task(side, rows=0):
    return recon.recon_task(0, 8, image(side, side), image(side, side), -1, 0, 0, rows)
def run(what):
    n = fake.fake_launches()
    if what == "plain":
        ok(lib.recon_dilate(ctx, ctypes.byref(image(64, 64)), ctypes.byref(image(64, 64)), 8, stream))
    elif what == "graph":
        ts = [task(64) for _ in range(20)]
        ok(lib.recon_batch(ctx, (recon.recon_task * 20)(*ts), 20, stream))
    elif what == "heights":
        ts = [task(64, r) for r in (16, 32, 64)]
        ok(lib.recon_batch(ctx, (recon.recon_task * 3)(*ts), 3, stream))
    else:
        for side in (64, 128, 16384):                      # lanes grow as requests do
            t = ctypes.c_uint64()
            ok(lib.recon_submit(ctx, ctypes.byref(task(side)), ctypes.byref(t)))
            ok(lib.recon_wait(ctx, t, 20000))
    assert fake.fake_launches() > n
run(sys.argv[2])
ok(lib.recon_destroy(ctx))
print("hazards", fake.fake_hazards())
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake_hip") / "libamdhip64.so.7")
    subprocess.run([kemu.CLANG, "-std=c++17", "-O1", "-fPIC", "-shared", "-I", kemu.SRC_DIR, "-w",
                    "-Wl,-soname,libamdhip64.so.7", "-o", out, os.path.join(FAKE, "fake_hip.cpp"), "-lpthread"], check=True)
    return out


@pytest.mark.parametrize("what", ["plain", "graph", "heights", "serving"])
def test_clearing_comes_before_the_launch(fake, what):
    p = subprocess.run([sys.executable, "-c", PROGRAM, fake, what], capture_output=True, text=True, timeout=120,
                       cwd=os.path.dirname(HERE))
    assert p.returncode == 0, p.stdout + p.stderr
    assert "hazards 0" in p.stdout, p.stdout
