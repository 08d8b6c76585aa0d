"""The route of every task of a launch is decided once: whatever the words it is decided by
hold while they are read, each task is on the component route or owns one range of ring positions,
the ranges lie end to end, and their sum is the launch's outstanding work."""
import subprocess

import pytest

import kemu


@pytest.fixture(scope="module")
def emu_exe(tmp_path_factory):
    return kemu.build(str(tmp_path_factory.mktemp("kemu_route")), sanitize=False)


@pytest.mark.parametrize("n", [1, 2, 16, 64, 65, 200])   # 64 tasks a step
def test_ring_ranges(emu_exe, n):
    p = subprocess.run([emu_exe, "decide", str(n), "40", str(n)], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and "broken 0" in p.stdout, p.stdout + p.stderr
