"""The words a mask is classified by change one after the other.  A wave that reads them between another wave's
two atomics (its OR is there, the AND still the identity) must not take the mask for one of two values already
known and skip its own rows: a grey mask then took the route of the two-valued ones, with a wrong
result, where the samples had met no foreground.  Emulated, under AddressSanitizer."""
import subprocess

import numpy as np
import pytest

import kemu


@pytest.fixture(scope="module")
def emu_exe(tmp_path_factory):
    return kemu.build(str(tmp_path_factory.mktemp("kemu_words")), sanitize=True)


def _classify(exe, tmp_path, mask, o, n):
    src = tmp_path / "mask"
    mask.tofile(src)
    p = subprocess.run([exe, "classify", str(mask.shape[0]), str(mask.shape[1]), str(src), str(o), str(n)],
                       capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout + p.stderr
    words = p.stdout.split()
    return int(words[1]), int(words[3])


@pytest.mark.parametrize("first,other", [(200, 72), (72, 200), (1, 255), (255, 1), (128, 127)])
def test_between_the_two_atomics(emu_exe, tmp_path, first, other):
    mask = np.zeros((70, 300), np.uint8)
    mask[3:60:7, 5::9] = first
    mask[69, 299] = other        # the last row of the last block
    want = (first | other, first & other)
    # as the words start, as another wave's first atomic leaves them, as its second does
    for o, n in ((0, 255), (first, 255), (first, first)):
        assert _classify(emu_exe, tmp_path, mask, o, n) == want, (o, n)
    mask[69, 299] = first        # one value: known as that from any of them
    for o, n in ((0, 255), (first, 255), (first, first)):
        assert _classify(emu_exe, tmp_path, mask, o, n) == (first, first), (o, n)
