"""What the distance transform holds and computes its values in: column distances are whole
32-bit elements of the plane between its two passes; squared distances and their root are exact
up to the largest sides it takes (16384: 2 * 16383^2 is below 2^30)."""
import subprocess

import numpy as np
import pytest

import kemu

NONE = 0x3fffffff   # no 0 pixel in the column


@pytest.fixture(scope="module")
def emu_exe(tmp_path_factory):
    return kemu.build(str(tmp_path_factory.mktemp("kemu_width")), sanitize=True)


@pytest.mark.parametrize("h,w", [(1, 1), (16, 4), (17, 64), (33, 67), (70, 260)])   # dword rows and odd ones, segment edges
def test_column_distances(emu_exe, tmp_path, h, w):
    img = (np.random.default_rng(h).random((h, w)) < 0.9).astype(np.uint8) * 255
    img[:, w // 2] = 1
    src, out = tmp_path / "img", tmp_path / "plane"
    img.tofile(src)
    subprocess.run([emu_exe, "cols", str(h), str(w), str(src), str(out)], check=True, timeout=120)
    y = np.arange(h)
    want = np.full((h, w), NONE, np.int64)
    for zy, zx in np.argwhere(img == 0):
        want[:, zx] = np.minimum(want[:, zx], abs(y - zy))
    assert np.array_equal(np.fromfile(out, np.int32).reshape(h, w), want)


def test_root(emu_exe):
    p = subprocess.run([emu_exe, "root"], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and "differ 0" in p.stdout, p.stdout + p.stderr


@pytest.mark.gpu
def test_largest_sides():
    """One 0 pixel in a corner of the largest image: every squared distance is known."""
    import torch
    import paper_1209_3332_amd as lib
    n = 16384
    img = torch.ones((n, n), dtype=torch.uint8, device="cuda")
    img[0, 0] = 0
    dist2 = torch.empty((n, n), dtype=torch.int32, device="cuda")
    sq = torch.arange(n, dtype=torch.int32, device="cuda") ** 2
    with lib.Recon(0) as ctx:
        ctx.distance(img, dist2)
        torch.cuda.synchronize()
        for y in range(0, n, 2048):
            assert torch.equal(dist2[y:y + 2048], sq[y:y + 2048, None] + sq[None]), y
        assert int(dist2[-1, -1]) == 2 * 16383 ** 2
