"""Regions of 128 rows (region_drain<16, 8>) on the GPU: a launch runs on them when its images hold more
than 256 regions of 64 x 256, on regions of 64 rows otherwise ((8192, 260) still does: 128 x 2).  The
last region of a column ends on every kind of row: the first, inside a strip of 16, on a strip's edge,
one short of the region's edge and on it."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _regions64(shapes):
    return sum(-(-h // 64) * -(-w // 256) for h, w in shapes)


@pytest.fixture(scope="module")
def lib():
    import paper_1209_3332_amd as p
    return p


def _pair(h, w):
    mask = synth.gaussian_tile(h, w, max(1, h * w // 4000), noise=(-8, 8), background=30, seed=h * 1000 + w)
    return synth.hdome_marker(mask, 20), mask


@pytest.mark.parametrize("conn", [8, 4])
@pytest.mark.parametrize("rest", [1, 15, 16, 17, 64, 127, 128])   # rows of the last region
def test_last_region(lib, oracle_mod, rest, conn):
    import torch
    h, w = 26 * 128 + rest, 1030
    assert _regions64([(h, w)]) > 256
    marker, mask = _pair(h, w)
    want = oracle_mod.recon_dilate(marker, mask, conn)
    with lib.Recon(0, component_route=-1) as ctx:
        for pad in (2, 5):   # dword rows, and rows without dword access
            j = torch.zeros((h, w + pad), dtype=torch.uint8, device="cuda")[:, :w]
            i = torch.zeros((h, w + pad), dtype=torch.uint8, device="cuda")[:, :w]
            j.copy_(torch.from_numpy(marker))
            i.copy_(torch.from_numpy(mask))
            ctx.dilate(j, i, conn)
            assert ctx.last_stats()["aborted"] == 0
            got = j.cpu().numpy()
            assert np.array_equal(got, want), "%d px differ (pad %d)" % (int((got != want).sum()), pad)


@pytest.mark.parametrize("conn", [8, 4])
def test_small_images_beside_large_ones(lib, oracle_mod, conn):
    """Single pixels, rows and columns, images of a region and one pixel more, in a launch of 128-row regions."""
    import torch
    shapes = [(1, 1), (1, 700), (300, 1), (127, 255), (128, 256), (129, 257), (257, 511), (16, 1030), (8271, 260), (1100, 4097)]
    assert _regions64(shapes) > 256
    pairs = [_pair(h, w) for h, w in shapes]
    js = [torch.from_numpy(m).cuda() for m, _ in pairs]
    with lib.Recon(0, component_route=-1) as ctx:
        ctx.batch([{"op": "dilate", "image": j, "mask": torch.from_numpy(k).cuda(), "conn": conn}
                   for j, (_, k) in zip(js, pairs)])
        assert ctx.last_stats()["aborted"] == 0
        for (m, k), j in zip(pairs, js):
            assert np.array_equal(j.cpu().numpy(), oracle_mod.recon_dilate(m, k, conn)), k.shape
