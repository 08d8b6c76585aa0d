"""Labelling tiles (16 x 256 pixels, 4 rows a wave) and the per-component maxima
of two-valued masks (4 rows a wave) against the oracle, at the sizes where they can go
wrong: one row less and more than a wave's rows and a tile's, columns around a
tile's, on masks from a few pixels to almost full, labyrinths and combs (links across
every border of waves and tiles)."""
import numpy as np
import pytest

HEIGHTS = (1, 3, 4, 5, 15, 16, 17, 33)
WIDTHS = (1, 255, 256, 257, 518)


def _masks(h, w):
    rng = np.random.default_rng(1000 * h + w)
    for p in (0.02, 0.5, 0.62, 0.98):
        yield (rng.random((h, w)) < p).astype(np.uint8) * 255
    y, x = np.mgrid[:h, :w]
    yield np.where((x % 2 == 0) | (y == h - 1), 255, 0).astype(np.uint8)          # a comb joined at the bottom
    yield np.where((y % 2 == 0) | (x == np.where(y % 4 == 1, w - 1, 0)), 255, 0).astype(np.uint8)   # a serpentine
    yield np.where((x + y) % 2 == 0, 255, 0).astype(np.uint8)                     # diagonal neighbours only


@pytest.fixture(scope="module")
def lib():
    import paper_1209_3332_amd as lib
    return lib


@pytest.mark.gpu
@pytest.mark.parametrize("conn", [8, 4])
@pytest.mark.parametrize("h", HEIGHTS)
def test_gpu_tiles(lib, oracle_mod, h, conn):
    import torch
    with lib.Recon(0) as ctx:
        for w in WIDTHS:
            for n, mask in enumerate(_masks(h, w)):
                what = "%dx%d mask %d" % (h, w, n)
                want, n_want = oracle_mod.label(mask, conn)
                for pad in (0, 3):   # rows one after the other, and label rows without 16-byte alignment
                    labels = torch.full((h, w + pad + (w + pad + 1) % 2), -7, dtype=torch.int32, device="cuda")[:, :w]
                    img = torch.zeros((h, w + pad), dtype=torch.uint8, device="cuda")[:, :w]
                    img.copy_(torch.from_numpy(mask))
                    ctx.label(img, labels, conn)
                    got = labels.cpu().numpy()
                    assert got.max(initial=0) == n_want and np.array_equal(got, want), what
                    ctx.area_threshold(img, 2, 40, conn)
                    assert np.array_equal(img.cpu().numpy(), oracle_mod.area_threshold(mask, 2, 40, conn)), what
                marker = np.random.default_rng(n).integers(0, 256, (h, w)).astype(np.uint8)
                for m in (marker, marker * (marker > 250)):   # offers nearly everywhere; few
                    j, i = torch.from_numpy(m).cuda(), torch.from_numpy(mask).cuda()
                    ctx.dilate(j, i, conn)
                    assert ctx.last_stats()["component_tasks"] == 1, what
                    assert np.array_equal(j.cpu().numpy(), oracle_mod.recon_dilate(m, mask, conn)), what
