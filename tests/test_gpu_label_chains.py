"""Components whose labels hang on long chains of tiles: serpentines, a comb and a spiral across many
labelling tiles, whose unions meet walks over entries that other waves are moving.  Labels, area filter and hole
filling against the oracle."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _masks(h, w):
    y, x = np.mgrid[:h, :w]
    turn = np.where((y // 3) % 2 == 0, w - 1, 0)
    yield "a leg every 3 rows", (y % 3 == 0) | (x == turn)
    yield "the same down the columns", (x % 3 == 0) | (y == np.where((x // 3) % 2 == 0, h - 1, 0))
    yield "a comb", (x % 2 == 0) | (y == h - 1)
    yield "a spiral", synth.spiral_tile(h, w, "outer")[1] > 0


@pytest.mark.parametrize("conn", [8, 4])
@pytest.mark.parametrize("h,w", [(300, 517), (1025, 1030), (2995, 1846), (5000, 64), (61, 5003)])
def test_chains(oracle_mod, h, w, conn):
    import torch
    import paper_1209_3332_amd as lib
    with lib.Recon(0) as ctx:
        for what, m in _masks(h, w):
            mask = np.where(m, 255, 0).astype(np.uint8)
            want, n = oracle_mod.label(mask, conn)
            img = torch.from_numpy(mask).cuda()
            labels = torch.full((h, w), -7, dtype=torch.int32, device="cuda")
            ctx.label(img, labels, conn)
            got = labels.cpu().numpy()
            assert got.max() == n and np.array_equal(got, want), what
            ctx.fill_holes(img, conn)
            assert np.array_equal(img.cpu().numpy(), oracle_mod.fill_holes(mask, conn)), what
            img = torch.from_numpy(mask).cuda()
            ctx.area_threshold(img, 2, h * w // 4, conn)
            assert np.array_equal(img.cpu().numpy(), oracle_mod.area_threshold(mask, 2, h * w // 4, conn)), what
