"""Strips, images of at most 192 rows: they run on regions of 64 rows whatever their length, and a
flood along them crosses a region in few passes.  Around the line, more than 256 regions of 64 rows, both
row alignments, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_1209_3332_amd as p
    return p


def _flood(rng, h, w):
    mask = np.clip(np.cumsum(rng.integers(-3, 4, (h, w)), axis=1) + 128, 0, 255).astype(np.uint8)
    marker = np.minimum(mask, 2)
    marker[h // 2, 0] = mask[h // 2, 0]
    return marker, mask


@pytest.mark.parametrize("conn", [8, 4])
@pytest.mark.parametrize("h,w", [(1, 70000), (3, 66001), (64, 66000), (65, 33100), (191, 22300), (192, 22303), (193, 22300)])
def test_floods(lib, oracle_mod, h, w, conn):
    import torch
    assert -(-h // 64) * -(-w // 256) > 256
    marker, mask = _flood(np.random.default_rng(h), h, w)
    want = oracle_mod.recon_dilate(marker, mask, conn)
    with lib.Recon(0) as ctx:
        for pad in (-w % 4, 4 - (w + 1) % 4 + 1):   # dword rows, and rows that are not
            j = torch.zeros((h, w + pad), dtype=torch.uint8, device="cuda")[:, :w]
            i = torch.zeros((h, w + pad), dtype=torch.uint8, device="cuda")[:, :w]
            j.copy_(torch.from_numpy(marker))
            i.copy_(torch.from_numpy(mask))
            ctx.dilate(j, i, conn)
            assert ctx.last_stats()["aborted"] == 0
            assert np.array_equal(j.cpu().numpy(), want), pad


def test_a_strip_beside_a_tile(lib, oracle_mod):
    """A launch of strips and one image that is none."""
    import torch
    rng = np.random.default_rng(5)
    pairs = [_flood(rng, h, w) for h, w in ((5, 30000), (192, 9000), (193, 9000), (1, 1), (192, 256))]
    for some in (pairs[:2], pairs):
        js = [torch.from_numpy(m).cuda() for m, _ in some]
        with lib.Recon(0) as ctx:
            ctx.batch([{"op": "dilate", "image": j, "mask": torch.from_numpy(k).cuda(), "conn": 4}
                       for j, (_, k) in zip(js, some)])
            for (m, k), j in zip(some, js):
                assert np.array_equal(j.cpu().numpy(), oracle_mod.recon_dilate(m, k, 4)), k.shape
