"""Masks whose foreground lies between the pixels that the first look at a mask samples (64 columns of 16 rows): every
wave of the classification then meets values that the task's words do not show yet.  One value: the
component route; one pixel of another value, wherever it lies: the block route.  Against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _unsampled(h, w, rng):
    mask = np.where(rng.random((h, w)) < 0.5, 200, 0).astype(np.uint8)
    mask[:, [((2 * k + 1) * w) // 128 for k in range(64)]] = 0
    return mask


@pytest.mark.parametrize("conn", [8, 4])
@pytest.mark.parametrize("h,w", [(130, 300), (1025, 1030), (2048, 2048)])
def test_routes(oracle_mod, h, w, conn):
    import torch
    import paper_1209_3332_amd as lib
    rng = np.random.default_rng(h + conn)
    mask = _unsampled(h, w, rng)
    marker = rng.integers(0, 256, (h, w)).astype(np.uint8)
    on = np.argwhere(mask > 0)
    with lib.Recon(0, component_route=1) as ctx:
        def run(m):
            j, i = torch.from_numpy(marker).cuda(), torch.from_numpy(m).cuda()
            ctx.dilate(j, i, conn)
            route = ctx.last_stats()["component_tasks"]
            assert np.array_equal(j.cpu().numpy(), oracle_mod.recon_dilate(marker, m, conn))
            return route
        assert run(mask) == 1
        for at in (0, len(on) // 2, -1):   # the first, a middle and the last foreground pixel
            grey = mask.copy()
            grey[tuple(on[at])] = 72       # (shares a bit with 200: neither word alone tells them apart)
            assert run(grey) == 0
        # a batch of both (a graph launch)
        pairs = [mask, grey] * 7
        js = [torch.from_numpy(marker).cuda() for _ in pairs]
        ctx.batch([{"op": "dilate", "image": j, "mask": torch.from_numpy(m).cuda(), "conn": conn}
                   for j, m in zip(js, pairs)])
        assert ctx.last_stats()["component_tasks"] == 7
        for j, m in zip(js, pairs):
            assert np.array_equal(j.cpu().numpy(), oracle_mod.recon_dilate(marker, m, conn))
