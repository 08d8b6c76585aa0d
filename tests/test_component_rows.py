"""The offers and the result of two-valued masks, a row to a wave (launches of at most 256 units of 4 rows) and 4
rows to a wave (larger ones), against the oracle: both sides of the line, every remainder of 4 rows, several tasks."""
import numpy as np
import pytest

import kemu


def _pair(rng, h, w, p, few):
    mask = np.where(rng.random((h, w)) < p, 200, 0).astype(np.uint8)
    marker = rng.integers(0, 256, (h, w)).astype(np.uint8)
    return (marker * (marker > 250) if few else marker), mask


@pytest.fixture(scope="module")
def emu_exe(tmp_path_factory):
    return kemu.build(str(tmp_path_factory.mktemp("kemu_rows")), sanitize=True)


@pytest.mark.parametrize("conn", [8, 4])
@pytest.mark.parametrize("h", [30, 1024, 1025, 1043])   # blocks of 16 rows, 4 units each: 8, 256, 260 and 264
def test_emulated(emu_exe, oracle_mod, h, conn):
    rng = np.random.default_rng(h + conn)
    tasks = [dict(zip(("marker", "mask"), _pair(rng, h, 9, 0.6, False)), op="dilate", conn=conn)]
    rc, outs, log = kemu.run(emu_exe, tasks, bh=16, n_waves=4, component=1)
    assert rc == 0 and "ERROR: AddressSanitizer" not in log and "runtime error" not in log, log[-2000:]
    assert int(log.split("route")[1].split()[0]) == len(tasks)
    for t, got in zip(tasks, outs):
        assert np.array_equal(got, oracle_mod.run_task(t))


@pytest.mark.gpu
@pytest.mark.parametrize("conn", [8, 4])
@pytest.mark.parametrize("h,w", [(5, 332), (64, 4096), (65, 4096), (1021, 511), (1022, 512), (1023, 513), (1024, 700)])
def test_gpu(oracle_mod, h, w, conn):
    import torch
    import paper_1209_3332_amd as lib
    rng = np.random.default_rng(h + conn)
    with lib.Recon(0) as ctx:
        for p, few in ((0.3, False), (0.6, True), (0.9, False)):
            marker, mask = _pair(rng, h, w, p, few)
            want = oracle_mod.recon_dilate(marker, mask, conn)
            j, i = torch.from_numpy(marker).cuda(), torch.from_numpy(mask).cuda()
            ctx.dilate(j, i, conn)
            assert ctx.last_stats()["component_tasks"] == 1
            assert np.array_equal(j.cpu().numpy(), want), (p, few)
            js = [torch.from_numpy(marker).cuda() for _ in range(14)]      # a graph launch
            ctx.batch([{"op": "dilate", "image": x, "mask": i, "conn": conn} for x in js])
            assert ctx.last_stats()["component_tasks"] == len(js)
            assert all(np.array_equal(x.cpu().numpy(), want) for x in js), (p, few)
