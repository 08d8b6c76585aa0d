"""A flood that runs along the rows of one strip crosses its region in two passes, the second of which
closes the rows along their whole length, instead of a pass per few columns.  Counted in passes beyond
the visit's first (reruns), on the emulated kernel: one region, one workgroup, so the count is exact."""
import numpy as np
import pytest

import kemu


@pytest.fixture(scope="module")
def emu_exe(tmp_path_factory):
    return kemu.build(str(tmp_path_factory.mktemp("kemu_floods")), sanitize=False)


@pytest.mark.parametrize("conn", [8, 4])
@pytest.mark.parametrize("h,y0", [(1, 0), (3, 0), (100, 50), (128, 125)])   # all inside one strip of 16 rows
@pytest.mark.parametrize("side", ["left", "right"])
def test_flood_along_rows(emu_exe, oracle_mod, h, y0, conn, side):
    mask = np.full((h, 256), 3, np.uint8)
    mask[y0:y0 + 3] = 220 - np.arange(256) // 8     # falling: the flood's front moves on at every column
    if side == "right":
        mask = mask[:, ::-1].copy()
    marker = np.minimum(mask, 3)                    # (at rest everywhere else)
    x = 0 if side == "left" else 255
    marker[y0, x] = mask[y0, x]
    task = {"op": "dilate", "marker": marker, "mask": mask, "conn": conn}
    rc, outs, log = kemu.run(emu_exe, [task], bh=128, n_waves=1)
    assert rc == 0, log[-2000:]
    assert np.array_equal(outs[0], oracle_mod.run_task(task))
    assert int(log.split("rerun")[1].split()[0]) == 1, log
