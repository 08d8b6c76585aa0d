"""Blocks whose pixel queue overflows in the staged pipeline's dense pass, which has no spill
queue: the block is seeded again until nothing is left, and nothing is written outside it.
Emulated, with LDS full of garbage as the hardware leaves it, under AddressSanitizer."""
import pytest

import kemu
import synth


@pytest.fixture(scope="module")
def emu_exe(tmp_path_factory):
    return kemu.build(str(tmp_path_factory.mktemp("kemu_staged")), sanitize=True)


@pytest.mark.parametrize("bh", [16, 32, 64])
@pytest.mark.parametrize("conn", [8, 4])
def test_dense_pass_overflow(emu_exe, oracle_mod, bh, conn):
    marker, mask, _ = synth.config2_tile(seed=synth.seed_for(2, 11), size=300, n_gauss=20)
    tasks = [{"op": "dilate", "marker": marker[:80], "mask": mask[:80], "conn": conn}]
    overflows = 0
    for rounds in (0, 1):
        for spill in (0, 64):   # (the revisits' queues; a block's own waves have none here)
            rc, outs, log = kemu.run(emu_exe, tasks, bh=bh, qcap=64, scan_rounds=rounds, n_waves=4, stop_after=3,
                                     spill=spill)
            assert rc == 0 and "ERROR: AddressSanitizer" not in log and "runtime error" not in log, log[-2000:]
            assert (outs[0] == oracle_mod.run_task(tasks[0])).all()
            overflows += int(log.split("overflow")[1].split()[0])
    assert overflows > 0
