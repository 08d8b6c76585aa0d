"""The queue kernel (revisit_drain) and what steers it: block rows, queue capacity, spill queues, drain
budgets and sweep rounds.  Launches whose tasks sweep run on the register-resident kernel, which reads
none of these, so every task here asks for no sweeps (scan_rounds -1) or goes through the staged
pipeline, and a counter that only the queue kernel moves (queue entries that did not fit the queue of
64) shows that it ran.  Against the oracle, bit for bit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

SMALL = dict(scan_rounds=-1, queue_capacity=64)


@pytest.fixture(scope="module")
def lib():
    import paper_1209_3332_amd as p
    return p


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _tasks(conn):
    """One task of each operation, their oracle tasks, and the image each one leaves its result in."""
    marker, mask, binary = synth.config2_tile(seed=synth.seed_for(2, 11), size=768, n_gauss=106)
    sm, smask, _ = synth.spiral_tile(300, 520, "inner")
    up = np.minimum(mask.astype(np.int32) + 30, 255).astype(np.uint8)
    want = [{"op": "dilate", "marker": marker, "mask": mask, "conn": conn},
            {"op": "erode", "marker": up, "mask": mask, "conn": conn},
            {"op": "hdome", "img": mask, "h": 30, "conn": conn},
            {"op": "regional_max", "img": mask, "conn": conn},
            {"op": "fill_holes", "img": binary, "conn": conn},
            {"op": "dilate", "marker": sm, "mask": smask, "conn": conn}]
    out = []
    for t in want:
        two = "mask" in t
        s = {"op": t["op"], "image": _dev(t["marker"] if two else t["img"]), "conn": conn, "h": t.get("h", 0)}
        if two:
            s["mask"] = _dev(t["mask"])
        out.append(s)
    return out, want


def _check(oracle_mod, spec, want, what):
    for i, (s, t) in enumerate(zip(spec, want)):
        got = s["image"].cpu().numpy()
        ref = oracle_mod.run_task(t)
        assert np.array_equal(got, ref), "%s task %d (%s): %d px differ" % (what, i, t["op"], int((got != ref).sum()))


@pytest.mark.parametrize("conn", [8, 4])
@pytest.mark.parametrize("cfg", [dict(block_rows=16), dict(block_rows=32), dict(block_rows=64), dict(spill_capacity=-1),
                                 dict(spill_capacity=64), dict(drain_budget=1, binary_drain_budget=1),
                                 dict(drain_budget=4096, binary_drain_budget=4096), dict(wg_per_cu=1)], ids=str)
def test_knobs(lib, oracle_mod, cfg, conn):
    spec, want = _tasks(conn)
    with lib.Recon(0, component_route=-1, **SMALL, **cfg) as ctx:
        ctx.batch(spec)
        st = ctx.last_stats()
        assert st["aborted"] == 0 and st["queue_overflows"] + st["queue_spills"] > 0
        assert (st["queue_spills"] > 0) == (cfg.get("spill_capacity") != -1)
        _check(oracle_mod, spec, want, str(cfg))


@pytest.mark.parametrize("conn", [8, 4])
@pytest.mark.parametrize("cfg", [dict(scan_rounds=1), dict(scan_rounds=8), dict(block_rows=16, scan_rounds=2),
                                 dict(block_rows=64, queue_capacity=64), dict(drain_budget=1, binary_drain_budget=1),
                                 dict(drain_budget=4096, binary_drain_budget=4096)], ids=str)
def test_staged_pipeline_with_sweeps(lib, oracle_mod, cfg, conn):
    spec, want = _tasks(conn)
    with lib.Recon(0, stop_after_stage=3, timing=1, **cfg) as ctx:
        ctx.batch(spec)
        st = ctx.last_stats()
        assert st["aborted"] == 0 and st["dense_ms"] > 0   # (only the staged pipeline has a dense pass)
        _check(oracle_mod, spec, want, str(cfg))


@pytest.mark.parametrize("copies", [1, 4])   # direct launches and graph replays per group
def test_mixed_block_heights(lib, oracle_mod, copies):
    """Tasks of every block height in one batch: a launch per height, whose counters are summed."""
    heights = [16, 32, 64, 0]
    with lib.Recon(0, component_route=-1, block_rows=32, queue_capacity=64) as ctx:
        for rep in range(2):   # the groups' contexts and graphs are reused
            spec, want = [], []
            for conn in (8, 4) * copies:
                s, t = _tasks(conn)
                spec += s
                want += t
            blocks = 0
            for i, s in enumerate(spec):
                s.update(scan_rounds=-1, block_rows=heights[(i + rep) % 4])
                h, w = s["image"].shape
                blocks += -(-h // (s["block_rows"] or 32)) * -(-w // 256)
            ctx.batch(spec)
            st = ctx.last_stats()
            # every block of every task visited first once, at the task's own height
            assert st["aborted"] == 0 and st["dense_visits"] == blocks
            assert st["queue_overflows"] + st["queue_spills"] > 0
            _check(oracle_mod, spec, want, "heights")
