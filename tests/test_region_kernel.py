"""The register-resident revisit kernel (csrc/region.hpp) against the oracle, at
the sizes where it can go wrong: the edges of a region (128 or 64 rows x 256 columns
as launched, 16 or 8 rows per wave), single rows and columns, rows that are not dword
aligned, long corridors, and the knobs that still choose the queue kernel."""
import numpy as np
import pytest

import kemu
import synth

# region edges in both directions, strip edges, ragged widths; the last two are
# above the 256 regions of 64 rows up to which a launch runs on those
SHAPES = [(1, 1), (1, 700), (300, 1), (8, 256), (17, 255), (63, 256), (64, 257), (65, 260), (129, 512), (257, 511),
          (8192, 260), (8193, 511)]


def _pairs(rng, h, w):
    """A grey nuclei-like pair, a few-level one (plateaus, marker above the mask) and a grey corridor."""
    mask = synth.gaussian_tile(h, w, max(1, h * w // 4000), noise=(-8, 8), background=30, seed=h * 1000 + w)
    yield synth.hdome_marker(mask, 20), mask
    yield synth.random_pair(rng, h, w, 3)[::-1]
    if h >= 16 and w >= 16:
        marker, corridor, _ = synth.spiral_tile(h, w, "outer")
        grey = np.where(corridor > 0, 200 + (np.arange(w) % 3)[None, :], 7).astype(np.uint8)
        yield np.minimum(marker, grey), grey


@pytest.fixture(scope="module")
def lib():
    import paper_1209_3332_amd as lib
    return lib


@pytest.fixture(scope="module")
def emu_exe(tmp_path_factory):
    return kemu.build(str(tmp_path_factory.mktemp("kemu_region")), sanitize=True)


@pytest.mark.parametrize("rows", [128, 8])   # as launched; 2 strips of 4 rows: many regions
@pytest.mark.parametrize("conn", [8, 4])
def test_emulated(emu_exe, oracle_mod, rows, conn):
    rng = np.random.default_rng(rows + conn)
    tasks = []
    for h, w in [(1, 1), (1, 300), (20, 1), (17, 255), (33, 260)] + ([(129, 257)] if rows == 128 else []):
        tasks += [{"op": "dilate", "marker": m, "mask": k, "conn": conn} for m, k in _pairs(rng, h, w)]
    grey = tasks[-2]["mask"]
    tasks += [{"op": "erode", "marker": np.full_like(grey, 255), "mask": grey, "conn": conn},
              {"op": "hdome", "img": grey, "h": 30, "conn": conn},
              {"op": "regional_max", "img": grey, "conn": conn},
              {"op": "fill_holes", "img": np.where(rng.random((40, 300)) < 0.6, 255, 0).astype(np.uint8), "conn": conn}]
    # 2 workgroups for all regions (taken from the ring), and one task with a
    # workgroup for each of its regions (which waits for its region's requests)
    for some, n_wg in ((tasks, 2), (tasks[12:13] if rows == 8 else tasks[-7:-6], 12)):
        rc, outs, log = kemu.run(emu_exe, some, bh=rows, n_waves=n_wg)
        assert rc == 0, log[-2000:]
        assert "ERROR: AddressSanitizer" not in log and "runtime error" not in log, log[-2000:]
        for i, (t, got) in enumerate(zip(some, outs)):
            assert np.array_equal(got, oracle_mod.run_task(t)), "task %d (%s)" % (i, t["op"])


def test_emulated_failed_claims(emu_exe):
    """Claims that keep failing give the launch up; every wave of every workgroup leaves."""
    m, k = synth.random_pair(np.random.default_rng(1), 140, 300, 4)
    rc, _, log = kemu.run(emu_exe, [{"op": "dilate", "marker": m, "mask": k, "conn": 8}], bh=128, n_waves=2,
                          test_fault=1, timeout=120)
    assert rc != 0 and "rc -3" in log and "aborted 1" in log, log[-2000:]


@pytest.mark.gpu
@pytest.mark.parametrize("conn", [8, 4])
@pytest.mark.parametrize("h,w", SHAPES)
def test_gpu_edges(lib, oracle_mod, h, w, conn):
    import torch
    rng = np.random.default_rng(h * 7 + w + conn)
    with lib.Recon(0, component_route=-1) as ctx:
        for marker, mask in _pairs(rng, h, w):
            for pad in (0, 5):   # rows one after the other, and rows 5 bytes further apart (no dword access)
                j = torch.zeros((h, w + pad), dtype=torch.uint8, device="cuda")[:, :w]
                i = torch.zeros((h, w + pad), dtype=torch.uint8, device="cuda")[:, :w]
                j.copy_(torch.from_numpy(marker))
                i.copy_(torch.from_numpy(mask))
                ctx.dilate(j, i, conn)
                st = ctx.last_stats()
                # first visits are counted in the caller's 32 x 256 blocks
                assert st["dense_visits"] == -(-h // 32) * -(-w // 256)
                want = oracle_mod.recon_dilate(marker, mask, conn)
                got = j.cpu().numpy()
                assert np.array_equal(got, want), "%d px differ (pad %d)" % (int((got != want).sum()), pad)
