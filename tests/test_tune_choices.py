"""What the autotuner may choose (CPU only): every candidate can run differently from the others (tasks that
sweep all run on the register-resident kernel, which reads no other knob), and a batch whose buckets
chose both kernels does not go to the queue kernel as a whole."""
import numpy as np

from paper_1209_3332_amd import tune


def _task(side, conn):
    return {"op": "dilate", "image": np.zeros((side, side), np.uint8), "mask": None, "conn": conn}


def test_candidates_run_differently():
    c = tune.candidates()
    sweeping = [x for x in c if x["scan_rounds"] >= 1]
    assert sweeping == [tune.config_for({}, 512, 512, 8)]     # one, the default
    queue = [(x["block_rows"], x["queue_capacity"]) for x in c if x["scan_rounds"] == -1]
    assert len(queue) == len(set(queue)) == len(c) - 1 == len(tune.BLOCK_ROWS) * len(tune.QUEUE_CAPACITY)


def test_one_bucket_does_not_take_the_others_to_the_queue_kernel():
    queue = {"block_rows": 64, "scan_rounds": -1, "queue_capacity": 512}
    cache = {"arch": "gfx950", "gfx950": {"small/conn8": queue}}
    _, qmax, out = tune.tuned_batch(cache, [_task(512, 8), _task(4096, 8)])
    assert all(t["scan_rounds"] >= 1 for t in out) and qmax == 2048
    bh, qmax, out = tune.tuned_batch(cache, [_task(512, 8), _task(700, 8)])   # all of them chose it
    assert [t["scan_rounds"] for t in out] == [-1, -1] and (bh, qmax) == (64, 512)
