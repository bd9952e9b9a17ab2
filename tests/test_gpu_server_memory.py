"""What admitted replicas take of the device against the footprints their
admission counted, for requests of more steps than a new system's counter log
holds at first."""
import threading
import time

import pytest

from gpu_util import say
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


def test_replicas_stay_within_their_footprints():
    import torch
    from paper_1409_7498_amd import binding
    reqs, steps = 4, 1025

    def serve(d, count):
        srv = binding.Server(8 << 30, count)
        ts = [srv.submit(dict(d, seed=k + 2), steps, 0.05) for k in range(count)]
        for t in ts:
            assert srv.wait(t, 120.0)[0] == srv.DONE
        srv.close()

    # 50^3 one-cell bricks: 489 closing groups, 16 KB of counters per step
    d = dict(n=65536, L=113.0, B=1, rule=workload.rule_for("step", workload.RC, 0.01),
             kind="step", gen_seed=2, sigma0=0.1, log_cap=65536, brick=1)
    one = binding.footprint(dict(d, seed=1), steps)
    serve(dict(d, n=1000, L=20.0), 1)  # kernels loaded, streams made
    free0, low, stop = torch.cuda.mem_get_info()[0], [1 << 62], threading.Event()

    def watch():
        while not stop.is_set():
            low[0] = min(low[0], torch.cuda.mem_get_info()[0])
            time.sleep(2e-4)

    w = threading.Thread(target=watch)
    w.start()
    serve(d, reqs)
    stop.set()
    w.join()
    taken = free0 - low[0]
    say("server memory: footprint", one, "x", reqs, "=", one * reqs, "taken", taken)
    # beside the replicas: the block maps of this round and the next (16 bytes for
    # each of 160,000 blocks a replica), allocations rounded up to 2 MiB, staging;
    # a log of 1,024 steps first and then one of 2,048 would take 128 MB more
    assert taken <= one * reqs + (64 << 20)
