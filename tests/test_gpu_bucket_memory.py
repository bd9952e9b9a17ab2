"""The fused-binning buckets are allocated by the first run that can use them, not
by runs with MD or without sorts; that run then takes them up, with the results
of the binning kernel."""
import numpy as np
import pytest

from gpu_util import say
from test_gpu_multi import chain_cfg, chain_init_prop
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", ["random", "nearest", "rules"])
def test_taken_when_used(which):
    import torch
    from paper_1409_7498_amd import binding
    N = 400000
    cfg = chain_cfg(N, 3)
    rules = (chain_init_prop(0.2, 0.2) if which == "rules"
             else workload.rule_for("chain", workload.RC, 0.2, which))
    out = []
    for fused in (1, 0):
        free = []

        def mark():
            torch.cuda.synchronize()
            free.append(torch.cuda.mem_get_info()[0])

        s = binding.System(N, cfg["L"], 2, rules, 5, log_cap=2 * N)
        s.set_fused_binning(fused)
        s.load(cfg)
        s.set_md(2, 0.0025, 1.0, 1.0, 1.0, 11)
        mark()
        s.run(1, 3, 0.0)
        mark()
        s.set_md(0, 0.0025, 1.0, 1.0, 1.0, 11)
        s.set_sort_period(0)
        s.run(4, 3, 0.05)
        mark()
        assert not s.fused_binning()
        s.set_sort_period(64)
        s.run(7, 3, 0.05)
        mark()
        nc, used = s.geometry()[0], [a - b for a, b in zip(free, free[1:])]
        # records and slots of every cell's bucket, overflow records and slots, positions
        buckets = nc ** 3 * (3 * 4 + 2 * 8 * 20) + N * (2 * 20 + 4)
        say("buckets", which, fused, "bytes", buckets, "taken by the runs", used)
        assert s.fused_binning() == bool(fused)
        assert used[0] < buckets // 2 and used[1] < buckets // 2
        if fused:
            assert buckets * 0.9 < used[2]
        got = s.read()
        out.append([got[k] for k in ("x", "y", "z", "state", "adj")] + [s.bonds()])
        s.close()
    assert len(out[0][5]) > 0
    for a, b in zip(*out):
        assert np.array_equal(a, b)
