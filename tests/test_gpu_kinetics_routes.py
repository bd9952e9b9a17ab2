"""The kinetics read-out on each of its routes against the oracle: sorted
storage with the region staged, brick edges above four, unsorted storage, T's
with more partners than a register holds, crowded cells, rows wider than four,
the largest numbers of states and bins, read-outs of changing shape in a row
and after a second load.  Whole numbers: no tolerance."""
import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, random_cfg, say
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,frac,B,brick,period", [
    (5000, 18.1, 0.05, 4, 0, 64), (5000, 18.1, 0.5, 4, 2, 64), (9000, 20.0, 0.3, 6, 4, 64),
    (9000, 20.0, 0.3, 4, 6, 64), (5000, 18.1, 0.2, 4, 0, 0), (700, 5.0, 0.4, 4, 0, 64)])
def test_routes(N, L, frac, B, brick, period):
    from paper_1409_7498_amd import binding
    rule = workload.rule_for("step", workload.RC, 0.4)
    s = None
    for seed in (1, 2):
        cfg = random_cfg(N, L, "step", seed, frac=frac)
        cfg["adj"] = np.full((N, B), -1, np.int32)
        if s is None:
            s = binding.System(N, cfg["L"], B, rule, 3, log_cap=4 * N, brick=brick)
            s.set_sort_period(period)
        s.load(cfg)
        first = 1
        for steps, nstate, nbins in ((0, 5, 7), (3, 64, 256), (2, 1, 1), (2, 5, 0)):
            if steps:
                s.run(first, steps, 0.05)
                first += steps
            say("kinetics route", N, L, frac, B, brick, period, nstate, nbins)
            pop, pairs, hist = s.kinetics(nstate, nbins)
            out = s.read()
            o = oracle.System(cfg["L"], out["x"], out["y"], out["z"], cfg["type"], out["state"],
                              out["adj"])
            want = oracle.kinetics(o, oracle_rule(rule), nstate=nstate, nbins=nbins)
            assert np.array_equal(pop, want[0]) and np.array_equal(pairs, want[1])
            assert np.array_equal(hist, want[2])
    s.close()
