"""Runs that jump in the step number, with empty runs and a longer sort period in
between: the fused binning's records belong to the step they were binned for.
Against the oracle: bit-equal, no tolerance."""
import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, random_cfg, say
from test_gpu_multi import _orules, cross_roles
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", ["random", "nearest", "rules"])
@pytest.mark.parametrize("empty", [(100, 0.05), (11, 0.02), (11, 0.05)])
def test_empty_run_then_a_longer_period(which, empty):
    from paper_1409_7498_amd import binding as B
    N, L = 3000, 16.0
    cfg = random_cfg(N, L, "step", 9, frac=0.1)
    cfg["state"][(cfg["type"] == 0) & (np.arange(N) % 3 == 0)] = 1
    rules = (cross_roles(0.1, 0.1) if which == "rules"
             else [workload.rule_for("step", 1.12, 0.1, which)])
    first, sigma = empty
    say("run jumps", which, empty)
    s = B.System(N, cfg["L"], 4, rules if which == "rules" else rules[0], 6, log_cap=4 * N)
    s.load(cfg)
    o = oracle.System(cfg["L"], *(cfg[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
    logs = []
    for f, n, sg in [(1, 10, 0.05), (first, 5, sigma)]:
        run = oracle.run_multi if which == "rules" else oracle.run
        code, log, _ = run(o, _orules(rules) if which == "rules" else oracle_rule(rules[0]), 6, f,
                           n, sg)
        assert code in (0, B.PR_ECAP)
        logs.append(log[:, :3])
    s.run(1, 10, 0.05)
    s.run(first, 0, sigma)
    s.set_sort_period(1000)
    s.run(first, 5, sigma)
    out, got = s.read(), s.bonds()
    s.close()
    want = np.concatenate(logs)
    assert len(logs[1]) > 0 and np.array_equal(got, want), (len(got), len(want))
    for k in ("x", "y", "z", "state", "adj"):
        assert np.array_equal(out[k], getattr(o, k)), k
