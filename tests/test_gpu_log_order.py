"""The order of the bond log at each read: step by step from the counters, or the
whole log sorted (a step with more rows than LDS holds, steps run twice or out of
order, a log that overflowed, a restored checkpoint), with reads between runs.
Against the oracle's rows in (step, id_A) order: no tolerance."""
import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, random_cfg, say
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


def _canon(rows):
    rows = np.concatenate(rows) if rows else np.empty((0, 3), np.int32)
    return rows[np.lexsort((rows[:, 1], rows[:, 0]))]


@pytest.mark.parametrize("N,p,runs", [
    (3000, 0.2, [(1, 5), (6, 70), (80, 3)]),        # in order, gaps, across a sort
    (3000, 0.2, [(10, 4), (1, 4), (20, 2)]),        # an earlier step after a later one
    (3000, 0.05, [(1, 4), (1, 4), (5, 2)]),         # the same steps twice
    (40000, 1.0, [(1, 2), (3, 2)]),                 # thousands of rows in a step
    (2000, 0.0, [(1, 3)]),                          # none
])
def test_reads_in_order(N, p, runs):
    from paper_1409_7498_amd import binding as B
    cfg = random_cfg(N, workload.box_for(N), "step", 5, frac=0.3)
    rule = workload.rule_for("step", workload.RC, p)
    say("log order", N, p, runs)
    s = B.System(N, cfg["L"], 4, rule, 2, log_cap=4 * N)
    s.load(cfg)
    o = oracle.System(cfg["L"], *(cfg[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
    logs = []
    for first, n in runs:
        s.run(first, n, 0.05)
        code, log, _ = oracle.run(o, oracle_rule(rule), 2, first, n, 0.05)
        assert code in (0, B.PR_ECAP)
        logs.append(log)
        assert np.array_equal(s.bonds(), _canon(logs))
        assert np.array_equal(s.bonds(), _canon(logs))  # again, nothing new
    if p == 1.0:
        assert max(np.bincount(_canon(logs)[:, 0])) > 4096
    # a checkpoint taken here continues in another handle
    t = B.System(N, cfg["L"], 4, rule, 2, log_cap=4 * N)
    t.restore(s.checkpoint())
    for h in (s, t):
        h.run(500, 3, 0.05)
    _, log, _ = oracle.run(o, oracle_rule(rule), 2, 500, 3, 0.05)
    logs.append(log)
    for h in (s, t):
        assert np.array_equal(h.bonds(), _canon(logs))
        h.close()


def test_overflowed_log_keeps_its_rows_in_order():
    import ctypes as C
    from paper_1409_7498_amd import binding as B
    N = 3000
    cfg = random_cfg(N, workload.box_for(N), "step", 5, frac=0.3)
    s = B.System(N, cfg["L"], 4, workload.rule_for("step", workload.RC, 0.2), 2, log_cap=100)
    s.load(cfg)
    s.run(1, 6, 0.05)
    rows, n = np.empty((100, 3), np.int32), C.c_int64(0)
    for _ in range(2):
        code = B.lib.pr_sys_bonds(s._h, rows.ctypes.data_as(C.c_void_p), 100, C.byref(n))
        assert code == B.PR_ECAP and n.value > 100
        assert np.array_equal(rows, _canon([rows]))
    s.close()
