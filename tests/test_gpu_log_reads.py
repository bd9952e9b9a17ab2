"""Reads of the bond log while a run goes on: each orders only the steps since the
read before it, so its work does not grow with the run; reads with a capacity
below the rows, of logs that overflow, of more new steps than are ordered one by
one, of steps with no row; after runs out of order.  Against the oracle's rows in
(step, id_A) order: no tolerance."""
import ctypes as C

import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, random_cfg, say
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


def _setup(N, p, log_cap, frac=0.3):
    from paper_1409_7498_amd import binding as B
    cfg = random_cfg(N, workload.box_for(N), "step", 5, frac=frac)
    rule = workload.rule_for("step", workload.RC, p)
    s = B.System(N, cfg["L"], 4, rule, 2, log_cap=log_cap)
    s.load(cfg)
    o = oracle.System(cfg["L"], *(cfg[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
    return s, o, rule


def _read(s, cap):
    """(code, rows written, total); what the call leaves unwritten stays -7."""
    from paper_1409_7498_amd import binding as B
    rows, n = np.full((cap + 3, 3), -7, np.int32), C.c_int64(-1)
    code = B.lib.pr_sys_bonds(s._h, rows.ctypes.data_as(C.c_void_p), cap, C.byref(n))
    m = min(cap, n.value)
    assert (rows[m:] == -7).all()
    return code, rows[:m], n.value


def _canon(rows):
    return rows[np.lexsort((rows[:, 1], rows[:, 0]))]


@pytest.mark.parametrize("p", [0.2, 0.002])
def test_short_reads_between_runs(p):
    s, o, rule = _setup(3000, p, 12000)
    log = np.empty((0, 3), np.int32)
    step = 1
    # runs of several lengths, one longer than the steps ordered one by one
    for n, cap in [(1, 1), (3, 5), (64, 40), (70, 12000), (1, 2), (4200, 3), (5, 12000), (2, 0),
                   (1, 12000), (300, 100), (7, 12000)]:
        say("log reads", p, "step", step, "+", n, "cap", cap)
        s.run(step, n, 0.05)
        code, more, _ = oracle.run(o, oracle_rule(rule), 2, step, n, 0.05)
        assert code == 0
        log = np.concatenate([log, more])
        for _ in range(2):
            code, rows, total = _read(s, cap)
            assert code == 0 and total == len(log)
            assert np.array_equal(rows, _canon(log)[:cap])
        step += n
    s.run(5, 2, 0.05)  # earlier steps again: sorted whole from here on
    log = np.concatenate([log, oracle.run(o, oracle_rule(rule), 2, 5, 2, 0.05)[1]])
    for cap in (4, 12000):
        code, rows, total = _read(s, cap)
        assert code == 0 and total == len(log) and np.array_equal(rows, _canon(log)[:cap])
    s.close()


def test_overflowed_log_holds_rows_of_the_run():
    from paper_1409_7498_amd import binding as B
    s, o, rule = _setup(3000, 0.2, 400)
    log, got = np.empty((0, 3), np.int32), []
    for step in range(1, 7):
        s.run(step, 1, 0.05)
        log = np.concatenate([log, oracle.run(o, oracle_rule(rule), 2, step, 1, 0.05)[1]])
        for _ in range(2):
            code, rows, total = _read(s, 400)
            assert total == len(log) and code == (B.PR_ECAP if total > 400 else 0)
            got.append((step, rows))
    assert len(log) > 450
    for step, rows in got:
        want = _canon(log[log[:, 0] <= step])
        if len(want) <= 400:
            assert np.array_equal(rows, want)
            continue
        # every step before the one that overflowed, then rows of that step, once each
        assert len(rows) == 400 and np.array_equal(rows, _canon(rows))
        first = rows[-1, 0]
        assert np.array_equal(rows[rows[:, 0] < first], want[want[:, 0] < first])
        of_log = {tuple(r) for r in want.tolist()}
        assert all(tuple(r) in of_log for r in rows.tolist())
        assert len({tuple(r) for r in rows.tolist()}) == 400
    over = [r for k, r in got if len(log[log[:, 0] <= k]) > 400]
    for r in over:
        assert np.array_equal(r, over[0])
    s.close()


def test_a_read_does_not_grow_with_the_run():
    import time
    s, _, _ = _setup(60000, 1e-5, 240000, frac=0.05)
    step, t = 1, {}
    for upto in (2000, 100000):
        s.run(step, upto - step, 0.05)
        _read(s, 240000)
        ts = []
        for k in range(20):
            s.run(upto + k, 1, 0.05)
            _read(s, 0)  # waits for the step
            a = time.perf_counter()
            _read(s, 16)
            ts.append(time.perf_counter() - a)
        step = upto + 20
        t[upto] = min(ts)
    say("log read us", {k: round(v * 1e6, 1) for k, v in t.items()})
    assert t[100000] < 3.0 * t[2000]
    s.close()
