"""Runs on a handle that was loaded before: the graphs captured by earlier runs
are replayed where they hold the same kernels and only there, so that every
run equals the run of a fresh handle (those equal the oracle elsewhere)."""
import numpy as np
import pytest

from gpu_util import say
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu
KEYS = ("x", "y", "z", "state", "adj")


def _fresh(B, N, L, rule, g, runs, prepare=None):
    s = B.System(N, L, g["adj"].shape[1], rule, 9, log_cap=4 * N)
    s.load(g)
    if prepare:
        prepare(s)
    for first, n, sigma in runs:
        s.run(first, n, sigma)
    out = s.read(), s.bonds(), s.stats()
    s.close()
    return out


def _same(a, b):
    for k in KEYS:
        assert np.array_equal(a[0][k], b[0][k]), k
    assert np.array_equal(a[1], b[1]) and a[2] == b[2]


@pytest.mark.parametrize("kind,policy", [("step", "random"), ("chain", "random"),
                                         ("step", "nearest")])
def test_reloaded_runs_equal_fresh_ones(kind, policy):
    import torch
    from paper_1409_7498_amd import binding as B
    N = 6000
    L = workload.box_for(N)
    rule = workload.rule_for(kind, workload.RC, 0.2, policy)
    one, two = (workload.generate(N, L, kind, s) for s in (1, 2))
    s = B.System(N, L, one["adj"].shape[1], rule, 9, log_cap=4 * N)

    def again(g, runs, prepare=None):
        s.load(g)
        if prepare:
            prepare(s)
        for first, n, sigma in runs:
            s.run(first, n, sigma)
            # the caller's own work between the replays
            torch.zeros(1000, device="cuda").add_(1).sum().item()
        return s.read(), s.bonds(), s.stats()

    long_run = [(1, 70, 0.05), (71, 70, 0.05)]
    odd = [(1, 3, 0.05), (4, 64, 0.05), (90, 5, 0.02)]
    period = lambda k: (lambda h: h.set_sort_period(k))
    md = lambda h: h.set_md(3, 0.0025, 1.0, 1.0, 1.0, 4)
    off = lambda h: h.set_md(0)
    for g, runs, prep, want in [
            (one, long_run, None, None), (two, long_run, None, None), (one, odd, None, None),
            (two, odd, None, None), (one, long_run, None, None),
            (one, [(1, 32, 0.05)], period(0), None), (two, [(1, 32, 0.05)], None, period(0)),
            (two, long_run, period(64), None), (one, [(1, 6, 0.0)], md, None),
            (two, [(1, 6, 0.0)], md, None), (two, long_run, off, None)]:
        say("reload", kind, policy, runs)
        _same(again(g, runs, prep), _fresh(B, N, L, rule, g, runs, want or prep))
    s.close()
