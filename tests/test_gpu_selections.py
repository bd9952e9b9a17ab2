"""The nearest selection and several rules on every route of the sweep: with
and without fused binning, one or two region cells per staging thread (brick
edges to 4 and above), sorted often and rarely, unsorted, ordinary and crowded
configurations (full cells, full lists, regions beyond the staging), runs that
continue and that jump.  Whole numbers and bit-equal positions: no tolerance."""
import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, random_cfg, say
from test_gpu_multi import _orules, chain_cfg, chain_init_prop, cross_roles, step_cfg
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu
RUNS = [(1, 9, 0.05), (10, 7, 0.05), (40, 5, 0.02)]


def _case(which):
    if which == "near step":
        return workload.generate(3000, workload.box_for(3000), "step", 3), \
            [workload.rule_for("step", workload.RC, 0.3, "nearest")]
    if which == "near chain":
        c = workload.generate(3000, workload.box_for(3000), "chain", 4)
        c["state"][::40] = 2
        return c, [workload.rule_for("chain", workload.RC, 0.6, "nearest")]
    if which == "near crowded":
        return random_cfg(9000, 21.0, "step", 6, frac=0.4), \
            [workload.rule_for("step", workload.RC, 0.2, "nearest")]
    if which == "rules chain":
        return chain_cfg(3000, 11), chain_init_prop(0.4, 0.6)
    if which == "rules cross":
        return step_cfg(3000, 12), cross_roles(0.3, 0.3)
    c = random_cfg(9000, 21.0, "step", 7, frac=0.4)
    c["state"][(c["type"] == 0) & (np.arange(9000) % 3 == 0)] = 1
    return c, cross_roles(0.5, 0.5)


@pytest.mark.parametrize("which", ["near step", "near chain", "near crowded", "rules chain",
                                   "rules cross", "rules crowded"])
def test_every_route(which):
    from paper_1409_7498_amd import binding as B
    cfg, rules = _case(which)
    o = oracle.System(cfg["L"], *(cfg[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
    logs, sts = [], []
    for first, n, sigma in RUNS:
        code, log, st = (oracle.run(o, oracle_rule(rules[0]), 5, first, n, sigma) if len(rules) == 1
                         else oracle.run_multi(o, _orules(rules), 5, first, n, sigma))
        assert code in (0, B.PR_ECAP)
        logs.append(log[:, :3])
        sts.append(st)
    log, st = np.concatenate(logs), np.concatenate(sts)
    assert len(log) > 100
    N, L, Bw = len(cfg["x"]), cfg["L"], cfg["adj"].shape[1]
    for fused, brick, period, graphs in [(1, 0, 64, 1), (1, 2, 4, 1), (1, 6, 64, 0), (0, 0, 5, 1),
                                         (0, 5, 64, 1), (0, 1, 3, 0), (1, 0, 0, 1)]:
        say("route", which, "fused", fused, "brick", brick, "period", period, "graphs", graphs)
        s = B.System(N, L, Bw, rules if len(rules) > 1 else rules[0], 5, log_cap=4 * N,
                     brick=brick)
        s.set_fused_binning(fused)
        s.set_sort_period(period)
        s.set_graphs(graphs)
        s.load(cfg)
        for first, n, sigma in RUNS:
            s.run(first, n, sigma)
            assert s.fused_binning() == bool(fused and period)
        out, got, gst = s.read(), s.bonds(), s.stats()
        s.close()
        assert np.array_equal(got, log), (len(got), len(log))
        for k in ("x", "y", "z", "state", "adj"):
            assert np.array_equal(out[k], getattr(o, k)), k
        assert np.array_equal(np.array([[r[f] for f in oracle.ST_NAMES] for r in gst]), st)
