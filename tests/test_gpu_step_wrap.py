"""Runs whose step numbers pass 2^32: the fused binning's rotation by the step
number mod 3 does not go on there, so such runs bin every step; the runs before
and after them fuse.  Against the oracle: bit-equal, no tolerance (the log is
ordered by the unsigned step number)."""
import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, random_cfg, say
from test_gpu_multi import _orules, cross_roles
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu
END = 1 << 32


def _canon(rows):
    return rows[np.lexsort((rows[:, 1], rows[:, 0].astype(np.uint32)))]


@pytest.mark.parametrize("which", ["random", "nearest", "rules"])
@pytest.mark.parametrize("runs", [
    [(END - 20, 10), (END - 10, 15), (5, 9)],       # fused, across, fused again (after a sort)
    [(END - 12, 10), (END - 2, 1), (END - 1, 1), (0, 3)],  # one by one
    [(END - 3, 1), (END - 2, 30)]])
def test_across(which, runs):
    from paper_1409_7498_amd import binding as B
    N, L = 3000, 16.0
    cfg = random_cfg(N, L, "step", 9, frac=0.1)
    cfg["state"][(cfg["type"] == 0) & (np.arange(N) % 3 == 0)] = 1
    rules = (cross_roles(0.05, 0.05) if which == "rules"
             else [workload.rule_for("step", 1.12, 0.05, which)])
    o = oracle.System(cfg["L"], *(cfg[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
    logs, sts = [], []
    for f, n in runs:
        run = oracle.run_multi if which == "rules" else oracle.run
        code, log, st = run(o, _orules(rules) if which == "rules" else oracle_rule(rules[0]), 6, f,
                            n, 0.05)
        assert code in (0, B.PR_ECAP)
        logs.append(log[:, :3])
        sts.append(st)
    want, st = np.concatenate(logs), np.concatenate(sts)
    for graphs in (1, 0):
        say("step wrap", which, runs, "graphs", graphs)
        s = B.System(N, cfg["L"], 4, rules if which == "rules" else rules[0], 6, log_cap=4 * N)
        s.set_sort_period(8)
        s.set_graphs(graphs)
        s.load(cfg)
        for f, n in runs:
            s.run(f, n, 0.05)
            if f + n + 1 >= END:
                assert not s.fused_binning()
            elif n >= 8:  # a sort came due
                assert s.fused_binning()
        out, got, gst = s.read(), s.bonds(), s.stats()
        s.close()
        assert len(want) > 0 and np.array_equal(got, _canon(want)), (len(got), len(want))
        for k in ("x", "y", "z", "state", "adj"):
            assert np.array_equal(out[k], getattr(o, k)), k
        assert np.array_equal(np.array([[r[f] for f in oracle.ST_NAMES] for r in gst]), st)


def test_batch_across():
    from paper_1409_7498_amd import binding as B
    reps = [dict(n=n, L=workload.box_for(n), B=4, rule=workload.rule_for("step", 1.12, 0.05),
                 seed=n, kind="step", gen_seed=n + 1, sigma0=0.1, log_cap=4 * n)
            for n in (900, 2500, 4000)]
    runs = [(END - 80, 70), (END - 10, 80), (70, 66)]
    b = B.Batch(reps)
    for f, n in runs:
        say("step wrap batch", f, n)
        b.run(f, n, 0.05)
    got = [(b.bonds(r), b.read(r)) for r in range(len(reps))]
    b.close()
    for r, (log, out) in zip(reps, got):
        g = workload.generate(r["n"], r["L"], "step", r["gen_seed"])
        o = oracle.System(g["L"], *(g[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
        logs = [oracle.run(o, oracle_rule(r["rule"]), r["seed"], f, n, 0.05)[1] for f, n in runs]
        assert np.array_equal(log, _canon(np.concatenate(logs)))
        for k in ("x", "y", "z", "state", "adj"):
            assert np.array_equal(out[k], getattr(o, k)), k
