"""Bricks shared among several sweep workgroups (small single systems): shares
of a brick that are empty, one particle, uneven; all particles in one brick;
brick counts on both sides of the rule's lines.  Against the oracle (small) or
the same run on unsorted storage: bit-equal, no tolerance."""
import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, random_cfg, say
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,cluster", [(1023, 12.0, 0), (1025, 12.0, 0), (2049, 13.5, 0),
                                         (3001, 24.0, 6.0), (600, 40.0, 3.0), (5000, 18.0, 0)])
@pytest.mark.parametrize("policy", ["random", "nearest"])
@pytest.mark.parametrize("fused", [0, 1])
def test_shares_of_a_brick(N, L, cluster, policy, fused):
    from paper_1409_7498_amd import binding as B
    cfg = random_cfg(N, L, "step", N, frac=0.1)
    if cluster:  # all but a few particles in one corner: the other bricks nearly empty
        for k in ("x", "y", "z"):
            cfg[k][N // 50:] *= np.float32(cluster / L)
    rule = workload.rule_for("step", workload.RC, 0.2, policy)
    say("split", N, L, cluster, policy, fused)
    s = B.System(N, cfg["L"], 4, rule, 6, log_cap=4 * N)
    s.set_fused_binning(fused)
    s.set_sort_period(5)
    s.load(cfg)
    s.run(1, 12, 0.05)
    out, log, st = s.read(), s.bonds(), s.stats()
    kin = s.kinetics(5, 8)
    s.close()
    o = oracle.System(cfg["L"], *(cfg[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
    code, olog, ost = oracle.run(o, oracle_rule(rule), 6, 1, 12, 0.05)
    assert code in (0, B.PR_ECAP)
    assert np.array_equal(log, olog), (len(log), len(olog))
    for k in ("x", "y", "z", "state", "adj"):
        assert np.array_equal(out[k], getattr(o, k)), k
    assert np.array_equal(np.array([[r[f] for f in oracle.ST_NAMES] for r in st]), ost)
    want = oracle.kinetics(o, oracle_rule(rule), nstate=5, nbins=8)
    for a, b in zip(kin, want):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("N", [32000, 64000, 130000, 290000, 400000])
def test_brick_counts_around_the_lines(N):
    from paper_1409_7498_amd import binding as B
    cfg = workload.generate(N, workload.box_for(N), "step", N)
    rule = workload.rule_for("step", workload.RC, 0.3)
    got = []
    for period in (64, 0):
        s = B.System(N, cfg["L"], 4, rule, 6, log_cap=2 * N)
        s.set_sort_period(period)
        s.load(cfg)
        s.run(1, 5, 0.05)
        say("split lines", N, s.geometry(), "period", period)
        out = s.read()
        got.append([out[k] for k in ("x", "y", "z", "state", "adj")] + [s.bonds(), s.stats()])
        s.close()
    assert len(got[0][5]) > 0 and got[0][6] == got[1][6]
    for a, b in zip(got[0][:6], got[1][:6]):
        assert np.array_equal(a, b)
