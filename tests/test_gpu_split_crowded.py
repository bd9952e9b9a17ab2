"""Bricks shared among two and four sweep workgroups where nearly all particles
lie in one corner: the corner's bricks in large shares, the others with 0, 1, 2,
3, 5 and a few more particles, so that shares are empty or hold one particle.
The rule's own lines are asserted, so that the cases keep what they are for.
Against the oracle: bit-equal, no tolerance."""
import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, random_cfg, say
from test_gpu_multi import _orules, cross_roles
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


def _cfg(N, L, edge):
    """N particles, all but a few of each other brick in the corner brick."""
    cfg = random_cfg(N, L, "step", N, frac=0.02)
    nb = int(round(L / edge))
    assert nb ** 3 * 6 < N // 4
    rng = np.random.default_rng(N)
    for k in "xyz":
        cfg[k] *= np.float32(0.98 * edge / L)
    at = 0
    for b in range(1, nb ** 3):
        m = (0, 1, 2, 3, 5, 6)[b % 6]
        for k, c in zip("xyz", (b % nb, b // nb % nb, b // nb ** 2)):
            cfg[k][at:at + m] = ((c + rng.uniform(0.1, 0.9, m)) * edge).astype(np.float32)
        at += m
    cfg["state"][(cfg["type"] == 0) & (np.arange(N) % 3 == 0)] = 1
    return cfg


# nc = 12 cells of 2.3, 27 bricks of 4 cells: 27 * 384 = 10,368 particles are four
# workgroups per brick, 27 * 224 = 6,048 two, one fewer whole bricks
@pytest.mark.parametrize("N,shift", [(10368, 2), (10367, 1), (6048, 1), (6047, 0)])
@pytest.mark.parametrize("which", ["random", "nearest", "rules"])
def test_shares(N, shift, which):
    from paper_1409_7498_amd import binding as B
    L, edge, sigma = 27.6, 9.2, 0.05
    cfg = _cfg(N, L, edge)
    rules = (cross_roles(0.005, 0.005) if which == "rules"
             else [workload.rule_for("step", 1.12, 0.005, which)])
    o = oracle.System(cfg["L"], *(cfg[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
    code, olog, ost = (oracle.run_multi(o, _orules(rules), 6, 1, 6, sigma) if which == "rules"
                       else oracle.run(o, oracle_rule(rules[0]), 6, 1, 6, sigma))
    assert code in (0, B.PR_ECAP)
    assert ost[:, oracle.ST_NAMES.index("in_rc")].min() > 0 and len(olog) > 0
    for fused in (1, 0):
        s = B.System(N, cfg["L"], 4, rules if which == "rules" else rules[0], 6, log_cap=4 * N)
        s.set_fused_binning(fused)
        s.set_sort_period(3)
        nc, bs, nbricks = s.geometry()
        assert (nc, bs, nbricks) == (12, 4, 27)
        per = N // nbricks
        assert shift == (0 if per < 224 else 1 if per < 384 else 2)
        say("split crowded", N, which, "fused", fused)
        s.load(cfg)
        s.run(1, 6, sigma)
        out, log, st = s.read(), s.bonds(), s.stats()
        if which != "rules":
            kin = s.kinetics(5, 8)
            for a, b in zip(kin, oracle.kinetics(o, oracle_rule(rules[0]), nstate=5, nbins=8)):
                assert np.array_equal(a, b)
        s.close()
        assert np.array_equal(log, olog[:, :3]), (len(log), len(olog))
        for k in ("x", "y", "z", "state", "adj"):
            assert np.array_equal(out[k], getattr(o, k)), k
        assert np.array_equal(np.array([[r[f] for f in oracle.ST_NAMES] for r in st]), ost)
