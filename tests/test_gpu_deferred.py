"""T's that leave the sweep's staged scan: drifted out of the staged region
between sorts, of bricks with too many records to stage, with bucket overflow
(fewer and more entries than lanes share them), in boxes of one, two and more
cells.  Against the oracle: bit-equal, no tolerance."""
import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, random_cfg, say
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("policy", ["random", "nearest"])
@pytest.mark.parametrize("fused", [0, 1])
@pytest.mark.parametrize("N,L,frac,sigma,pile", [
    (6000, 30.0, 0.05, 0.5, 0),    # drift of several cells
    (6000, 16.0, 0.6, 0.05, 0),    # crowded regions
    (3000, 24.0, 0.1, 0.02, 20),   # 20 A's at one point: overflow
    (3000, 24.0, 0.1, 0.02, 9),    # one entry beyond the cell
    (300, 2.5, 0.3, 0.05, 0), (600, 5.0, 0.2, 0.1, 0), (900, 7.0, 0.3, 0.2, 0)])
def test_deferred(N, L, frac, sigma, pile, policy, fused):
    from paper_1409_7498_amd import binding as B
    cfg = random_cfg(N, L, "step", N, frac)
    if pile:
        a = np.flatnonzero(cfg["type"] == 1)[:pile]
        for k in "xyz":
            cfg[k][a] = np.float32(L / 3) + np.arange(pile, dtype=np.float32) * np.float32(1e-3)
    rule = workload.rule_for("step", 1.12, 0.1, policy)
    say("deferred", N, L, frac, sigma, pile, policy, fused)
    s = B.System(N, cfg["L"], 4, rule, 6, log_cap=8 * N)
    s.set_fused_binning(fused)
    s.set_sort_period(10)
    s.load(cfg)
    s.run(1, 20, sigma)
    out, log, st = s.read(), s.bonds(), s.stats()
    s.close()
    o = oracle.System(cfg["L"], *(cfg[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
    code, olog, ost = oracle.run(o, oracle_rule(rule), 6, 1, 20, sigma)
    assert code in (0, B.PR_ECAP)
    assert len(log) > 0 and np.array_equal(log, olog), (len(log), len(olog))
    for k in ("x", "y", "z", "state", "adj"):
        assert np.array_equal(out[k], getattr(o, k)), k
    assert np.array_equal(np.array([[r[f] for f in oracle.ST_NAMES] for r in st]), ost)
