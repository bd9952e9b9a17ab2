"""The overflow list of A records, shared by the eight lanes of a T that scans the
buckets: lists shorter and longer than the lanes and than what a lane has in
flight, with every selection, the binning kernel and fused binning, brick edges
with one and with two region cells per staging thread.  Against the oracle:
bit-equal, no tolerance."""
import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, random_cfg, say
from test_gpu_multi import _orules, cross_roles
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu
CELL = 8  # records a cell's bucket holds


@pytest.mark.parametrize("beyond", [1, 7, 8, 9, 31, 32, 33, 63, 65, 200])
@pytest.mark.parametrize("which", ["random", "nearest", "rules"])
def test_lists(beyond, which):
    from paper_1409_7498_amd import binding as B
    N, L = 2500, 24.0
    cfg = random_cfg(N, L, "step", beyond, 0.0)
    # every A in the middle of one cell (width L / nc), T's around them and elsewhere
    nc = int(L / (2 * 1.12 * (1 + 1 / 1024)))
    rng = np.random.default_rng(beyond)
    a = np.arange(CELL + beyond) * 3
    for k in "xyz":
        cfg[k][a] = (3.5 * L / nc + rng.uniform(-0.2, 0.2, len(a))).astype(np.float32)
        cfg[k][1:1500:3] = (3.5 * L / nc + rng.uniform(-3, 3, 500)).astype(np.float32)
    cfg["type"][a], cfg["state"][a] = 1, 4
    cfg["state"][2::3] = 1
    rules = (cross_roles(0.05, 0.0) if which == "rules"
             else [workload.rule_for("step", 1.12, 0.05, which)])
    o = oracle.System(cfg["L"], *(cfg[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
    code, olog, ost = (oracle.run_multi(o, _orules(rules), 6, 1, 4, 0.0) if which == "rules"
                       else oracle.run(o, oracle_rule(rules[0]), 6, 1, 4, 0.0))
    assert code in (0, B.PR_ECAP)
    in_rc, bonds = (ost[:, oracle.ST_NAMES.index(f)] for f in ("in_rc", "bonds"))
    assert in_rc[0] > len(a)
    assert which == "nearest" or bonds.sum() > 0  # a nearest pair has one draw in twenty
    for fused, brick in [(1, 0), (0, 0), (1, 6), (0, 6)]:
        say("overflow list", beyond, which, "fused", fused, "brick", brick)
        s = B.System(N, cfg["L"], 4, rules if which == "rules" else rules[0], 6, log_cap=4 * N,
                     brick=brick)
        s.set_fused_binning(fused)
        s.load(cfg)
        s.run(1, 4, 0.0)
        assert s.geometry()[0] == nc and s.fused_binning() == bool(fused)
        out, log, st = s.read(), s.bonds(), s.stats()
        s.close()
        assert np.array_equal(log, olog[:, :3]), (len(log), len(olog))
        for k in ("x", "y", "z", "state", "adj"):
            assert np.array_equal(out[k], getattr(o, k)), k
        assert np.array_equal(np.array([[r[f] for f in oracle.ST_NAMES] for r in st]), ost)
