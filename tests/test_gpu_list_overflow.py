"""Steps in which the lists of some, most or all sweep workgroups overflow (every
workgroup then sets one flag for the resolve): the stateless step and a resident
system, sorted and unsorted.  Against the
oracle: bit-equal, no tolerance."""
import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, say, to_dev
from test_gpu_multi import _orules, cross_roles, step_cfg
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [0.5, 0.7, 1.0])
@pytest.mark.parametrize("which", ["random", "rules"])
def test_many_lists(p, which):
    from paper_1409_7498_amd import binding as B
    N = 30011 if which == "rules" else 120011
    cfg = step_cfg(N, 5)
    rules = cross_roles(p, p) if which == "rules" else [workload.rule_for("step", 1.12, p)]
    multi = which == "rules"
    say("list overflow", which, p)
    dev = to_dev(cfg)
    args = (dev["x"], dev["y"], dev["z"], dev["type"], dev["state"], dev["adj"], cfg["L"])
    o = oracle.System(cfg["L"], *(cfg[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
    if multi:
        code, bonds, st = B.react_step_multi(*args, rules, 6, 1, raise_on_error=False)
        ocode, obonds, ost = oracle.react_step_multi(o, _orules(rules), 6, 1)
    else:
        code, bonds, st = B.react_step(*args, rules[0], 6, 1, raise_on_error=False)
        ocode, obonds, ost = oracle.react_step(o, oracle_rule(rules[0]), 6, 1)
    # pairs per 256 particles against the 32 that a list holds
    assert ost["accepted"] * 256 / N > (18 if p == 0.5 else 24)
    assert code == ocode and np.array_equal(bonds.cpu().numpy(), obonds) and st == ost
    assert np.array_equal(dev["state"].cpu().numpy(), o.state)
    assert np.array_equal(dev["adj"].cpu().numpy(), o.adj)
    o = oracle.System(cfg["L"], *(cfg[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
    run = oracle.run_multi if multi else oracle.run
    ocode, olog, ost = run(o, _orules(rules) if multi else oracle_rule(rules[0]), 6, 1, 3, 0.05)
    assert ocode in (0, B.PR_ECAP)
    for period in (64, 0):
        s = B.System(N, cfg["L"], 4, rules if multi else rules[0], 6, log_cap=4 * N)
        s.set_sort_period(period)
        s.load(cfg)
        s.run(1, 3, 0.05)
        out, log, st = s.read(), s.bonds(), s.stats()
        s.close()
        assert np.array_equal(log, olog[:, :3])
        for k in ("x", "y", "z", "state", "adj"):
            assert np.array_equal(out[k], getattr(o, k)), k
        assert np.array_equal(np.array([[r[f] for f in oracle.ST_NAMES] for r in st]), ost)
