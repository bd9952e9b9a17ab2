"""A kinetics read-out of a run that ended with a device error (a particle the MD
left outside the box): the error, nothing written, and the counters of the next
configuration right, on sorted storage (staged and not) and unsorted."""
import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, oracle_system, say
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("brick,period", [(0, 64), (6, 64), (0, 0)])
def test_kinetics_after_an_error(brick, period):
    from paper_1409_7498_amd import binding
    N = 3000
    L = workload.box_for(N)
    g = workload.generate(N, L, "step", 7)
    rule = workload.rule_for("step", workload.RC, 0.1)
    say("kinetics error", brick, period)
    s = binding.System(N, L, 4, rule, 5, brick=brick)
    s.set_sort_period(period)
    s.load(g)
    want = oracle.kinetics(oracle_system(g), oracle_rule(rule), nstate=5, nbins=8)
    for _ in range(2):
        for a, b in zip(s.kinetics(5, 8), want):
            assert np.array_equal(a, b)
        s.set_md(2, 100.0, 1.0, 1.0, 1.0, 11)
        s.run(1, 3, 0.0)
        for _ in range(2):
            with pytest.raises(binding.PrError) as e:
                s.kinetics(5, 8)
            assert e.value.code == binding.PR_EINVAL
        s.set_md(0, 1.0, 1.0, 1.0, 1.0, 11)
        s.load(g)
        s.run(1, 1, 0.0)  # sorted again where sorts are on
        s.load(g)
    s.close()
