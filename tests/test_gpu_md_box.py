"""A drift of a box length or more in one MD step: the particle is outside the box
after the single wrap, and the run reports it (no later kernel looks for the
cell of such a position).  The handle takes another configuration afterwards."""
import numpy as np
import pytest

from gpu_util import say
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", ["free", "bonded"])
@pytest.mark.parametrize("period", [64, 0])
def test_leaving_the_box(which, period):
    from paper_1409_7498_amd import binding
    N = 600
    L = workload.box_for(N)
    g = workload.generate(N, L, "step", 7)
    g["adj"][4, 0], g["adj"][5, 0] = 5, 4
    for k in "xyz":
        g[k][4] = g[k][5] = np.float32(3.0)
    g["x"][5] = np.float32(4.3)  # beyond sigma_c: a force
    say("md box", which, period)
    s = binding.System(N, L, 4, workload.rule_for("step", workload.RC, 0.1), 5)
    s.set_sort_period(period)
    s.load(g)
    # free: thermal velocities times dt exceed L; bonded: cold but for one bond
    s.set_md(2, *((100.0, 1.0, 1.0, 1.0) if which == "free" else (0.1, 1.0, 1e8, 0.0)), 11)
    s.run(1, 3, 0.0)
    with pytest.raises(binding.PrError) as e:
        s.read()
    assert e.value.code == binding.PR_EINVAL
    s.load(g)
    s.set_md(2, 0.0025, 1.0, 1.0, 1.0, 11)
    s.run(1, 3, 0.0)
    out = s.read()
    for k in "xyz":
        assert (out[k] >= 0).all() and (out[k] < np.float32(L)).all()
    s.close()
