"""Loaded adjacency rows with entries that name no particle, under the MD: they
are no bonds.  Positions and velocities equal those of the same rows without
them, bit for bit, and the rows come back as loaded."""
import numpy as np
import pytest

from gpu_util import say
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,B", [(600, 4), (1300, 2), (257, 5)])
@pytest.mark.parametrize("beyond", [0, 1, 1 << 20, 2 ** 31 - 1])
def test_entries_beyond_the_particles(N, B, beyond):
    from paper_1409_7498_amd import binding
    L = workload.box_for(N)
    got = []
    for fill in (min(N + beyond, 2 ** 31 - 1), -1):
        g = workload.generate(N, L, "step", 17, B=B)
        g["adj"][::3, B - 1] = fill
        g["adj"][4, 0], g["adj"][5, 0] = 5, 4  # and a bond
        for k in "xyz":
            g[k][4], g[k][5] = np.float32(3.0), np.float32(3.75)
        say("md rows", N, B, beyond, fill)
        s = binding.System(N, L, B, workload.rule_for("step", workload.RC, 0.0), 5)
        s.load(g)
        s.set_md(3, 0.0025, 1.0, 1.0, 1.5, 11)
        s.load(g)  # looked at again, the MD being on
        s.set_md(3, 0.0025, 1.0, 1.0, 1.5, 11)
        s.run(1, 6, 0.0)
        out = s.read()
        assert np.array_equal(out["adj"], g["adj"])
        got.append([out[k] for k in "xyz"] + list(s.velocities()))
        s.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
