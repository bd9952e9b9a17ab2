"""The first sort after a load and the read-out around the size where they
move particles as records: rows of two, four and five, velocities, several
rules' role masks.  Against the same run on storage that is never sorted (which
equals the oracle in the other tests), element by element."""
import numpy as np
import pytest

from gpu_util import random_cfg, say
from test_gpu_multi import cross_roles
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [262143, 262144, 262401])
@pytest.mark.parametrize("what", ["step 4", "chain 2", "step 5", "md", "rules"])
def test_first_sort_and_read_out(N, what):
    from paper_1409_7498_amd import binding as B
    kind = "chain" if what.startswith("chain") else "step"
    cfg = random_cfg(N, workload.box_for(N), kind, 17 + N)
    if what == "step 5":
        cfg["adj"] = np.full((N, 5), -1, np.int32)
    rule = cross_roles(0.2, 0.2) if what == "rules" else workload.rule_for(kind, workload.RC, 0.2)
    got = []
    for period in (64, 0):
        say("fresh sort", N, what, "period", period)
        s = B.System(N, cfg["L"], cfg["adj"].shape[1], rule, 3, log_cap=2 * N)
        s.set_sort_period(period)
        s.load(cfg)
        if what == "md":
            s.set_md(2, 0.0025, 1.0, 1.0, 1.0, 5)
        s.run(1, 3, 0.0 if what == "md" else 0.05)
        out = s.read()
        got.append([out[k] for k in ("x", "y", "z", "state", "adj")] + [s.bonds()] +
                   (list(s.velocities()) if what == "md" else []))
        s.close()
    assert len(got[0][5]) > 0
    for a, b in zip(*got):
        assert np.array_equal(a, b)
