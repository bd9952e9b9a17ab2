"""The MD between reaction steps over the bonded particles alone: sizes at the
edges of a wavefront and a workgroup, one, odd and even sub-steps, every row
width class, and loaded rows that name a particle whose own row is empty.
Every value equals the oracle's (FP32 in one order: no tolerance)."""
import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, say
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


def _pairs(g, L, count, both):
    """Bonds between disjoint pairs about 1.25 apart (beyond sigma_c: each
    feels a force from the first sub-step)."""
    x = np.stack([g["x"], g["y"], g["z"]], 1).astype(np.float64)
    d = x[:, None] - x[None]
    d -= L * np.round(d / L)
    r = np.abs(np.sqrt((d ** 2).sum(-1)) - 1.25) + 1e9 * np.eye(len(x))
    used = set()
    for k in np.argsort(r, axis=None):
        i, j = divmod(int(k), len(x))
        if i in used or j in used:
            continue
        g["adj"][i][0] = j
        if both:
            g["adj"][j][0] = i
        used |= {i, j}
        if len(used) >= 2 * count:
            return


@pytest.mark.parametrize("N,kind,B,theta,loaded", [
    (128, "step", 4, 1, "none"), (257, "step", 4, 2, "both"), (255, "chain", 2, 3, "both"),
    (512, "step", 5, 5, "one-sided"), (1000, "step", 4, 4, "one-sided"),
    (769, "step", 7, 1, "both")])
def test_bonded_particles_alone(N, kind, B, theta, loaded):
    from paper_1409_7498_amd import binding
    L = workload.box_for(N)
    g = workload.generate(N, L, kind, 31 + N, B=B)
    if loaded != "none":
        _pairs(g, L, N // 8, loaded == "both")
    rule = workload.rule_for(kind, workload.RC, 0.3)
    say("md compact", N, kind, B, theta, loaded)
    s = binding.System(N, L, B, rule, 5, log_cap=4 * N)
    s.set_sort_period(3)
    s.load(g)
    s.set_md(theta, 0.0025, 1.0, 1.0, 1.5, 11)
    s.run(1, 8, 0.0)
    first = s.read()
    v = s.velocities()
    log = s.bonds()
    o = oracle.System(L, *(g[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
    md = oracle.MD(N, seed=11, temp=1.5)
    code, olog, _ = oracle.run_md(o, md, oracle_rule(rule), 5, 1, 8, theta)
    # a loaded bond takes a row entry and no valence: a row may overflow (ECAP)
    assert code in (0, binding.PR_ECAP) and np.array_equal(log, olog)
    for k in ("x", "y", "z", "state", "adj"):
        assert np.array_equal(first[k], getattr(o, k)), k
    for a, b in zip(v, (md.vx, md.vy, md.vz)):
        assert np.array_equal(a, b)
    # the same configuration loaded again, MD still on: new velocities, the
    # rows looked at again
    s.load(g)
    s.set_md(theta, 0.0025, 1.0, 1.0, 1.5, 11)
    s.run(1, 8, 0.0)
    again = s.read()
    for k in ("x", "y", "z", "state", "adj"):
        assert np.array_equal(first[k], again[k]), k
    s.close()
