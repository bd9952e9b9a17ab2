"""The nearest sweep that merges a staged A's pairs in LDS (whole bricks): many
T's per A and several passes per brick, on both sides of the brick count where
bricks stop being shared.  Against the same run on unsorted storage, whose sweep
takes every pair by itself: bit-equal, no tolerance."""
import numpy as np
import pytest

from gpu_util import say
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("exclude", [0, 1])
@pytest.mark.parametrize("fused", [0, 1])
@pytest.mark.parametrize("N,rho", [(330000, 0.85), (400000, 0.85), (900000, 2.0)])
def test_merged_pairs(N, rho, fused, exclude):
    from paper_1409_7498_amd import binding as B
    L = float(np.float32((N / rho) ** (1.0 / 3.0)))
    cfg = workload.generate(N, L, "step", N)
    rule = workload.rule_for("step", workload.RC, 0.3, "nearest")
    rule["exclude_bonded"] = exclude
    got = []
    for period in (4, 0):
        s = B.System(N, cfg["L"], 4, rule, 6, log_cap=2 * N)
        s.set_fused_binning(fused)
        s.set_sort_period(period)
        s.load(cfg)
        s.run(1, 6, 0.05)
        say("near merge", N, rho, fused, exclude, s.geometry(), "period", period)
        out = s.read()
        got.append([out[k] for k in ("x", "y", "z", "state", "adj")] + [s.bonds(), s.stats()])
        s.close()
    assert len(got[0][5]) > 0 and got[0][6] == got[1][6]
    for a, b in zip(got[0][:6], got[1][:6]):
        assert np.array_equal(a, b)
