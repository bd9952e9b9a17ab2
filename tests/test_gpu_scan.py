"""The sweep's scan by integer positions: cutoffs that give its units their
smallest, middle and finest scale and the scale where no integer test applies;
pairs one rounding inside and outside the cutoff, in one axis, in all three and
across the box edge; full blocks and T's with too many candidates for its
registers.  Against the oracle: bit-equal, no tolerance."""
import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, random_cfg, say
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


def run_both(cfg, rule, jitter=0.0, steps=3):
    from paper_1409_7498_amd import binding as B
    n = len(cfg["x"])
    s = B.System(n, cfg["L"], cfg["adj"].shape[1], rule, 6, log_cap=4 * n)
    s.set_sort_period(2)
    s.load(cfg)
    s.run(1, steps, jitter)
    out, log, st = s.read(), s.bonds(), s.stats()
    s.close()
    o = oracle.System(cfg["L"], *(cfg[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
    code, olog, ost = oracle.run(o, oracle_rule(rule), 6, 1, steps, jitter)
    assert code == 0
    assert np.array_equal(log, olog), (len(log), len(olog))
    for k in ("x", "y", "z", "state", "adj"):
        assert np.array_equal(out[k], getattr(o, k)), k
    assert np.array_equal(np.array([[r[f] for f in oracle.ST_NAMES] for r in st]), ost)
    return ost


# rc / L from just below a half (units of L / 2^16) to 1/4096 (L / 2^22)
@pytest.mark.parametrize("policy", ["random", "nearest"])
@pytest.mark.parametrize("rel,scale", [(0.499, 1.0), (0.0626, 1.0), (0.0624, 3e-12), (0.02, 7.0), (0.003, 1.0),
                                       (1.0 / 1024, 1e15), (1.0 / 4096, 1.0), (0.05, 1e-17)])
def test_pairs_at_the_cutoff(rel, scale, policy):
    L = float(np.float32(64.0 * scale))
    rc = float(np.float32(rel * L))
    rng = np.random.default_rng(5)
    n = 1200 if rel < 0.1 else 60
    cfg = random_cfg(2 * n, L, "step", 3)
    f = np.float32
    a = np.stack([cfg[k][:n] for k in "xyz"])
    a[:, ::7] = np.where(rng.random(a[:, ::7].shape) < 0.5, f(0), np.nextafter(f(L), f(0)))
    u = rng.normal(size=(3, n))
    u[:, ::3] = np.eye(3)[rng.integers(0, 3, n)].T[:, ::3] * rng.choice([-1, 1], n)[::3]
    u /= np.linalg.norm(u, axis=0)
    # within a few roundings of a position of the cutoff, both sides
    b = a.astype(np.float64) + u * rc + rng.integers(-3, 4, (3, n)) * float(np.spacing(f(L))) * 0.5
    b = np.mod(b, L).astype(f)
    b[b >= f(L)] = 0
    for i, k in enumerate("xyz"):
        cfg[k][:n], cfg[k][n:] = a[i], b[i]
    cfg["type"][:n], cfg["type"][n:] = 0, 1
    cfg["state"][:n], cfg["state"][n:] = 2, 4
    rule = workload.rule_for("step", rc, 0.5, policy)
    say("scan cutoff", rel, scale, policy)
    ost = run_both(cfg, rule)
    if scale > 1e-15:
        assert ost.sum() > 0


@pytest.mark.parametrize("policy", ["random", "nearest"])
@pytest.mark.parametrize("per_cell", [8, 7, 5, 4, 3])
def test_crowded_blocks(per_cell, policy):
    # 12^3 cells of width 2.5; A's in one 3x3x3 group of them only, per_cell in each
    L, w, rng = 30.0, 2.5, np.random.default_rng(per_cell)
    corner = np.array([(i, j, k) for i in range(4, 7) for j in range(4, 7) for k in range(4, 7)])
    pos = (np.repeat(corner, per_cell, axis=0) + rng.uniform(0.02, 0.98, (27 * per_cell, 3))) * w
    n_a, n = len(pos), 4000
    cfg = random_cfg(n, L, "step", 8)
    for i, k in enumerate("xyz"):
        cfg[k][:n_a] = pos[:, i]
        cfg[k][n_a:] = cfg[k][n_a:] * np.float32(0.25) + np.float32(10.0)
    cfg["type"] = (np.arange(n) < n_a).astype(np.int32)
    cfg["state"] = np.where(cfg["type"] == 1, 4, 2).astype(np.int32)
    rule = workload.rule_for("step", 1.2, 0.05, policy)
    say("scan crowded", per_cell, policy)
    assert run_both(cfg, rule).sum() > 0
