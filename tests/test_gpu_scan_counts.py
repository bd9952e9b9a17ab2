"""The sweep's scan at the cutoff, counter by counter: the oracle's in-range pairs
are what the configurations are made for (some pairs just inside the cutoff, some
just outside), and the library finds exactly these, for every scale of the scan,
with every selection.  Bit-equal, no tolerance."""
import numpy as np
import pytest

import oracle
from gpu_util import oracle_rule, random_cfg, say
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("policy", ["random", "nearest"])
@pytest.mark.parametrize("fused", [1, 0])
@pytest.mark.parametrize("rel", [0.2, 0.0626, 0.0624, 0.02, 0.0079, 0.0039, 0.00196, 1.0 / 1024,
                                 1.0 / 4096])
def test_pairs_inside_and_outside(rel, fused, policy):
    from paper_1409_7498_amd import binding as B
    f, L = np.float32, 64.0
    rc = float(f(rel * L))
    n = 60 if rel > 0.1 else 1200
    rng = np.random.default_rng(int(1 / rel))
    cfg = random_cfg(2 * n, L, "step", 3)
    a = np.stack([cfg[k][:n] for k in "xyz"])
    a[:, ::5] = np.where(rng.random(a[:, ::5].shape) < 0.5, f(0), np.nextafter(f(L), f(0)))
    u = rng.normal(size=(3, n))
    u /= np.linalg.norm(u, axis=0)
    # pair i at rc (1 -+ 2e-4), inside and outside in turn, beyond any rounding
    # of positions down to L / 4096 (2^-18 of the cutoff)
    side = np.where(np.arange(n) % 2 == 0, 1 - 2e-4, 1 + 2e-4)
    b = np.mod(a.astype(np.float64) + u * rc * side, L).astype(f)
    b[b >= f(L)] = 0
    for i, k in enumerate("xyz"):
        cfg[k][:n], cfg[k][n:] = a[i], b[i]
    cfg["type"][:n], cfg["type"][n:] = 0, 1
    cfg["state"][:n], cfg["state"][n:] = 2, 4
    rule = workload.rule_for("step", rc, 0.5, policy)
    o = oracle.System(cfg["L"], *(cfg[k].copy() for k in ("x", "y", "z", "type", "state", "adj")))
    code, olog, ost = oracle.run(o, oracle_rule(rule), 6, 1, 3, 0.0)
    assert code == 0
    in_rc, bonds = (ost[:, oracle.ST_NAMES.index(q)] for q in ("in_rc", "bonds"))
    # the pairs lie where they were made to
    d = a.astype(np.float64) - b
    r = np.sqrt(((d - L * np.round(d / L)) ** 2).sum(0))
    assert np.array_equal(r < rc, np.arange(n) % 2 == 0)
    assert in_rc[0] >= n // 2 and bonds.sum() > 0
    say("scan counts", rel, policy, "fused", fused, "in range", in_rc[0], "of", n)
    s = B.System(2 * n, cfg["L"], 4, rule, 6, log_cap=8 * n)
    s.set_fused_binning(fused)
    s.load(cfg)
    s.run(1, 3, 0.0)
    log, st = s.bonds(), s.stats()
    s.close()
    assert np.array_equal(np.array([[r[q] for q in oracle.ST_NAMES] for r in st]), ost)
    assert np.array_equal(log, olog)
