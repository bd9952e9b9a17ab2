"""The stateless step's counters beyond 32 bits: every pair of 65,536 T's and
70,000 A's is in range, and the T's are those of the sweep workgroups that one
wavefront of the last kernel adds up.  The count is known without the oracle."""
import numpy as np
import pytest

from gpu_util import say, to_dev
from paper_1409_7498_amd import workload

pytestmark = pytest.mark.gpu


def test_pairs_beyond_32_bits():
    from paper_1409_7498_amd import binding as B
    n, L, n_a = 1 << 20, 100.0, 70000
    i = np.arange(n)
    t = (i // 256) % 1024 < 64
    a = np.flatnonzero(~t)[:n_a]
    rng = np.random.default_rng(3)
    cfg = dict(L=L, type=np.full(n, 2, np.int32), state=np.full(n, 2, np.int32),
               adj=np.full((n, 2), -1, np.int32))
    for k in "xyz":
        cfg[k] = (50.0 + rng.uniform(-0.1, 0.1, n)).astype(np.float32)
    cfg["type"][t], cfg["type"][a], cfg["state"][a] = 0, 1, 4
    dev = to_dev(cfg)
    say("pairs beyond 32 bits")
    code, bonds, st = B.react_step(dev["x"], dev["y"], dev["z"], dev["type"], dev["state"],
                                   dev["adj"], L, workload.rule_for("step", 1.12, 0.0), 1, 1)
    assert t.sum() * n_a > 1 << 32
    assert code == 0 and len(bonds) == 0
    assert (st["a_elig"], st["t_elig"], st["in_rc"]) == (n_a, t.sum(), int(t.sum()) * n_a)
