"""A batch's descriptions are validated before anything is sized by their number,
and before any device call (CPU)."""
import ctypes
import resource

import pytest

from paper_1409_7498_amd import binding as b
from paper_1409_7498_amd import workload


def _desc(**kw):
    d = dict(n=1000, L=20.0, B=4, rule=workload.rule_for("step", workload.RC, 0.1), seed=1,
             kind="step", gen_seed=2, sigma0=0.1)
    d.update(kw)
    return b.replica_desc(d)


@pytest.mark.parametrize("bad,text", [(dict(n=0), b"n=0"), (dict(B=0), b"B=0"),
                                      (dict(brick=7), b"brick=7"), (dict(L=2.0), b"2*rc")])
def test_first_bad_replica_of_many(bad, text):
    arr = (b.ReplicaDesc * 3)(_desc(), _desc(**bad), _desc())
    h = ctypes.c_void_p()
    before = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss
    # a count far beyond the array: the bad description ends the walk
    code = b.lib.pr_batch_create(ctypes.byref(h), arr, 2 ** 31 - 1, None)
    grown = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss - before  # KiB
    assert code == b.PR_EINVAL and not h
    assert b"replica 1" in b.lib.pr_last_error() and text in b.lib.pr_last_error()
    assert grown < 1 << 20
