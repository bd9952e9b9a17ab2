"""The units and threshold of the sweep's integer scan on the host: no pair that the
FP32 test accepts may fall at the integer one, for boxes and cutoffs over the
whole range of units (L / 2^16 to L / 2^22) and of FP32 sizes; and the threshold
is tight enough to be of use."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("scan") / "check")
    subprocess.run([shutil.which("g++"), "-O2", "-std=c++17", "-ffp-contract=off", "-o", exe,
                    os.path.join(HERE, "scan_units_check.cpp")], check=True)
    return exe


RATIOS = [0.4999, 0.25, 0.0626, 0.0624, 0.0313, 0.0312, 0.0157, 0.0156, 0.0079, 0.0078, 0.004,
          0.0039, 0.00196, 0.00195, 0.00098, 0.00097, 1.0 / 4096, 1e-4, 1e-5]


@pytest.mark.parametrize("L", [1.0, 105.6, 64.0, 167.7, 1.7e-9, 3e15])
def test_no_accepted_pair_is_dropped(check, L):
    for rel in RATIOS:
        rc = rel * L
        out = subprocess.run([check, repr(L), repr(rc), "200000"], check=True,
                             capture_output=True, text=True).stdout.split()
        tries, accepted, candidates, lost = map(int, out)
        assert lost == 0, (L, rel, out)
        # pairs on both sides of the cutoff were tried
        assert 0.2 * tries < accepted < 0.8 * tries, (L, rel, out)


def test_far_pairs_are_no_candidates(check):
    # with the cutoff 4096 units or more, a tenth of a per cent beyond it suffices
    src = os.path.join(HERE, "..", "paper_1409_7498_amd", "csrc", "scan_units.hpp")
    prog = ('#include "%s"\n#include <cstdio>\nint main() { for (double rel : {0.4999, 0.0626, 0.02, '
            '0.002, 0.00098}) { const pr::ScanUnits u = pr::scan_units(100.0f, (float)(100.0 * rel)); '
            'std::printf("%%.9g\\n", std::sqrt((double)u.thr) / (rel * 100.0 * u.scale)); } }' % src)
    exe = check + "_ratio"
    subprocess.run([shutil.which("g++"), "-std=c++17", "-x", "c++", "-", "-o", exe], input=prog,
                   text=True, check=True)
    for line in subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split():
        assert 1.0 < float(line) < 1.002
