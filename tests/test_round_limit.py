"""The pixel backward's bound on the staged entries that a pixel composited
(msplat::round_limit, compiled for the host from the header the kernels use):
an entry of a round counts exactly when its list position lies below the
pixel's last one, whatever the list's length (up to 2^30 pairs are accepted)."""
import os
import shutil
import subprocess

import pytest

from paper_2411_12788_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which(B.HIPCC) is None and not os.path.exists(B.HIPCC), reason="hipcc not available")
def test_round_limit_of_long_lists(tmp_path):
    exe = str(tmp_path / "round_limit_host")
    subprocess.check_call([B.HIPCC, "-O2", "-std=c++17", "-w", "-I", os.path.join(ROOT, "include"), "-I", B.CSRC,
                           os.path.join(ROOT, "tests", "round_limit_host.cpp"), "-o", exe])
    cases = [(last, first, batch) for batch in (192, 256)
             for last in (0, 1, 63, 64, 191, 192, 193, 256, 257, 1 << 20, (1 << 28) - 1, 1 << 28, (1 << 28) + 5,
                          (1 << 29) + 17, 1 << 30)
             for first in (0, 1, 64, 192, 256, (1 << 20) - 3, (1 << 28) - 64, 1 << 28, (1 << 30) - 100)]
    out = subprocess.run([exe], input="\n".join("%d %d %d" % c for c in cases), capture_output=True, text=True,
                         check=True)
    got = [int(x) for x in out.stdout.split()]
    assert len(got) == len(cases)
    for (last, first, batch), lim in zip(cases, got):
        for k in {0, 1, batch // 2, batch - 1, max(0, min(batch - 1, last - first)),
                  max(0, min(batch - 1, last - first - 1))}:
            assert (16 * k < lim) == (first + k < last), (last, first, batch, k, lim)
