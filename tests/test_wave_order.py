"""LDS that the lanes of one wave share without a barrier.  Its accesses run in
order; what has to hold is that the compiler keeps them so, reads after writes
and writes after reads: every wave-wide fence of the kernels orders both
directions, and 32-bit accesses to the streams of smaller elements are of a
type that may alias them.  Read off the device code that the compiler gets."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2411_12788_amd import build as B


@pytest.mark.skipif(shutil.which(B.HIPCC) is None and not os.path.exists(B.HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("src", ["render.hip", "tiles.hip"])
def test_wave_fences_order_both_directions(tmp_path, src):
    out = tmp_path / (src + ".ll")
    # before the optimiser, which may merge or drop fences
    cmd = [B.HIPCC, *B.CFLAGS, "-Xclang", "-disable-llvm-passes", "--cuda-device-only", "-emit-llvm", "-S",
           os.path.join(B.CSRC, src), "-o", str(out)]
    subprocess.check_call(cmd, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    orders = re.findall(r'fence syncscope\("wavefront(?:-one-as)?"\) (\w+)', out.read_text())
    assert orders and set(orders) == {"acq_rel"}, orders


def test_streams_are_read_through_a_type_that_may_alias():
    text = open(os.path.join(B.CSRC, "render.hip")).read()
    accesses = [l for l in text.splitlines() if "reinterpret_cast" in l and "stream" in l]
    assert len(accesses) == 3 and all("AliasedU32" in l for l in accesses), accesses
