"""The server's reservation for a batch covers what its buffers hold: records,
offsets, lists, the workspaces the library asks for, ranges, tile order and
outputs (no GPU: sizes only)."""
import math

import pytest

from paper_2411_12788_amd import raster as R
from paper_2411_12788_amd.serve import GpuExecutor


@pytest.mark.parametrize("n", [1, 4096, 200_000, 3_000_000])
@pytest.mark.parametrize("V", [1, 4, 16])
@pytest.mark.parametrize("pairs_per_record", [0.0, 0.5, 2.0, 12.0])
def test_reservation_covers_the_buffers(n, V, pairs_per_record):
    ex = GpuExecutor.__new__(GpuExecutor)  # without its streams
    ex.R = R
    lib = R.L.lib()
    w, h = 1280, 720
    pairs, pixels = int(n * V * pairs_per_record), V * w * h
    tiles = V * math.ceil(w / 16) * math.ceil(h / 16)
    held = V * n * (4 * R.L.GS_REC_FLOATS + 16)          # records, boxes
    held += V * n * 4 + lib.gs_bin_count_workspace_size(V * n)
    held += pairs * 4 + lib.gs_bin_sort_workspace_size(pairs)
    held += tiles * (8 + 4)                              # ranges, tile order
    held += pixels * (3 + 4) * 4                         # colour, depth, index, transmittance, last
    assert held <= ex._bytes(n, V, pixels, pairs)
