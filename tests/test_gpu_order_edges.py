"""The spatial order's kernels at the edges of their steps: permute at 8 x 256
rows per workgroup for every element size, and the bounding box at 256
workgroups of 256 threads with four rows each, with the extremes in the last
rows and in the rows of the last, partly filled step."""
import numpy as np
import pytest
import torch

import gs_inputs
from tests.test_gpu_order import _check, raster

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 256, 257, 1793, 2047, 2048, 2049, 4097])
@pytest.mark.parametrize("dtype", [torch.uint8, torch.int16, torch.int32, torch.int64, torch.complex128])
@pytest.mark.parametrize("planes", [1, 3])
def test_permute_edges(gpu_lib, n, dtype, planes):
    R = raster()
    g = gs_inputs.rng(n + planes)
    src = torch.from_numpy(g.integers(0, 100, size=(planes, n))).to(dtype).cuda()
    perm = g.permutation(n)
    out = R.permute(src, torch.from_numpy(perm.astype(np.int32)).cuda())
    assert torch.equal(out.cpu(), src.cpu()[:, torch.from_numpy(perm)])


@pytest.mark.parametrize("n", [65_535, 65_536, 196_609, 262_143, 262_144, 262_145, 300_001])
def test_box_edges(gpu_lib, n):
    g = gs_inputs.rng(n)
    m = g.uniform(-1.0, 1.0, size=(3, n)).astype(np.float32)
    m[0, n - 1], m[1, n - 2], m[2, n - 3] = 7.0, -5.0, 3.0
    m[0, min(65_536, n - 4)], m[1, n // 2] = -4.0, 6.0
    m[2, n - 5] = np.nan
    _check(m, f"box n={n}")
