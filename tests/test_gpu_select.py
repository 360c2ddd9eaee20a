"""Selection passes at the sizes where their batches (8 elements of a thread),
steps (4096 of a workgroup) and problems meet, and with keys one apart: the
mass threshold's next larger key then lies inside or outside the last pass's
group, and sampling takes all or a part of the values equal to the k-th.  The
values are multiples of 2^-24 below 1, so every sum is exact in float64 in any
order and the results must equal the oracle's."""
import numpy as np
import pytest
import torch

import gs_inputs
import oracle

pytestmark = pytest.mark.gpu

VALUE, MASS = oracle.THRESHOLD_VALUE, oracle.THRESHOLD_MASS


def D():
    from paper_2411_12788_amd import densify
    return densify


def _close_keys(n, seed, spread):
    g = gs_inputs.rng(seed)
    v = (0.5 + g.integers(0, spread, size=n) * 2.0 ** -24).astype(np.float32)
    v[g.random(n) < 0.1] = 0.0  # not selected
    return v


@pytest.mark.parametrize("n", [1, 7, 255, 257, 2047, 2049, 4095, 4096, 4097, 8193, 70_001])
@pytest.mark.parametrize("spread", [1, 3, 300])
def test_thresholds_at_close_keys(gpu_lib, n, spread):
    imp = np.stack([_close_keys(n, 7 * n + k, spread) for k in range(3)])
    for mode in (VALUE, MASS):
        for keep in (0.0, 0.003, 0.25, 0.5, 0.77, 0.99, 1.0):
            print(f"n={n}, spread={spread}, mode={mode}, keep={keep}", flush=True)
            vis, tau = D().visibility(torch.from_numpy(imp).cuda(), keep, mode)
            vis, tau = vis.cpu().numpy(), tau.cpu().numpy()
            for k in range(3):
                vo, to, _ = oracle.visibility(imp[k], keep, mode)
                assert tau[k] == to or (np.isnan(tau[k]) and np.isnan(to)), (k, tau[k], to)
                assert (vis[k] == vo).all(), k


@pytest.mark.parametrize("n", [1, 255, 2049, 4095, 4097, 70_001])
@pytest.mark.parametrize("spread", [1, 5])
def test_sample_takes_all_or_first_ties(gpu_lib, n, spread):
    imp = np.ones(n, np.float32)
    expo = _close_keys(n, n, spread) + np.float32(0.0)
    expo[expo == 0.0] = 0.25
    order = np.sort(expo)
    edges = np.flatnonzero(np.diff(order)) + 1  # k that ends a group of ties
    ks = {0, 1, n // 2, n, n + 5, *(int(e) for e in edges[:3]), *(int(e) + 1 for e in edges[:2])}
    for k in sorted(ks):
        print(f"n={n}, spread={spread}, k={k}", flush=True)
        sel, cnt = D().sample(torch.from_numpy(imp).cuda(), torch.from_numpy(expo).cuda(), k)
        assert (sel.cpu().numpy() == oracle.sample(imp, expo, k)).all()
        assert int(cnt.cpu()[0]) == min(k, n)
