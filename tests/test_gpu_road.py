"""Moments, fit and transformation of the road at the sizes where the kernels'
shares end: columns by 256 threads, rows by blocks, eight pixels a thread
loaded ahead; without a mask, and with pixels that are no disparity."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle.road as ORD
from synth import workload

pytestmark = pytest.mark.gpu
api = pytest.importorskip("paper_1904_06017_amd.api")

@pytest.mark.parametrize("W,H", [(5, 3), (255, 2), (256, 241), (257, 240), (33, 1500), (2049, 9),
                                 (2100, 500)])
@pytest.mark.parametrize("masked", [False, True])
def test_fit_at_share_edges(W, H, masked):
    """FP64 sums of exact products over at most 1.1 M pixels leave the fit
    within 1e-6 of the oracle's (it stops at steps below 1e-6 rad)."""
    rng = np.random.Generator(np.random.PCG64(W + H))
    psi = 0.04
    v, u = np.mgrid[:H, :W]
    d = (20.0 + 0.05 * (v * np.cos(psi) - u * np.sin(psi)) +
         rng.normal(0.0, 0.01, (H, W))).astype(np.float32)
    if W * H > 100:
        d[0, 1], d[H - 1, W - 1], d[H // 2, W // 2] = np.nan, np.inf, -np.inf
    mask = rng.random((H, W)) < 0.8 if masked else None
    w = replace(workload("c1"), name="edge", width=W, height=H, num_disp=8)
    plan = api.Plan.from_workload(w)
    want, dt = ORD.road_transform(d.astype(np.float64), mask=mask, delta_t=1.5)
    m = None if mask is None else torch.from_numpy(mask.astype(np.uint8)).cuda()
    got, out = api.road_transform(plan, torch.from_numpy(d).cuda(), m, delta_t=1.5)
    out = out.cpu().numpy()
    assert got["n_points"] == np.count_nonzero(np.isfinite(d) & (True if mask is None else mask))
    assert abs(got["psi"] - want.psi) <= 1e-6
    fin = np.isfinite(d)
    assert np.array_equal(np.isnan(out), np.isnan(dt))
    assert np.abs(out[fin] - dt[fin]).max() <= 1e-5 + 1e-6 * 0.05 * max(W, H)
