"""Gradient maps of wide range and with non-finite pixels in the backward of
the soft-argmin head, window radii 6 to 8: the gradients of pixels out of reach
of an extreme one are what they are without it."""
from dataclasses import replace

import numpy as np
import pytest
import torch
from scipy import ndimage

import oracle.soft as SO
from synth import workload

pytestmark = pytest.mark.gpu
api = pytest.importorskip("paper_1904_06017_amd.api")

W, H, r = 90, 96, 2
D, SIGMA_R = 32, 12.0


def _host(x):
    torch.cuda.synchronize()
    return x.cpu().numpy().astype(np.float64)


def _setup(R, num_disp=D, sigma_r=SIGMA_R):
    w = replace(workload("c1"), name="range", width=W, height=H, num_disp=num_disp, dtype="f32",
                bil_radius=R, sigma_s=0.6 * R + 0.7, sigma_r=sigma_r, ncc_radius=r,
                perspective=True, delta_p=10.0, plane=(10.0, 0.01, 0.0))
    rng = np.random.Generator(np.random.PCG64(R))
    t = 128.0 + 6.0 * ndimage.gaussian_filter(rng.normal(0.0, 20.0, (H, W + num_disp)), 1.0)
    ref, tar = (np.ascontiguousarray(x, np.float32) for x in (t[:, :W], t[:, 9:9 + W]))
    g = (1.0 + 0.5 * ndimage.gaussian_filter(rng.normal(size=(H, W)), 1.5)).astype(np.float32)
    return w, ref, tar, g


def _backward(w, ref, tar, g, engine=2, grad_levels=None):
    plan = api.Plan.from_workload(w)
    plan.set_tuning("agg_engine", engine)
    if grad_levels:
        plan.set_tuning("grad_levels", grad_levels)
    dref, dtar = torch.from_numpy(ref).cuda(), torch.from_numpy(tar).cuda()
    _, saved = api.soft_forward(plan, dref, dtar, w.plane)
    return [_host(x) for x in api.backward(plan, dref, dtar, w.plane, saved,
                                           torch.from_numpy(g).cuda())]


@pytest.mark.parametrize("R,num_disp,levels", [(6, 32, None), (7, 40, None), (7, 70, 32),
                                               (8, 61, None)])
@pytest.mark.parametrize("kind", ["outliers", "halves"])
def test_small_gradients_beside_large_ones(R, num_disp, levels, kind):
    """One pixel's gradient reaches 2 R + 2 r rows.  Rows further away keep the
    accuracy of an even map (1e-4 of the FP64 adjoint in L2: FP32 exponents
    E / T <= 20 leave the softmax weights within 2e-6, which the block variances
    of this texture amplify by less than 50), whatever the rest of the map
    holds: two pixels at 1e4 and 1e10, or an upper half at 1e8."""
    w, ref, tar, g = _setup(R, num_disp)
    far = slice(24 + 2 * (R + r), None)
    fwd = SO.soft_forward(ref, tar, w.plane, w)
    if kind == "outliers":
        g[3, 5], g[9, 60] = 1e4, 1e10
    else:
        g[:24] *= 1e8
    alone = g.astype(np.float64)
    alone[:24] = 0.0
    exact = SO.soft_backward(ref, tar, w.plane, w, fwd, alone)
    got = _backward(w, ref, tar, g, grad_levels=levels)
    for a, e in zip(got[:2], exact[:2]):
        assert np.linalg.norm(a[far] - e[far]) <= 1e-4 * np.linalg.norm(e[far])


@pytest.mark.parametrize("R,num_disp", [(6, 32), (7, 70), (8, 40)])
@pytest.mark.parametrize("what", ["nan", "inf", "image"])
def test_reach_of_a_non_finite_pixel(R, num_disp, what):
    """A pixel whose gradient (or reference value) is not finite spoils the
    pixels whose windows hold it, no others: the same gradients of the reference
    are finite as in the vector ALU's backward, which sums each pixel's own
    window, and equal to them; so are the rows of the target's out of reach."""
    w, ref, tar, g = _setup(R, num_disp)
    y, x = 46, 43
    if what == "image":
        ref[y, x] = np.nan
    else:
        g[y, x] = np.float32(what)
    plan = api.Plan.from_workload(w)
    dref, dtar, dg = (torch.from_numpy(a).cuda() for a in (ref, tar, g))
    _, saved = api.soft_forward(plan, dref, dtar, w.plane)
    out = []
    for engine in (2, 0):
        plan.set_tuning("agg_engine", engine)
        out.append([_host(t) for t in api.backward(plan, dref, dtar, w.plane, saved, dg)])
    (a, at, _), (v, vt, _) = out
    assert np.array_equal(np.isfinite(a), np.isfinite(v))
    assert not np.isfinite(a[y, x]) and np.isfinite(a[0, 0])
    ok = np.isfinite(v)
    assert np.linalg.norm(a[ok] - v[ok]) <= 1e-4 * np.linalg.norm(v[ok])
    reach = R + r if what != "image" else 2 * R + 2 * r + 4
    far = [i for i in range(H) if abs(i - y) > reach]
    assert np.linalg.norm(at[far] - vt[far]) <= 1e-4 * np.linalg.norm(vt[far])
