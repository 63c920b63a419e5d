"""The streamed split-FP16 aggregation at the sizes where its cuts fall: strip
and block-row remainders, level blocks and sweeps (16 levels each, 64 per
sweep), every window radius, against the FP64 oracle; both volumes in one
launch against one launch per volume; the soft-argmin over several sweeps."""
import ctypes
from dataclasses import replace

import numpy as np
import pytest
import torch
from scipy import ndimage

import oracle.soft as SO
import oracle.stereo as OS
from synth import workload
from tests import parity_rules as PR

pytestmark = pytest.mark.gpu
api = pytest.importorskip("paper_1904_06017_amd.api")

# (R, width, height, levels): one pixel and one level either side of a strip
# (16 columns), a block row (4 rows), a level block and a sweep
SIZES = [(1, 16, 4, 3), (1, 33, 9, 17), (2, 47, 13, 16), (2, 90, 30, 65), (3, 64, 12, 64),
         (3, 95, 31, 40), (4, 49, 27, 33), (4, 17, 70, 96), (5, 130, 41, 128), (5, 31, 6, 30),
         (6, 81, 18, 66), (7, 112, 45, 64), (7, 97, 23, 129), (8, 65, 50, 48), (8, 50, 21, 81)]


def _pair(R, W, H, D, dtype):
    rng = np.random.Generator(np.random.PCG64(1000 * R + W))
    t = 128.0 + 6.0 * ndimage.gaussian_filter(rng.normal(0.0, 20.0, (H, W + D)), 1.0)
    ref, tar = t[:, :W], t[:, D // 3:D // 3 + W]
    if dtype == "u8":
        return (np.clip(np.rint(x), 0, 255).astype(np.uint8) for x in (ref, tar))
    return (np.ascontiguousarray(x, np.float32) for x in (ref, tar))


def _workload(R, W, H, D, dtype, **kw):
    return replace(workload("c1"), name="edge", width=W, height=H, num_disp=D, dtype=dtype,
                   bil_radius=R, sigma_s=0.6 * R + 0.7, sigma_r=12.0, ncc_radius=2, **kw)


def _host(x):
    torch.cuda.synchronize()
    return x.cpu().numpy()


@pytest.mark.parametrize("R,W,H,D", SIZES)
def test_match_at_cut_edges(R, W, H, D):
    dtype = "u8" if R % 2 else "f32"
    w = _workload(R, W, H, D, dtype, perspective=False, delta_p=0.0)
    ref, tar = _pair(R, W, H, D, dtype)
    plan = api.Plan.from_workload(w)
    dref, dtar = torch.from_numpy(ref).cuda(), torch.from_numpy(tar).cuda()
    out = api.match(plan, dref, dtar, want_target=True)
    got = {k: _host(v) for k, v in out.items()}
    ora = OS.match(ref, tar, w, keep_volumes=True)
    PR.check_selection(w, ora, got["dint_R"], got["dint_T"], got["dsub"], got["valid"],
                       got["disp"])
    # the profiled form launches the volumes one by one
    two = {k: torch.empty_like(v) for k, v in out.items()}
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(7)]
    for e in ev:
        e.record()
    lib, ws = api._lib.load(), plan.workspace("cuda")
    api.check(lib.stereo_match_profiled(
        plan.handle, api._p(dref), api._p(dtar), api._p(two["dint_R"]), api._p(two["dint_T"]),
        api._p(two["dsub"]), api._p(two["valid"]), api._p(two["disp"]), api._p(ws),
        plan.workspace_bytes, (ctypes.c_void_p * 7)(*[e.cuda_event for e in ev]),
        api._stream()))
    for k in got:
        assert np.array_equal(got[k], _host(two[k]), equal_nan=True), k


@pytest.mark.parametrize("R,W,H,D", [(3, 50, 18, 64), (4, 33, 21, 65), (7, 63, 30, 140)])
def test_soft_forward_over_sweeps(R, W, H, D):
    """The softmax state carried between sweeps: FP32 sums of E in [0, 2] over
    T = 0.1 keep the exponents within 2e-5, so the soft level of D levels is
    within 2e-5 D of the oracle's (its softmax weights move by at most that
    relative amount)."""
    w = _workload(R, W, H, D, "f32", perspective=True, delta_p=float(D // 3),
                  plane=(float(D // 3), 0.0, 0.0))
    ref, tar = _pair(R, W, H, D, "f32")
    plan = api.Plan.from_workload(w)
    disp, saved = api.soft_forward(plan, torch.from_numpy(ref).cuda(),
                                   torch.from_numpy(tar).cuda(), w.plane)
    fwd = SO.soft_forward(ref, tar, w.plane, w)
    assert np.abs(_host(saved)[2] - fwd["dh"]).max() <= 2e-5 * D
    assert np.abs(_host(disp) - fwd["disp"]).max() <= 2e-5 * D


@pytest.mark.parametrize("R,W,H,D", [(1, 16, 4, 16), (2, 33, 9, 17), (3, 47, 31, 64), (4, 31, 14, 65),
                                     (5, 65, 13, 33), (6, 49, 27, 40), (6, 130, 22, 64),
                                     (7, 81, 18, 70), (7, 17, 45, 48), (8, 50, 21, 30),
                                     (8, 97, 12, 129)])
def test_backward_at_cut_edges(R, W, H, D):
    """Both backward passes at strip, block-row, level-block and level-tile
    remainders.  FP32 exponents E / T <= 20 leave the softmax weights within
    2e-6, which the block variances of this texture amplify by less than 50:
    each gradient within 1e-4 of the FP64 adjoint in L2, and of the vector
    ALU's.  The plane terms cancel: 1e-3 of the largest, as for that one."""
    w = _workload(R, W, H, D, "f32", perspective=True, delta_p=float(D // 3),
                  plane=(float(D // 3), 0.01, 0.0))
    ref, tar = _pair(R, W, H, D, "f32")
    rng = np.random.Generator(np.random.PCG64(R + W))
    g = ndimage.gaussian_filter(rng.normal(size=(H, W)), 1.5).astype(np.float32)
    fwd = SO.soft_forward(ref, tar, w.plane, w)
    exact = SO.soft_backward(ref, tar, w.plane, w, fwd, g.astype(np.float64))
    dref, dtar, dg = (torch.from_numpy(x).cuda() for x in (ref, tar, g))
    got = []
    for engine in (2, 0):
        plan = api.Plan.from_workload(w)
        plan.set_tuning("agg_engine", engine)
        _, saved = api.soft_forward(plan, dref, dtar, w.plane)
        got.append([_host(x).astype(np.float64)
                    for x in api.backward(plan, dref, dtar, w.plane, saved, dg)])
    for a, v, e, tol in zip(*got, exact, (1e-4, 1e-4, 1e-3)):
        assert np.linalg.norm(a - e) <= tol * np.linalg.norm(e)
        assert np.linalg.norm(a - v) <= tol * np.linalg.norm(e)


def test_backward_keeps_its_scale_beside_an_infinite_gradient():
    """The FP16 scale of pass 2's input comes from the finite gradients alone:
    a pixel whose gradient is infinite leaves the others, far from it, where
    they are without it (1e-6: the same products at the same scale, other
    neighbours)."""
    R, W, H, D = 6, 96, 80, 32
    w = _workload(R, W, H, D, "f32", perspective=True, delta_p=10.0, plane=(10.0, 0.0, 0.0))
    ref, tar = _pair(R, W, H, D, "f32")
    g = np.full((H, W), 1e-6, np.float32)
    dref, dtar = torch.from_numpy(ref).cuda(), torch.from_numpy(tar).cuda()
    plan = api.Plan.from_workload(w)
    _, saved = api.soft_forward(plan, dref, dtar, w.plane)
    plain = _host(api.backward(plan, dref, dtar, w.plane, saved, torch.from_numpy(g).cuda())[0])
    g[2, 2] = np.inf
    odd = _host(api.backward(plan, dref, dtar, w.plane, saved, torch.from_numpy(g).cuda())[0])
    far = (slice(60, None), slice(None))
    assert np.linalg.norm(odd[far] - plain[far]) <= 1e-6 * np.linalg.norm(plain[far])


@pytest.mark.parametrize("W,H,D,dtype", [(41, 9, 5, "u8"), (700, 130, 33, "u8"),
                                         (1931, 1083, 18, "f32"), (2561, 1441, 17, "u8")])
def test_every_cost_tile_is_written(W, H, D, dtype):
    """The cost tiles are dealt out by XCD in runs bounded by their input
    bytes (one, and at the larger sizes two and three runs of level blocks of
    16, 32 and 64): over a workspace of NaNs every level block size gives the
    same results, bit for bit, so no tile is left out."""
    w = _workload(2, W, H, D, dtype, perspective=False, delta_p=0.0)
    ref, tar = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in _pair(2, W, H, D, dtype))
    want = None
    for levels in (16, 32, 64):
        plan = api.Plan.from_workload(w)
        plan.set_tuning("ncc_levels", levels)
        plan.workspace("cuda").fill_(255)
        got = {k: _host(v) for k, v in api.match(plan, ref, tar, want_target=True).items()}
        if want is None:
            want = got
            assert not np.isnan(got["dsub"]).any()
        for k in got:
            assert np.array_equal(got[k], want[k], equal_nan=True), (levels, k)


@pytest.mark.parametrize("r", range(1, 9))
@pytest.mark.parametrize("W,H", [(5, 3), (64 - 3, 16), (131, 37)])
def test_block_statistics_of_every_radius(r, W, H):
    """The statistics kernel has a form per block radius: costs of both
    volumes at map sizes below, at and beyond its 64 x 16 tiles, within the
    bound of the cost's FP32 arithmetic."""
    D = 7
    dtype = "u8" if r % 2 else "f32"
    w = replace(_workload(2, W, H, D, dtype, perspective=False, delta_p=0.0), ncc_radius=r)
    ref, tar = _pair(2, W, H, D, dtype)
    ora = OS.match(ref, tar, w, keep_volumes=True)
    plan = api.Plan.from_workload(w)
    cR, cT = api.cost_volume(plan, torch.from_numpy(ref).cuda(),
                             torch.from_numpy(np.asarray(tar, np.float32)).cuda())
    PR.assert_cost_close(_host(cR), ora["C_R"], "C_R")
    PR.assert_cost_close(_host(cT), ora["C_T"], "C_T")


@pytest.mark.parametrize("D", [3, 7, 8, 9, 15, 16, 17, 24, 33, 64])
def test_selection_over_chunks_of_levels(D):
    """The materialised selection reads its levels in chunks of eight: first
    minimum, sub-pixel offset and non-finite costs as a plain walk of the
    levels gives them (the same FP32 arithmetic: equal)."""
    H, W = 5, 67
    rng = np.random.Generator(np.random.PCG64(D))
    E = rng.integers(0, 9, (D, H, W)).astype(np.float32) / 8
    E[rng.random(E.shape) < 0.1] = np.nan
    E[rng.random(E.shape) < 0.05] = np.inf
    E[:, 0, :3] = np.nan
    best, at = np.full((H, W), np.finfo(np.float32).max, np.float32), np.zeros((H, W), int)
    for d in range(D):
        low = E[d] < best
        best, at = np.where(low, E[d], best), np.where(low, d, at)
    get = lambda d: np.take_along_axis(E, np.clip(d, 0, D - 1)[None], 0)[0]
    with np.errstate(all="ignore"):
        lo, hi = get(at - 1), get(at + 1)
        den = 2 * lo + 2 * hi - 4 * best
        off = np.where((at > 0) & (at < D - 1) & (den > 0), (lo - hi) / den, np.float32(0))
    plan = api.Plan(api.make_params(W, H, D))
    dint, dsub = api.wta_subpixel(plan, torch.from_numpy(E).cuda())
    assert np.array_equal(_host(dint), at)
    assert np.array_equal(_host(dsub), at.astype(np.float32) + off.astype(np.float32),
                          equal_nan=True)


@pytest.mark.parametrize("W,H,D,levels", [(31, 9, 3, 8), (33, 40, 8, 8), (70, 65, 9, 8), (64, 33, 40, 8),
                                          (129, 50, 17, 16), (90, 70, 48, 16), (640, 480, 31, 8)])
def test_aggregation_in_level_parts(W, H, D, levels):
    """The materialised aggregation cuts its levels into parts by the number
    of tiles; a level's sum is the same in every cut: equal to the aggregation
    of that level among eight, alone in its part."""
    w = _workload(4, W, H, D, "u8")
    ref, _ = _pair(4, W, H, D, "u8")
    rng = np.random.Generator(np.random.PCG64(D))
    cost = torch.from_numpy(rng.random((D, H, W), dtype=np.float32)).cuda()
    guide = torch.from_numpy(ref).cuda()
    plan = api.Plan.from_workload(w)
    plan.set_tuning("agg_levels_u8", levels)
    whole = _host(api.bilateral_aggregate(plan, guide, cost))
    few = api.Plan.from_workload(replace(w, num_disp=8))
    few.set_tuning("agg_levels_u8", 8)
    for d in {0, D // 2, D - 1}:
        part = torch.zeros(8, H, W, device="cuda")
        part[d % 8] = cost[d]
        assert np.array_equal(whole[d], _host(api.bilateral_aggregate(few, guide, part))[d % 8])


@pytest.mark.parametrize("W,H", [(40, 9), (300, 70)])
@pytest.mark.parametrize("value", [1.0, -0.37, 0.0, float("nan")])
def test_loss_gradient_on_the_device(W, H, value):
    """A loss gradient left in device memory gives what its value gives: the
    same FP64 quotient, so the same bits."""
    w = _workload(2, W, H, 8, "f32", perspective=True, delta_p=3.0, plane=(3.0, 0.0, 0.0))
    ref, tar = (torch.from_numpy(x).cuda() for x in _pair(2, W, H, 8, "f32"))
    disp = torch.full((H, W), 2.6, device="cuda")
    plan = api.Plan.from_workload(w)
    want = api.photometric_l1_bwd(plan, ref, tar, disp, value)
    pair = torch.tensor([7.0, value], dtype=torch.float64, device="cuda")
    for grad in (pair[1], pair[1:], pair[1].float(), pair[1].cpu()):
        got = api.photometric_l1_bwd(plan, ref, tar, disp, grad)
        if grad.dtype == torch.float64:
            assert all(torch.equal(a.nan_to_num(9.0), b.nan_to_num(9.0)) for a, b in zip(got, want))


@pytest.mark.parametrize("R,W,H,D,dtype", [(1, 90, 41, 16, "u8"), (2, 130, 22, 100, "f32"),
                                           (3, 95, 31, 16, "u8"), (3, 500, 300, 128, "u8"),
                                           (4, 66, 50, 48, "f32"), (4, 500, 300, 113, "f32")])
def test_two_workgroups_a_cu_give_the_same_bits(R, W, H, D, dtype):
    """Small radii run with two workgroups on a CU, radii 3 and 4 by a rule on
    levels and block rows (at 500 x 300 two volumes in one launch are enough
    for it, one is not): the match, each volume alone and the queue of a batch,
    whose other pair has 64 levels and so one workgroup on a CU, agree bit for
    bit."""
    w = _workload(R, W, H, D, dtype, perspective=False, delta_p=0.0)
    ref, tar = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in _pair(R, W, H, D, dtype))
    plan = api.Plan.from_workload(w)
    out = api.match(plan, ref, tar, want_target=True)
    got = {k: _host(v) for k, v in out.items()}
    alone = {k: torch.empty_like(v) for k, v in out.items()}
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(7)]
    for e in ev:
        e.record()
    ws = plan.workspace(ref.device)
    api.check(api._lib.load().stereo_match_profiled(
        plan.handle, api._p(ref), api._p(tar), api._p(alone["dint_R"]), api._p(alone["dint_T"]),
        api._p(alone["dsub"]), api._p(alone["valid"]), api._p(alone["disp"]), api._p(ws),
        plan.workspace_bytes, (ctypes.c_void_p * 7)(*[e.cuda_event for e in ev]), api._stream()))
    for k in got:
        assert np.array_equal(got[k], _host(alone[k]), equal_nan=True), k
    v = _workload(R, 70, 33, 64, dtype, perspective=False, delta_p=0.0)
    other = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in _pair(R, 70, 33, 64, dtype)]
    for pairs in ([(plan, ref, tar)], [(plan, ref, tar), (api.Plan.from_workload(v), *other)]):
        res = api.Batch(pairs).submit()[0]
        for k in ("dint_R", "valid", "disp"):
            assert np.array_equal(got[k], _host(res[k]), equal_nan=True), (len(pairs), k)
