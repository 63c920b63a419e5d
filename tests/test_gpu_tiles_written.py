"""Every element of the cost volumes is written, whatever the order in which
their tiles are dealt out over the XCDs."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from synth import workload

pytestmark = pytest.mark.gpu
api = pytest.importorskip("paper_1904_06017_amd.api")

R, r = 2, 2


def _workspace(plan):
    """The buffer that calls on tensors of the current device use."""
    return plan.workspace(torch.device("cuda", torch.cuda.current_device()))


def _plan(W, H, D, dtype, levels, soft=False):
    w = replace(workload("c1"), name="tiles", width=W, height=H, num_disp=D, dtype=dtype,
                bil_radius=R, sigma_s=2.0, sigma_r=12.0, ncc_radius=r, perspective=soft,
                delta_p=3.0 if soft else 0.0, plane=(3.0, 0.0, 0.0))
    plan = api.Plan.from_workload(w)
    plan.set_tuning("ncc_levels", levels)
    _workspace(plan).fill_(255)
    g = torch.Generator(device="cuda").manual_seed(W)
    im = [255 * torch.rand(H, W, device="cuda", generator=g) for _ in range(2)]
    return plan, [x.to(torch.uint8) if dtype == "u8" else x for x in im]


def _split_volumes(plan, W, H, D, n):
    """The first n split volumes of the workspace, as halves: after the warped
    target [H][W] and four statistics maps [H][W + 2 r], every region 256-byte
    aligned; blocks of 16 levels, two parts each, of H stored rows (an even
    number; R is even) of the 16-pixel strips' columns and 8 more."""
    align = lambda b: (b + 255) // 256 * 256
    off = align(4 * W * H) + align(16 * (W + 2 * r) * H)
    halves = 2 * (-(-D // 16)) * 16 * (H + H % 2) * ((W + 15) // 16 * 16 + 8)
    ws = _workspace(plan)
    return [ws[off + k * align(2 * halves):][:2 * halves].view(torch.int16) for k in range(n)]


def _runs(W, H, D, dtype):
    """Runs of an XCD's share of 60 x 16 tiles: at most 3 MB of images and
    statistics (element + 20 bytes a pixel) each."""
    nx = -(-((W + 15) // 16 * 16 + 8 + -(-D // 16) * 16) // 60)
    share = -(-nx * -(-H // 16) // 8) * 60 * 16 * (21 if dtype == "u8" else 24)
    return -(-share // (3 << 20))


# a whole range in a fraction of a tile row, 8-row tiles, and one to four runs
# of 16-row ones
SIZES = [(41, 9, 5, "u8", 1), (700, 130, 33, "u8", 1), (1283, 719, 40, "u8", 1),
         (1501, 871, 17, "u8", 2), (1931, 1083, 18, "f32", 3), (2561, 1441, 17, "u8", 4)]


@pytest.mark.parametrize("W,H,D,dtype,runs", SIZES)
@pytest.mark.parametrize("levels", [0, 16, 32, 64])
def test_no_element_of_the_split_volumes_is_left_out(W, H, D, dtype, runs, levels):
    """Costs are finite, so no half of a written element has the bits of the
    workspace's filling (a NaN)."""
    assert _runs(W, H, D, dtype) == runs
    plan, (ref, tar) = _plan(W, H, D, dtype, levels)
    api.match(plan, ref, tar, want_target=True)
    left = [int((vol == -1).sum()) for vol in _split_volumes(plan, W, H, D, 2)]
    assert left == [0, 0]


@pytest.mark.parametrize("W,H,D", [(41, 10, 5), (700, 130, 33), (1931, 1083, 18)])
def test_no_element_of_the_soft_volume_is_left_out(W, H, D):
    plan, (ref, tar) = _plan(W, H, D, "f32", 0, soft=True)
    api.soft_forward(plan, ref, tar, (3.0, 0.0, 0.0))
    left = int((_split_volumes(plan, W, H, D, 1)[0] == -1).sum())
    assert left == 0


@pytest.mark.parametrize("W,H,D,dtype,runs", SIZES)
@pytest.mark.parametrize("levels", [0, 16, 32])
def test_no_element_of_the_planar_volumes_is_left_out(W, H, D, dtype, runs, levels):
    plan, (ref, tar) = _plan(W, H, D, dtype, levels)
    vols = [torch.full((D, H, W), float("nan"), device="cuda") for _ in range(2)]
    tarw, ws, lib = tar.float(), _workspace(plan), api._lib.load()
    api.check(lib.stereo_cost_volume(plan.handle, api._p(ref), api._p(tarw), api._p(vols[0]),
                                     api._p(vols[1]), api._p(ws), plan.workspace_bytes,
                                     api._stream()))
    left = [int(v.isnan().sum()) for v in vols]
    assert left == [0, 0]
