"""Workspace sizes of plans above 64 levels (host only, CPU): the selection's
state between sweeps of 64 levels lies in regions that are idle by then."""
import ctypes

import pytest

from paper_1904_06017_amd import _lib
from paper_1904_06017_amd.api import make_params


def _bytes(W, H, D, dtype):
    lib = _lib.load()
    p = make_params(W, H, D, dtype=dtype, delta_p=8, plane=(8, 0, 0.1), ncc_radius=3,
                    bil_radius=6, sigma_s=5, sigma_r=12)
    h, n = ctypes.c_void_p(), ctypes.c_size_t()
    assert lib.stereo_plan_create(ctypes.byref(p), ctypes.byref(h)) == 0
    assert lib.stereo_plan_workspace_bytes(h, ctypes.byref(n)) == 0
    lib.stereo_plan_destroy(h)
    return n.value


@pytest.mark.parametrize("W,H", [(1920, 1080), (317, 243), (33, 20)])
@pytest.mark.parametrize("dtype,state", [("u8", 16), ("f32", 0)])
def test_selection_state_above_64_levels(W, H, dtype, state):
    """From 64 to 65 levels the two cost volumes gain a block of 16 levels (4
    bytes a stored column and level, 16 more columns than whole strips and a
    row more to a pair), the backward's maps of the target one column each (16
    of 4 bytes a row cover them), and the state at most `state` bytes a pixel."""
    pitch, rows = (W + 15) // 16 * 16 + 16, H + 1
    grown = _bytes(W, H, 65, dtype) - _bytes(W, H, 64, dtype)
    assert grown <= 2 * 4 * 16 * pitch * rows + 16 * 4 * (H + 6) + state * W * H + 32 * 256
