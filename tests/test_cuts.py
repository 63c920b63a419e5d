"""How launches are cut into workgroups' shares (csrc/cuts.h): host arithmetic,
compiled here and called on the CPU."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1904_06017_amd", "csrc")
WRAP = r"""
#include "cuts.h"
extern "C" int level_part(long tiles, int chunks, int cus, int held) {
  return stereo::level_part(tiles, chunks, cus, held);
}
"""


@pytest.fixture(scope="module")
def cuts(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("cuts")
    (d / "w.cpp").write_text(WRAP)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "w.cpp"),
                    "-o", str(d / "w.so")], check=True)
    return ctypes.CDLL(str(d / "w.so"))


@pytest.mark.parametrize("cus", [256, 64])
@pytest.mark.parametrize("tiles", [0.1, 0.3, 0.94, 1.0, 1.2, 3.0, 3.6])
@pytest.mark.parametrize("chunks", [1, 2, 4, 6, 16])
def test_level_parts_of_workgroups_alone_on_a_cu(cuts, cus, tiles, chunks):
    """Where a CU holds one workgroup (16 levels per pass, R = 8), the rounds of
    a cut are the workgroups of the fullest CU: the cut taken is the cheapest by
    that count, so rounds that are full are not cut up (a cut costs 0.05 of a chunk)."""
    t = max(1, int(tiles * cus))
    rounds = lambda per: -(-t * -(-chunks // per) // cus) * (per + 0.05)
    per = cuts.level_part(ctypes.c_long(t), chunks, cus, 1)
    assert rounds(per) == min(rounds(k) for k in range(1, chunks + 1))
    if t % cus == 0:
        assert per == chunks
