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
extern "C" void queue_cut(int n, const double* w, const int* tx, const int* br, int wgs, int fill,
                          int* out) {
  std::vector<stereo::QueueVol> v;
  for (int k = 0; k < n; ++k) v.push_back({w[k], tx[k], br[k]});
  const std::vector<int> cut = stereo::queue_cut(v, wgs, fill);
  for (int k = 0; k < n; ++k) out[k] = cut[k];
}
extern "C" int duo_launch(int nblk, long rows, int cus) { return stereo::duo_launch(nblk, rows, cus); }
extern "C" int sweep_blocks(int nblk, int most) { return stereo::sweep_blocks(nblk, most); }
extern "C" int cost(int nblk, int most) { return (int)stereo::block_row_cost(nblk, most); }
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


@pytest.mark.parametrize("wgs", [512, 256, 64])
@pytest.mark.parametrize("fill", [4, 6])
@pytest.mark.parametrize("vols", [
    [(10, 50, 146)] * 2, [(8, 27, 82)] * 2 + [(5, 21, 62)] * 2 + [(4, 14, 43)] * 2,
    [(9, 20, 60)], [(11, 27, 77)] * 2 + [(9, 21, 62)] * 2 + [(7, 16, 46)] * 2,
    [(6, 80, 180)] * 2 + [(8, 120, 270)] * 2 + [(5, 40, 120)] * 2, [(3, 1, 1)], [(7, 2, 3)] * 4,
    [(10, 120, 270)] * 128])
def test_segments_of_a_queued_launch(cuts, vols, wgs, fill):
    """Segments run longest first, one a workgroup and round.  The cut covers
    every strip with segments of at least four block rows (or the strip), and
    its longest workgroup is at most 1.4 times an even share of the block rows
    plus the one filling that nothing avoids, or the shortest cut there is."""
    out = (ctypes.c_int * len(vols))()
    arr = lambda t, k: (t * len(vols))(*[v[k] for v in vols])
    cuts.queue_cut(len(vols), arr(ctypes.c_double, 0), arr(ctypes.c_int, 1),
                   arr(ctypes.c_int, 2), wgs, fill, out)

    def longest(lens):
        c = sorted((w * (min(n, br - r) + fill) for (w, tx, br), n in zip(vols, lens)
                    for r in range(0, br, n) for _ in range(tx)), reverse=True)
        return max(sum(c[p::wgs]) for p in range(min(wgs, len(c))))

    assert all(min(4, br) <= n <= br for n, (_, _, br) in zip(out, vols))
    share = sum(w * tx * br for w, tx, br in vols) / wgs
    w = max(v[0] for v in vols)
    least = longest([min(4, br) for _, _, br in vols])
    assert longest(out) <= max(1.4 * share + w * fill, least if least < w * 24 else 0)


@pytest.mark.parametrize("most", [3, 4])
@pytest.mark.parametrize("nblk", range(1, 17))
def test_sweeps_compute_every_level_block_once(cuts, nblk, most):
    """As few sweeps as hold the blocks, none empty, each block in one of them;
    the cost of a block row counts the weights of each sweep and the blocks."""
    left, sweeps = nblk, []
    while left > 0:
        sweeps.append(cuts.sweep_blocks(left, most))
        left -= sweeps[-1]
    assert left == 0 and min(sweeps) >= 1 and max(sweeps) <= most
    assert len(sweeps) == -(-nblk // most) and max(sweeps) - min(sweeps) <= 1
    assert cuts.cost(nblk, most) == 2 * len(sweeps) + nblk


@pytest.mark.parametrize("cus", [256, 64])
@pytest.mark.parametrize("nblk", range(1, 17))
def test_two_workgroups_on_a_cu(cuts, nblk, cus):
    """Radii 3 and 4 sweep three level blocks at a time where two workgroups
    share a CU.  More than one sweep needs a state, which plans above 64 levels
    (four blocks) have: never at four blocks.  Where it takes more sweeps than
    four blocks at a time, only with eight block rows a workgroup."""
    few, many = (cuts.duo_launch(nblk, ctypes.c_long(n), cus) for n in (16 * cus - 1, 16 * cus))
    if nblk == 4:
        assert (few, many) == (0, 0)
    else:
        assert many == 1 and few == (-(-nblk // 3) == -(-nblk // 4))
