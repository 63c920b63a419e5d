// How launches are cut into workgroups' shares: host arithmetic on sizes and
// the number of CUs, without any device call.
#pragma once
#include <algorithm>

namespace stereo {

// Level blocks of the streamed aggregation's next sweep with nblk blocks still
// to do: even shares of at most `most`, the larger ones first (13 in sweeps of
// at most 4: 4, 3, 3, 3).
constexpr int sweep_blocks(int nblk, int most) {
  const int n = (nblk + most - 1) / most;
  return (nblk + n - 1) / n;
}

// Cost of a block row of nblk level blocks in sweeps of at most `most`: the
// weights once per sweep (2), the products per block.
inline double block_row_cost(int nblk, int most) {
  return 2.0 * ((nblk + most - 1) / most) + nblk;
}

// Block rows of a segment of a queued launch: br block rows of cost w each, cut
// so that the launch (total cost) makes about four segments for each of its
// cus workgroups.  A segment fills and drains its pipeline of block rows, so
// it has at least eight.
inline int segment_rows(double total, double w, int br, int cus) {
  const int want = std::max(8, (int)(total / (4.0 * cus) / w));
  const int n = std::max(1, (br + want - 1) / want);
  return (br + n - 1) / n;
}

// Levels of a materialised aggregation in parts of `per` chunks each, where
// that evens out the CUs' shares (tiles: workgroups of one part, chunks: level
// chunks in all, held: workgroups that share a CU).  A part costs per + 0.05
// (every chunk forms its own weights anyway); a workgroup alone on a CU that
// holds two takes 0.62 of a pair's time.
inline int level_part(long tiles, int chunks, int cus, int held) {
  double best = 1e30;
  int at = chunks;
  for (int per = chunks; per >= 1; --per) {
    const int z = (chunks + per - 1) / per;
    const long m = (tiles * z + cus - 1) / cus;        // workgroups of the fullest CU
    const double rounds = held > 1 ? (double)(m / 2) + (m & 1 ? 0.62 : 0.0) : (double)m;
    const double cost = rounds * (per + 0.05);
    if (cost < best) { best = cost; at = per; }
  }
  return at;
}

}  // namespace stereo
