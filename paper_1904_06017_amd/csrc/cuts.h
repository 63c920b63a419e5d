// How launches are cut into workgroups' shares: host arithmetic on sizes and
// the number of CUs, without any device call.
#pragma once

namespace stereo {

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
