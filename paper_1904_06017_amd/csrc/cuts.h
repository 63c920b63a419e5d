// How launches are cut into workgroups' shares: host arithmetic on sizes and
// the number of CUs, without any device call.
#pragma once
#include <algorithm>
#include <utility>
#include <vector>

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

// Radii whose streamed aggregation may run with two workgroups on a CU, and the
// level blocks of a sweep that leave the LDS room for them at radii 3 and 4.
constexpr int kDuoR = 4, kDuoBlocks = 3;

// Radii 3 and 4: two workgroups a CU (1) or one (0), for nblk level blocks and
// rows block rows in the launch.  Not for four blocks: two sweeps there would
// need a state between them that plans up to 64 levels have no room for.
// Where three blocks a sweep make more sweeps than four do, only in launches of
// at least eight block rows a workgroup; in shorter ones the sweeps' ends cost
// more than the wait.  Match at R = 4, one workgroup -> two: 1280x720, 16 levels
// 207 -> 161 us, 80 levels 550 -> 436; 320x240, 80 levels 74.3 -> 66.3; two
// sweeps -> three: 128 levels, 640x480 251 -> 246, 320x240 86.0 -> 88.9 (soft
// forward 65.0 -> 69.4).
inline int duo_launch(int nblk, long rows, int cus) {
  if (nblk == 4) return 0;
  if ((nblk + 2) / 3 == (nblk + 3) / 4) return 1;
  return rows >= 16l * cus ? 1 : 0;
}

// A volume of a queued launch: tx strips of br block rows of cost w each.
struct QueueVol {
  double w;
  int tx, br;
};
constexpr int kMinSegRows = 4;          // block rows of the shortest segment

// Block rows per segment of each volume of a queued launch.  A segment costs its
// block rows and `fill` more, in which its pipeline fills and drains; segments
// run longest first, one a workgroup and round.  Of cuts from two segments a
// workgroup's share down to an eighth of it, the one whose longest workgroup is
// shortest: four segments a workgroup throughout, the rule before, spent a third
// of the time on filling where a volume's shares are short.
inline std::vector<int> queue_cut(const std::vector<QueueVol>& v, int wgs, int fill) {
  double total = 0.0, best = 1e300;
  for (const QueueVol& q : v) total += q.w * q.tx * q.br;
  std::vector<int> at(v.size()), len(v.size());
  std::vector<double> load(wgs);
  for (double T = 2.0 * total / wgs; T > 0.12 * total / wgs; T *= 0.93) {
    std::vector<std::pair<double, long>> runs;         // cost of a segment, how many
    for (size_t k = 0; k < v.size(); ++k) {
      const QueueVol& q = v[k];
      const int want = std::max(kMinSegRows, std::min(q.br, (int)(T / q.w)));
      const int n = (q.br + want - 1) / want;
      len[k] = std::max(std::min(kMinSegRows, q.br), (q.br + n - 1) / n);
      const int full = q.br / len[k], rest = q.br - full * len[k];
      runs.push_back({q.w * (len[k] + fill), (long)full * q.tx});
      if (rest) runs.push_back({q.w * (rest + fill), q.tx});
    }
    std::sort(runs.begin(), runs.end(), [](const auto& a, const auto& c) { return a.first > c.first; });
    std::fill(load.begin(), load.end(), 0.0);
    size_t p = 0;
    for (const auto& r : runs)
      for (long c = 0; c < r.second; ++c, p = p + 1 == load.size() ? 0 : p + 1) load[p] += r.first;
    const double longest = *std::max_element(load.begin(), load.end());
    if (longest < best) {
      best = longest;
      at = len;
    }
  }
  return at;
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
