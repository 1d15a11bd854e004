// Rules that shape launches (host code, no device headers).
#pragma once
#include <algorithm>
#include <cstdint>
#include <utility>
#include <vector>

namespace ppe {

// Equal images of a pipelined 3x3 launch: tiles of each, workgroup columns that each of
// them is run for (images x output channel blocks x K shares), and upper and lower halves
// of the tiles that hold rows of the image.
struct ConvpPart {
  int64_t tiles, copies, halves;
};

struct ConvpRuns {
  int64_t run = 1;     // tiles per workgroup
  int64_t wgs = 0;     // workgroups of the launch
  int64_t span = 1;    // tiles one after another on the busiest compute unit
  bool fills = false;  // see convp_fills
};

inline int64_t convp_wgs(const std::vector<ConvpPart>& parts, int64_t run) {
  int64_t n = 0;
  for (const ConvpPart& p : parts) n += p.copies * (int64_t)(((uint32_t)p.tiles + (uint32_t)run - 1) / (uint32_t)run);
  return n;
}

// Tiles that the busiest compute unit works off, and in how many workgroups. Up to a
// second round that is not full its workgroups follow the shortest runs of the
// first (a run ends with its image); beyond that whole rounds are counted.
inline std::pair<int64_t, int64_t> convp_span(const std::vector<ConvpPart>& parts, int64_t run, int64_t wgs,
                                              int64_t cus) {
  const int64_t rounds = (wgs + cus - 1) / cus;
  if (rounds <= 1) return {run, 1};
  if (rounds > 2) return {rounds * run, rounds};
  std::vector<std::pair<int64_t, int64_t>> shorts;  // (length, workgroups) of the images' last runs
  for (const ConvpPart& p : parts)
    if (p.tiles % run) shorts.push_back({p.tiles % run, p.copies});
  std::sort(shorts.begin(), shorts.end());
  // the workgroups past the first round, the last one first
  std::vector<int64_t> late;
  for (int64_t need = wgs - cus, k = (int64_t)parts.size() - 1; need > 0; k = k ? k - 1 : (int64_t)parts.size() - 1) {
    const int64_t n = (parts[k].tiles + run - 1) / run;
    for (int64_t i = n - 1; i >= 0 && need > 0; --i, --need) late.push_back(std::min(run, parts[k].tiles - i * run));
  }
  int64_t span = run;
  size_t q = 0;
  int64_t used = 0;
  for (size_t i = late.size(); i-- > 0;) {
    while (q < shorts.size() && used >= shorts[q].second) ++q, used = 0;
    span = std::max(span, late[i] + (q < shorts.size() ? shorts[q].first : run));
    ++used;
  }
  return {span, 2};
}

// A run ends with its image, so with several images the workgroups that a run length
// gives can pass the compute units although the tiles over them would not: 24 images of
// 128 tiles in runs of ceil(3072 / 256) = 12 are 264 workgroups, whose last eight start
// when the others end. So the run is the one with which the busiest compute unit has
// least to do, counted in tiles and one more for every workgroup (weights and the first
// inputs), between the shortest that could do and the shortest whose workgroups fit
// the rounds. A forward of 24 grids of 256 x 256 takes 841 us, with runs of ceil(tiles
// over compute units) 1079 us; 6 of them 321 and 356 us, 48 of 256 x 160 1115 and 1355 us.
inline ConvpRuns convp_runs(const std::vector<ConvpPart>& parts, int64_t cus) {
  int64_t longest = 1, images = 0, tiles = 0, halves = 0;
  for (const ConvpPart& p : parts) {
    longest = std::max(longest, p.tiles);
    images += p.copies;
    tiles += p.copies * p.tiles;
    halves += p.copies * p.halves;
  }
  ConvpRuns best;
  int64_t cost = 0;
  const int64_t even = (tiles + cus - 1) / cus;
  const int64_t first = std::max<int64_t>(1, (images + cus - 1) / cus);  // one run per image needs these rounds
  for (int64_t k = first; k < first + 4; ++k) {
    if (cost && cost <= even + 2) break;  // no unit with two workgroups has less
    int64_t run = std::min(longest, std::max<int64_t>(1, (tiles + k * cus - 1) / (k * cus)));
    // (steps of a thirty-second of the run: a grouped launch is planned on each call)
    for (;; run = std::min(longest, run + std::max<int64_t>(1, run / 32))) {
      if (cost && run + 1 >= cost) break;
      const int64_t wgs = convp_wgs(parts, run);
      const auto [span, chain] = convp_span(parts, run, wgs, cus);
      if (!cost || span + chain < cost) {
        cost = span + chain;
        best.run = run;
        best.wgs = wgs;
        best.span = span;
      }
      if (wgs <= k * cus || run == longest) break;
    }
  }
  const int64_t slots = cus * best.span;
  best.fills = 4 * tiles >= 3 * cus * even && (slots == cus || (3 * tiles >= 2 * slots && halves >= slots));
  return best;
}

// Whether the coarsest multigrid solve (nx x ny cells, nb right-hand sides) takes the two
// launches that load every matrix value ahead. Their first one runs a workgroup per mode and
// right-hand side, one on a compute unit (registers), and a round of them takes as
// long for short axes as for axes of 128 cells, whereas the three launches get
// shorter with the axes. Coarsest solve, two launches against three: 17 and 26 us at 128 x 128 x 2,
// 28 and 32 us at 128 x 128 x 4 (two rounds), 47 and 47 us at 128 x 128 x 8; 24 and 22 us at 80 x 64 x 4,
// 26 and 17 us at 64 x 32 x 8, 36 and 21 us at 96 x 32 x 8. A V-cycle of 64 right-hand sides on 256 x 256 takes
// 162 us with two launches and 96 us with three, of 128 on 128 x 128 153 and 99 us.
inline bool mg_two_launches(int64_t nx, int64_t ny, int64_t nb, int64_t cus) {
  const int64_t rounds = (nx * nb + cus - 1) / cus;
  return rounds == 1 || std::min(nx, ny) > std::min<int64_t>(32 * rounds, 96);
}

}  // namespace ppe
