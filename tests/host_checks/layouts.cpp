// Prints the tile size and the layouts (shrink tiles' kind, expand's) that the runtime
// chooses for a batch (salt_launch.h built without HIP): "M wide quad".
// Arguments: esize T C r_c n_slots sum_rank n_jobs, in and out of each, then per
// centroid id -1 .. C - 1 its tokens and its largest residual rank.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "salt_launch.h"

int main(int argc, char** argv) {
  using namespace salt;
  int at = 1;
  auto next = [&]() {
    if (at >= argc) std::exit(2);
    return std::atoi(argv[at++]);
  };
  ApplyLaunch a{};
  a.esize = next();
  a.T = next();
  a.C = next();
  a.r_c = next();
  const int n_slots = next(), sum_rank = next();
  a.n_jobs = next();
  for (int j = 0; j < a.n_jobs; ++j) {
    a.jobs[j].in = next();
    a.jobs[j].out = next();
  }
  std::vector<int> per_c(a.C + 1), rank_c(a.C + 1);
  int groups = 0, groups_c = 0;
  for (int g = 0; g <= a.C; ++g) {
    per_c[g] = next();
    rank_c[g] = next();
    groups += per_c[g] > 0;
    groups_c += g > 0 && per_c[g] > 0;
    a.r_u = std::max(a.r_u, rank_c[g]);
  }
  a.nq = std::max(1, cdiv(a.r_u, kRankChunk));
  std::vector<int4> tiles;
  BatchTiles b = cut_batch(per_c, rank_c, choose_tile_tokens(a.esize, a.T, groups, groups_c > 0), a.r_u, tiles);
  b.n_slots = n_slots;
  a.tiles = tiles.data();
  choose_layouts(a, b, sum_rank);
  std::printf("%d %d %d\n", a.M, a.wide, a.quad);
  return 0;
}
