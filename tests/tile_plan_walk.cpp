// Walks plans of the tile kernel with one workgroup per CU as its workgroups do (csrc/even_plan.h): every tile is met exactly
// once, the tiles of every 256-channel block cover every row exactly once, and no tile is higher than the kernel's accumulators or
// of a height its K loops do not have.  Prints the number of plans, or the sizes of one that fails.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>

#include <random>
#include <vector>

#include <hip/hip_runtime_api.h>

#include "even_plan.h"

using namespace gpusq;

static const char* walk(int64_t M, int64_t N, int cus, int ksteps, bool gelu) {
  const EvenPlan p = even_plan(M, N, cus, ksteps, gelu);
  const int64_t total = even_total(p), blocks = (N + kTileBN - 1) / kTileBN, units = (M + 31) / 32;
  const int grid = 8 * p.grid8;
  if (p.tiles_n != blocks) return "channel blocks";
  if (grid < 8 || grid > (cus + 7) / 8 * 8 || grid - 8 >= total) return "grid";
  const int loops = (even_units(p) + 1) / 2;  // a wavefront has a loop for this many slabs and for one less
  if (loops < 1 || loops > 4) return "height";
  std::vector<char> met(total, 0);
  std::vector<int64_t> rows(blocks, 0);  // each block's tiles, taken in order, continue where the last one ended
  for (int place = 0; place < grid; ++place) {
    const int items = p.rounds + (place < p.last_round ? 1 : 0);
    for (int i = 0; i < items; ++i) {
      const int64_t t = (int64_t)i * grid + place;
      if (t >= total || met[t]) return "tile met twice or outside the plan";
      met[t] = 1;
    }
  }
  for (int64_t t = 0; t < total; ++t) {
    if (!met[t]) return "tile not met";
    const EvenTile e = even_tile(p, (int)t);
    if (e.n_blk != t % blocks) return "channel block of a tile";
    if (e.m0 != rows[e.n_blk] * 32 || e.m0 >= M) return "first row of a tile";
    const int most = (e.slabs + 3) / 4, least = e.slabs / 4;  // slabs of a wavefront
    if (e.slabs < 2 || most > loops || (loops > 1 && least < loops - 1)) return "slabs of a tile";
    rows[e.n_blk] += e.slabs / 2;
  }
  for (int64_t b = 0; b < blocks; ++b)
    if (rows[b] < units) return "rows not covered";
  return nullptr;
}

int main(int argc, char** argv) {
  const int plans = argc > 1 ? atoi(argv[1]) : 1000;
  const int cus[] = {256, 64, 304, 8, 100, 1};
  std::mt19937_64 rng(1);
  auto log_uniform = [&](double hi) { return (int64_t)exp2(std::uniform_real_distribution<double>(0, hi)(rng)); };
  for (int i = 0; i < plans; ++i) {
    int64_t M = log_uniform(17), N = 4 * log_uniform(i % 8 ? 11 : 15);
    if (i % 3 == 0) M = (M + 31) / 32 * 32;
    if (M * N > ((int64_t)1 << 31)) M = ((int64_t)1 << 31) / N + 1;
    const int ksteps = (int)log_uniform(8), c = cus[i % 6];
    const char* wrong = walk(M, N, c, ksteps, i & 1);
    if (wrong) {
      printf("%s: M %lld N %lld cus %d ksteps %d gelu %d\n", wrong, (long long)M, (long long)N, c, ksteps, i & 1);
      return 1;
    }
  }
  printf("%d plans\n", plans);
  return 0;
}
