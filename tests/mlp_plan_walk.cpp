// Walks plans of the kernel for the layers behind attention as its workgroups do (csrc/mlp_plan.h): the chunks cover every row exactly once in
// whole slabs, none without a row, none higher than the kernel's accumulators, and their codes fit the LDS; the wavefronts have the narrow layers' channels.
// Prints the number of plans, or the sizes of one that fails.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>

#include <random>

#include <hip/hip_runtime_api.h>

#include "mlp_plan.h"

using namespace gpusq;

static const char* walk(int64_t M, int64_t D, int64_t H, int cus) {
  const MlpPlan p = mlp_plan(M, D, H, cus);
  if (p.chunks == 0) return mlp_lds(D, H, 1) > kMlpLds ? nullptr : "no plan";
  int64_t next = 0;
  for (int c = 0; c < p.chunks; ++c) {
    const MlpChunk k = mlp_chunk(p, c);
    if (k.m0 != next || k.m0 >= M) return "rows left out, met twice, or none";
    if (k.slabs < 1 || k.slabs > kMlpSlabs || k.slabs > mlp_slabs(p) || k.slabs < mlp_slabs(p) - 1) return "height";
    if (mlp_lds(D, H, k.slabs) > p.lds) return "LDS of a chunk";
    next += 16 * k.slabs;
  }
  if (next < M) return "rows not covered";
  if (p.lds > kMlpLds) return "LDS";
  const int F = mlp_fragments(D), ksteps = (int)ceil_div(D, 128);
  if (p.waves % 4 != 0 || p.waves * 16 * F < D || (p.waves - 4) * 16 * F >= D) return "wavefronts";
  if (64 * p.waves > (F == 4 || ksteps < 3 ? 512 : 768)) return "launch bounds";
  if ((F == 4) != (ksteps == 4)) return "instantiation";
  return nullptr;
}

int main(int argc, char** argv) {
  const int plans = argc > 1 ? atoi(argv[1]) : 1000;
  const int cus[] = {256, 64, 304, 8, 100, 1};
  std::mt19937_64 rng(1);
  for (int i = 0; i < plans; ++i) {
    const int64_t M = (int64_t)exp2(std::uniform_real_distribution<double>(0, i % 16 ? 17 : 24)(rng)), D = 64 * (1 + (int64_t)(rng() % 8)), H = 64 * (1 + (int64_t)(rng() % (D / 8)));
    if (!mlp_takes_sizes(D, H)) continue;
    if (const char* wrong = walk(M, D, H, cus[i % 6])) {
      printf("%s: M %lld D %lld H %lld cus %d\n", wrong, (long long)M, (long long)D, (long long)H, cus[i % 6]);
      return 1;
    }
  }
  printf("%d plans\n", plans);
  return 0;
}
