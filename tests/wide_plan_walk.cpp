// Walks plans of the kernel that quantises whole rows as its workgroups do (csrc/wide_plan.h): every row chunk of every column block is met
// exactly once, the chunks cover every row exactly once and are no higher than the kernel's accumulators, the column blocks cover every
// channel and fit a workgroup, and the workgroups of a CU fit its LDS.  Prints the number of plans, or the sizes of one that fails.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <random>
#include <vector>

#include <hip/hip_runtime_api.h>

#include "wide_plan.h"

using namespace gpusq;

static const char* walk(int64_t M, int64_t N, int cus, bool fp32) {
  const WidePlan p = wide_plan(M, N, cus, fp32);
  if (p.chunks == 0) return cus / 8 >= p.tiles_n ? "no plan" : nullptr;
  if (p.blocks < 1 || p.blocks > kWideBlocks || (int64_t)p.tiles_n * p.blocks * 64 < N || (int64_t)(p.tiles_n - 1) * p.blocks * 64 >= N) return "column blocks";
  if (p.base < 1 || wide_slabs(p) < 1 || wide_slabs(p) > kWideSlabs) return "height";
  if (wide_lds(wide_slabs(p), fp32) > 160 * 1024) return "LDS";
  std::vector<std::vector<std::pair<int64_t, int>>> met(p.tiles_n);
  for (int w = 0; w < 8 * p.per_xcd; ++w) {
    const WidePlace at = wide_place(p, w);
    if (at.n_blk < 0 || at.n_blk >= p.tiles_n) return "column block of a workgroup";
    if (w == 0 && at.items == 0) return "the first workgroup, which writes the scale, has nothing to do";
    for (int i = 0; i < at.items; ++i) {
      const WideChunk c = wide_chunk(p, at, i);
      if (c.rows < 1 || c.rows > 16 * wide_slabs(p)) return "rows of a chunk";
      met[at.n_blk].push_back({c.m0, c.rows});
    }
  }
  for (auto& block : met) {
    std::sort(block.begin(), block.end());
    int64_t next = 0;
    for (const auto& c : block) {
      if (c.first != next) return "a chunk met twice, or rows left out";
      next += c.second;
    }
    if (next != M) return "rows not covered";
  }
  return nullptr;
}

int main(int argc, char** argv) {
  const int plans = argc > 1 ? atoi(argv[1]) : 1000;
  const int cus[] = {256, 64, 304, 8, 100, 1};
  std::mt19937_64 rng(1);
  auto log_uniform = [&](double hi) { return (int64_t)exp2(std::uniform_real_distribution<double>(0, hi)(rng)); };
  for (int i = 0; i < plans; ++i) {
    const int64_t M = log_uniform(i % 16 ? 17 : 22), N = 4 * log_uniform(i % 8 ? 10 : 14);
    const int c = cus[i % 6];
    if (const char* wrong = walk(M, N, c, i & 1)) {
      printf("%s: M %lld N %lld cus %d fp32 %d\n", wrong, (long long)M, (long long)N, c, i & 1);
      return 1;
    }
  }
  printf("%d plans\n", plans);
  return 0;
}
