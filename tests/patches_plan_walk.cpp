// Walks plans of the kernel for patch embeddings on images as its workgroups do (csrc/patches_plan.h): every patch in one workgroup, none higher than the
// accumulators, two workgroups' LDS to a CU; and every pair of values of a workgroup's patches, the zeros behind them included, at a place of its own inside its LDS,
// where a fragment read finds it.  Prints the number of plans, or the sizes of one that fails.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>

#include <random>
#include <vector>

#include <hip/hip_runtime_api.h>

#include "patches_plan.h"

using namespace gpusq;

static const char* walk(int64_t M, int64_t K_pad, int64_t D, int cus, bool every_byte) {
  const int64_t ksteps = ceil_div(K_pad, 64);
  const PatchPlan p = patch_plan(M, ksteps, D, cus);
  if (p.chunks == 0) return patch_lds(ksteps, 1) > kPatchLds ? nullptr : "no plan";
  if (p.slabs < 1 || p.slabs > kPatchSlabs) return "height";
  if ((int64_t)p.chunks * 16 * p.slabs < M || ((int64_t)p.chunks - 1) * 16 * p.slabs >= M) return "patches not covered, or a workgroup without one";
  if (p.units * 64 != D || p.ksteps * 64 < K_pad || (p.ksteps - 1) * 64 >= K_pad) return "units or K steps";
  if (patch_lds(p.ksteps, p.slabs) > kPatchLds) return "LDS";
  if (!every_byte) return nullptr;
  std::vector<uint8_t> met((size_t)patch_lds(p.ksteps, p.slabs), 0);
  for (int r = 0; r < 16 * p.slabs; ++r)
    for (uint32_t kb = 0; kb < (uint32_t)p.ksteps * 128; kb += 4) {
      const uint32_t at = patch_lds_at(kb, r, patch_swizzle(r), p.slabs);
      if (at + 4 > met.size() || met[at]) return "a pair outside, or on another";
      met[at] = 1;
      // slab r / 16, lane (kb / 16 % 4) 16 + r % 16, half kb / 64 % 2 of a fragment read, as the kernel computes it
      const int lane = (int)(kb / 16 % 4) * 16 + r % 16;
      const uint32_t lo = (uint32_t)((lane & 15) * 128 + (((lane >> 4) ^ ((lane & 15) >> 1)) << 4));
      if (kb / 128 * (uint32_t)(p.slabs * 2048) + (uint32_t)(r / 16) * 2048 + (kb & 64 ? lo ^ 64u : lo) + kb % 16 != at) return "not where a fragment read looks";
    }
  return nullptr;
}

int main(int argc, char** argv) {
  const int plans = argc > 1 ? atoi(argv[1]) : 1000;
  const int cus[] = {256, 64, 304, 8, 100, 1};
  std::mt19937_64 rng(1);
  for (int i = 0; i < plans; ++i) {
    const auto log_of = [&](double lo, double hi) { return (int64_t)llround(exp(std::uniform_real_distribution<double>(log(lo), log(hi))(rng))); };
    const int64_t M = log_of(1, 2e9), K_pad = 16 * log_of(1, 200), D = 64 * log_of(1, 100);
    const int c = cus[i % 6];
    if (const char* what = walk(M, K_pad, D, c, i % 100 == 0)) {
      printf("%s: M %lld K_pad %lld D %lld on %d CUs\n", what, (long long)M, (long long)K_pad, (long long)D, c);
      return 1;
    }
  }
  printf("%d plans\n", plans);
  return 0;
}
