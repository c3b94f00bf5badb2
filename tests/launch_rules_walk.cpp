// Checks the host's rules of csrc/launch_rules.h over sizes that no test launches.  Prints "ok", or what fails.
#include <math.h>
#include <stdio.h>

#include <random>

#include "launch_rules.h"

using namespace gpusq;

// the runs of chunks that the grid's workgroups (x, z) have, in order: they follow on each other, and cover every chunk once
static const char* prune_grid(int64_t N, int64_t K) {
  const PrunePairsGrid g = prune_pairs_grid(N, K);
  const int64_t chunks = N * (K / 8);
  if (g.y < 1 || g.y > 65535 || g.z < 1 || g.z > 65535) return "dimension";
  if (g.per_rows < 1 || 256 * g.y < g.per_rows || 256 * (g.y - 1) >= g.per_rows) return "workgroups of a run";
  if (8 * g.z * g.per_rows < chunks || 8 * (g.z - 1) * g.per_rows >= chunks) return "runs";
  if (g.per_rows == K / 2 ? ceil_div(N, 32) != g.z : g.per_rows % 256 != 0) return "whole rows or whole workgroups";
  return nullptr;
}

// every byte offset of Y, and of X's and the workspace's, at sizes small enough to compare byte by byte
static const char* operands() {
  static char space[4096];
  static float scale, other;
  for (int xb = 2; xb <= 4; xb += 2)
    for (int yb = 1; yb <= 4; yb *= 2)
      for (int at = 0; at < 600; ++at) {
        const int M = 3, N = 8, K = 16, x0 = 200, w0 = 420, range = 40;
        char met[sizeof space] = {0};
        for (int i = 0; i < M * N * yb; ++i) met[at + i] = 1;
        bool over_x = false, over_w = false;
        for (int i = 0; i < M * K * xb; ++i) over_x |= met[x0 + i];
        for (int i = 0; i < range; ++i) over_w |= met[w0 + i];
        for (int given = 0; given < 2; ++given)
          for (int own = 0; own < 2; ++own)
            for (int pass = 0; pass < 2; ++pass) {
              const bool expected = !over_x && (given || (!own && !(pass && over_w)));
              if (may_quantise_inside(space + x0, xb, space + at, yb, M, N, K, &scale, given, own ? &scale : &other, given ? nullptr : space + w0,
                                      pass ? range : 0) != expected)
                return "operands that overlap";
            }
      }
  return nullptr;
}

int main() {
  const int64_t sizes[][2] = {{1, 8}, {3, 24}, {100, 136}, {1, 504}, {5, 512}, {31, 520}, {33, 520}, {1, 33553920}, {1, 33553928}, {1, 33554432}, {1, 33554440},
                              {1, (int64_t)1 << 30}, {(int64_t)1 << 10, (int64_t)1 << 30}, {2097120, 512}, {2097121, 512}, {2147483647, 512}, {2147483647, 8},
                              {2097120, 8}, {2097152, 504}};
  for (const auto& s : sizes)
    if (const char* wrong = prune_grid(s[0], s[1])) return printf("%s: N %lld K %lld\n", wrong, (long long)s[0], (long long)s[1]), 1;
  std::mt19937_64 rng(1);
  for (int i = 0; i < 200000; ++i) {
    auto log_uniform = [&](double hi) { return (int64_t)exp2(std::uniform_real_distribution<double>(0, hi)(rng)); };
    const int64_t K = 8 * log_uniform(27), N = log_uniform(std::min(30.9, 40 - log2((double)K)));
    if (const char* wrong = prune_grid(N, K)) return printf("%s: N %lld K %lld\n", wrong, (long long)N, (long long)K), 1;
  }
  if (const char* wrong = operands()) return printf("%s\n", wrong), 1;
  printf("ok\n");
  return 0;
}
