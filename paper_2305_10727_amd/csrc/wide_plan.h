// Which rows and channels each workgroup of the kernel for whole rows (wide.hip) takes, as the host plans it and as the kernel reads
// it.  Plain C++, so that a host program can walk every plan.
#pragma once
#include <stdint.h>

#include "launch_rules.h"

namespace gpusq {

constexpr int kWideWaves = 16, kWideBlocks = kWideWaves - 4;  // wavefronts of a workgroup at most; 64-channel blocks at most
constexpr int kWideSlabs = 4;                                 // 16-row slabs of a chunk at most

// Rows in `chunks` chunks of `base` rows, the first `over` of them one more.  The workgroups of an XCD are tiles_n to a lane of chunks
// (so that those which share rows of X meet in one L2): lane l takes chunks l, l + lanes, ...
struct WidePlan {
  int tiles_n, blocks;      // column blocks; 64-channel blocks in each
  int per_xcd, lanes_xcd;   // workgroups and lanes of chunks of an XCD
  int chunks, base, over;
};
struct WidePlace {
  int n_blk, lane, items;
};
struct WideChunk {
  int64_t m0;
  int rows;
};
inline int wide_slabs(const WidePlan& p) { return (p.base + (p.over > 0 ? 1 : 0) + 15) / 16; }
__host__ __device__ inline WidePlace wide_place(const WidePlan& p, int workgroup) {
  const int j = workgroup >> 3;
  WidePlace r;
  r.n_blk = j % p.tiles_n;
  r.lane = (workgroup & 7) * p.lanes_xcd + j / p.tiles_n;
  const int lanes = 8 * p.lanes_xcd;
  r.items = r.lane < p.chunks ? (p.chunks - r.lane + lanes - 1) / lanes : 0;
  return r;
}
__host__ __device__ inline WideChunk wide_chunk(const WidePlan& p, const WidePlace& at, int item) {
  const int c = at.lane + item * 8 * p.lanes_xcd;
  WideChunk r;
  r.m0 = (int64_t)c * p.base + (c < p.over ? c : p.over);
  r.rows = p.base + (c < p.over ? 1 : 0);
  return r;
}

// LDS of a workgroup: X as it is in memory, kWideDepth K steps of it, two buffers of codes, the constants of every channel.
constexpr int kWideDepth = 3;
inline int wide_lds(int slabs, bool fp32) { return 1024 * (kWideDepth * slabs * (fp32 ? 8 : 4) + 4 * slabs) + kWideBlocks * 64 * 8 + 128; }

// The plan of chunks of at most `slabs` slabs.  chunks == 0: none (fewer than 8 workgroups to a column block).
inline WidePlan wide_plan_of(int64_t M, int64_t N, int resident, int slabs, bool fp32) {
  WidePlan p{};
  const int64_t all = ceil_div(N, 64);
  p.tiles_n = (int)ceil_div(all, kWideBlocks);
  p.blocks = (int)ceil_div(all, p.tiles_n);
  const int by_waves = kWideWaves / (4 + p.blocks), by_lds = 160 * 1024 / wide_lds(slabs, fp32);
  p.lanes_xcd = resident / 8 * (by_waves < by_lds ? by_waves : by_lds) / p.tiles_n;
  p.per_xcd = p.lanes_xcd * p.tiles_n;
  if (p.lanes_xcd < 1) return p;
  const int64_t lanes = 8 * (int64_t)p.lanes_xcd;
  const int64_t rounds = ceil_div(M, lanes * 16 * slabs);
  int64_t chunks = rounds * lanes;
  if (chunks > ceil_div(M, 16)) chunks = ceil_div(M, 16);
  p.chunks = (int)chunks;
  p.base = (int)(M / chunks);
  p.over = (int)(M % chunks);
  return p;
}
// Chunks as high as they go (64 rows are 2 % behind the best of 16, 32, 48 and 64 of each of 1381 sizes), but for many fp32 rows of up to 256
// channels, of which LDS then holds one workgroup to a CU: 32 rows are 2 to 7 % ahead there.
inline WidePlan wide_plan(int64_t M, int64_t N, int resident, bool fp32) {
  return wide_plan_of(M, N, resident, fp32 && N <= 256 && M >= 8192 ? 2 : kWideSlabs, fp32);
}

// Run time in microseconds of that kernel, without the range pass, and of the quantiser and a GEMM of `gemm_us` behind it: fitted to 2448 sizes
// timed on MI355X (M 2048 ... 65792, K 64 ... 5120, N 64 ... 1536, fp16 and fp32, both outputs, with and without GELU, three buffers in turn; 9 % and
// 8 %, on 14022 others 10 % and 10 %).  A K step of the former is a chain of 0.4 us, or what its operands take on their way into the CU and its codes in the vector units,
// shared by the workgroups on a CU.
inline double wide_us(const WidePlan& p, int64_t M, int64_t N, int64_t K, int resident, bool fp32, bool gelu, bool int8_out) {
  const int slabs = wide_slabs(p), lanes = 8 * p.lanes_xcd;
  const int64_t rounds = ceil_div(p.chunks, lanes), groups = (int64_t)(p.chunks < lanes ? p.chunks : lanes) * p.tiles_n;
  const double sharing = groups > resident ? (double)groups / resident : 1.0;
  const double work = sharing * (0.18 + 0.019 * p.blocks + 0.015 * slabs * p.blocks + (fp32 ? 0.115 : 0.061) * slabs);
  const double chunk = (double)ceil_div(K, 128) * (work > 0.395 ? work : 0.395) + 0.5 * slabs * (1.0 + (gelu ? 0.9 : 0.0) + (int8_out ? 0.5 : 0.0));
  const double bytes = (double)M * K * (fp32 ? 5 : 3) + (double)M * N * (int8_out ? 1 : 2);
  return 3.8 + (rounds * chunk > bytes / 5.0e6 ? rounds * chunk : bytes / 5.0e6);
}
inline double quantise_and_gemm_us(double gemm_us, int64_t M, int64_t N, int64_t K, bool fp32, bool int8_out) {
  const double pass = 2.2 + (double)M * K * (fp32 ? 5 : 3) / 5.83e6;
  return 1.3 + (pass > 2.8 ? pass : 2.8) + 0.9 * gemm_us + (int8_out ? 0.48e-7 * M * N : 0.0);
}
// Of that estimate, how much the other may be at most for the kernel for whole rows to be taken; smaller than 1 by what the estimates miss (their ratio is
// off by 10 %, one standard deviation; a long K is estimated 8 % short).
inline double wide_margin(int64_t K, bool fp32) { return K > 24 * 128 ? 0.9 : (fp32 ? 0.92 : 0.97); }
// Behind a range pass the quantiser is faster than those estimates, which are of a given scale: what the pass read last it finds in the L2s (32 MB),
// and all of X in the last level cache (256 MB) where the codes leave it there.  Where that decides (of 20022 sizes timed with either, X and Y in MB):
//   one block of channels, up to 3 K steps, X beyond 6: whole rows slower in most fp32 sizes, whatever the estimates, in half of fp16 from a ratio of 0.88 on
//   fp32, Y below 30, X of 9 to 48, or more than 12 K steps: level from a ratio of 0.85 on
//   fp16, X of 115 to 160 (with the codes 172 to 240): level from 0.8 on for a ragged K, whose codes whole rows leave in the caches as well, from
//   0.86 on for a Y of 10 to 30; elsewhere 10 % ahead
inline double wide_margin_behind_range(int64_t M, int64_t N, int64_t K, bool fp32, bool int8_out) {
  const double x = (double)M * K * (fp32 ? 4e-6 : 2e-6), y = (double)M * N * (int8_out ? 1e-6 : 2e-6), margin = wide_margin(K, fp32);
  double most = margin;
  if (N <= 64 && K <= 3 * 128 && x > 6)
    most = fp32 ? 0.7 : 0.88;
  else if (fp32 && y < 30 && ((x > 9 && x < 48) || K > 12 * 128))
    most = 0.85;
  else if (!fp32 && x > 115 && x < 160 && K % 128 != 0)
    most = 0.8;
  else if (!fp32 && x > 115 && x < 160 && y > 10 && y < 30)
    most = 0.86;
  return most < margin ? most : margin;
}

}  // namespace gpusq
