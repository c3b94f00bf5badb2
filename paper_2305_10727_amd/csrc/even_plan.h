// The tile decomposition of the tile kernel with one workgroup per CU (tile1.h): which rows and channels each workgroup takes,
// as the host plans it and as the kernel reads it.  Plain C++, so that a host program can walk every plan.
#pragma once
#include <stdint.h>

namespace gpusq {

constexpr int kTileBN = 256;  // output channels of a tile = one packed weight tile

// The tiles of a launch of the kernel with one workgroup per CU: the rows in chunks of whole 32-row units, the first `higher` of
// them a unit higher than the others, times the 256-channel blocks (n fastest); behind them, perhaps, tail chunks of
// `tail_units`.  Round i takes the tiles from i * grid on, in runs of grid / 8 to an XCD, so that tiles that share an X slab
// meet in one L2.  The higher ones all come in the first round or rounds: no workgroup meets more of them than another by more
// than one.  (What a workgroup begins with, it executes from a cold instruction cache and scalar cache: with the higher chunks
// spread over the XCDs, which took it sixty more instructions or another line of kernel arguments, every launch took 1.4 us
// longer.)
struct EvenPlan {
  int tiles_n, chunks;
  int units, higher;
  int tail_chunks, tail_units;
  uint32_t inv;  // tile / tiles_n = (tile * inv >> 32) >> shift for tiles below 2^31 (Granlund & Montgomery 1994); tiles_n = 1: unused
  int shift;
  int rounds, last_round;  // whole rounds of tiles; tiles behind them
  int grid8;               // grid / 8
};
struct EvenTile {
  int n_blk, slabs;  // height in slabs of 16 rows
  int64_t m0;
};
inline int even_units(const EvenPlan& p) { return p.units + (p.higher > 0); }  // of the highest tile
inline int64_t even_total(const EvenPlan& p) { return (int64_t)(p.chunks + p.tail_chunks) * p.tiles_n; }
__host__ __device__ inline EvenTile even_tile(const EvenPlan& p, int idx) {
  const int chunk = p.tiles_n > 1 ? (int)((uint32_t)(((uint64_t)(uint32_t)idx * p.inv) >> 32) >> p.shift) : idx;
  const int over = chunk - p.chunks;  // >= 0: in the tail
  EvenTile t;
  t.n_blk = idx - chunk * p.tiles_n;
  t.slabs = 2 * (over < 0 ? p.units + (chunk < p.higher ? 1 : 0) : p.tail_units);
  const int main = over < 0 ? chunk : p.chunks, tail = over < 0 ? 0 : over;
  t.m0 = (int64_t)(main * p.units + (main < p.higher ? main : p.higher) + tail * p.tail_units) * 32;  // (units of 32 rows: below 2^26)
  return t;
}

inline int64_t plan_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// The plan the tile kernel with one workgroup per CU runs.  For each number of rounds over the CUs from the fewest
// (tiles of at most 8 units of 32 rows) on: as many chunks as fill them.  Where the rows are a few more than whole rounds of the
// highest tiles: those, and the rest in tail chunks.  The shortest estimate wins (microseconds, fitted to timings of every plan of
// sixteen layers' sizes on MI355X): a K step of u units takes 0.24 + 0.113 u and no less than 0.41, so rows spread over more
// rounds cost 0.24 per K step and round.  A tail tile's K steps are those of a lone workgroup, and part of its time vanishes
// in the 5 % by which the workgroups' ends differ anyway (65792 x 5120 -> 1280: 6 even rounds 291 us, 5 and a tail 269).
inline EvenPlan even_plan(int64_t M, int64_t N, int resident, int ksteps, bool gelu) {
  constexpr int kTallest = 8, kTail = 6;  // (a tail tile is one that the loop for tiles of 7 and 8 units can run)
  const int tiles_n = (int)plan_div(N, kTileBN);
  const int64_t units = plan_div(M, 32);
  const double epi_unit = gelu ? 0.5 : 0.3;
  auto round_cost = [&](double u) {
    const double step = 0.24 + 0.113 * u;
    return ksteps * (step > 0.41 ? step : 0.41) + 0.3 + epi_unit * u;
  };
  EvenPlan best{};
  double best_cost = -1;
  auto consider = [&](int64_t main_units, int64_t chunks, int64_t tail_units, double cost) {
    if (best_cost >= 0 && cost >= best_cost) return;
    best_cost = cost;
    best.tiles_n = tiles_n;
    best.chunks = (int)chunks;
    best.units = (int)(main_units / chunks);
    best.higher = (int)(main_units % chunks);
    best.tail_units = kTail;
    best.tail_chunks = (int)plan_div(tail_units, kTail);
  };
  const int64_t least = plan_div(plan_div(units, kTallest) * tiles_n, resident);
  for (int64_t rounds = least; rounds <= least + 2; ++rounds) {
    int64_t chunks = rounds * resident / tiles_n;  // (>= units / kTallest)
    if (chunks > units) chunks = units;
    const int64_t r = plan_div(chunks * tiles_n, resident);
    // what the workgroup with the most higher tiles has
    const int64_t most = r * (units / chunks) + plan_div((units % chunks) * tiles_n, resident);
    consider(units, chunks, 0, r * round_cost((double)most / r));
  }
  const int64_t whole = (least - 1) * resident / tiles_n;  // chunks of the highest tiles that fill the rounds but the last
  const int64_t rest = units - whole * kTallest;
  if (least >= 4 && whole > 0 && rest > 0 && plan_div(rest, kTail) * tiles_n <= resident) {
    const double all = (least - 1) * round_cost(kTallest), tail = ksteps * 0.5 + 0.3 + epi_unit * kTail - 0.05 * all;
    consider(whole * kTallest, whole, rest, all + (tail > 0 ? tail : 0));
  }
  const int64_t total = even_total(best);
  best.grid8 = (int)plan_div(total < resident ? total : resident, 8);  // one workgroup per CU, never more workgroups than tiles
  best.rounds = (int)(total / (8 * best.grid8));
  best.last_round = (int)(total % (8 * best.grid8));
  int log2 = 1;
  while (((int64_t)1 << log2) < tiles_n) ++log2;
  best.shift = log2 - 1;
  best.inv = tiles_n > 1 ? (uint32_t)(((uint64_t)1 << (31 + log2)) / tiles_n + ((((uint64_t)1 << (31 + log2)) % tiles_n) != 0)) : 0u;
  return best;
}

}  // namespace gpusq
