// Which rows each workgroup of the kernel for the layers behind attention (mlp.hip) takes, and how it uses its LDS: as the host plans it and as
// the kernel reads it.  Plain C++, so that a host program can walk every plan.
#pragma once
#include <stdint.h>

#include "launch_rules.h"

namespace gpusq {

constexpr int kMlpSlabs = 4;   // 16-row slabs of a workgroup at most
constexpr int kMlpMaxD = 512;  // width of a row at most: 8 wavefronts of 64 channels
constexpr int kMlpLds = 160 * 1024;

// The 16-row slabs of the rows in `chunks` chunks of `base` slabs, the first `over` of them one more; a chunk's codes lie in LDS as panels of 128 codes of
// all its rows, whole slabs of them.
struct MlpPlan {
  int chunks, base, over;
  int waves, lds;
};
struct MlpChunk {
  int64_t m0;
  int slabs;
};
__host__ __device__ inline MlpChunk mlp_chunk(const MlpPlan& p, int chunk) {
  MlpChunk r;
  r.m0 = 16 * ((int64_t)chunk * p.base + (chunk < p.over ? chunk : p.over));
  r.slabs = p.base + (chunk < p.over ? 1 : 0);
  return r;
}
inline int mlp_slabs(const MlpPlan& p) { return p.base + (p.over > 0 ? 1 : 0); }
__host__ __device__ constexpr int mlp_fragments(int64_t D) { return D > 384 ? 4 : 2; }  // 16-channel fragments of a wavefront
inline int64_t mlp_lds(int64_t D, int64_t H, int slabs) {
  const int64_t narrow = ceil_div(D, 128), wide = ceil_div(H, 128);  // (the codes of attention stand where those of the hidden layer will)
  return (narrow + (wide > narrow ? wide : narrow)) * slabs * 16 * 128;
}
inline bool mlp_takes_sizes(int64_t D, int64_t H) { return D % 64 == 0 && D >= 64 && D <= kMlpMaxD && H % 64 == 0 && H >= 64 && H <= 8 * D; }

// chunks == 0: none
inline MlpPlan mlp_plan(int64_t M, int64_t D, int64_t H, int resident) {
  MlpPlan p{};
  int most = kMlpSlabs;
  while (most > 0 && mlp_lds(D, H, most) > kMlpLds) --most;
  if (most == 0) return p;
  const int64_t slabs = ceil_div(M, 16);
  int64_t chunks = ceil_div(slabs, (int64_t)most * resident) * resident;
  if (chunks > slabs) chunks = slabs;
  p.base = (int)(slabs / chunks);
  p.over = (int)(slabs % chunks);
  p.waves = (int)(ceil_div(D / 16 / mlp_fragments(D), 4) * 4);
  p.lds = (int)mlp_lds(D, H, mlp_slabs(p));
  p.chunks = (int)chunks;
  return p;
}

}  // namespace gpusq
