// How the kernel for patch embeddings on images (patches.hip) splits the patches and where their values lie in LDS: as the host plans it and
// as the kernel reads it.  Plain C++, so that a host program can walk every plan.
#pragma once
#include <stdint.h>

#include "launch_rules.h"

namespace gpusq {

constexpr int kPatchThreads = 256;
constexpr int kPatchSlabs = 4;          // 16-patch slabs of a workgroup at most
constexpr int kPatchLds = 80 * 1024;    // two workgroups to a CU
constexpr int kPatchPanelBytes = 128;   // of a patch in a panel: one K step

// Workgroup c has the patches 16 slabs c .. + 16 slabs - 1; `units` blocks of 64 channels.
struct PatchPlan {
  int chunks, slabs, units, ksteps;
};
inline int64_t patch_lds(int64_t ksteps, int slabs) { return ksteps * 16 * slabs * kPatchPanelBytes; }
// Byte kb (even) of the flattened patch r of a workgroup: panels of one K step of all its patches, 16-byte piece c of a patch at c ^ ((r >> 1) & 7)
__host__ __device__ inline uint32_t patch_swizzle(int r) { return (uint32_t)(r >> 1 & 7) << 4; }
__host__ __device__ inline uint32_t patch_lds_at(uint32_t kb, int r, uint32_t swizzle, int slabs) {
  return (uint32_t)r * kPatchPanelBytes + (kb / kPatchPanelBytes) * (uint32_t)(16 * slabs * kPatchPanelBytes) + ((kb % kPatchPanelBytes) ^ swizzle);
}

// Whether the kernel takes the sizes: whole pairs of pixels, whole blocks of 64 channels, lane offsets of 32 bits inside the images and 64 rows of Y
inline bool patch_takes_sizes(int x_bytes, int64_t B, int64_t C, int64_t H, int64_t W, int64_t P, int64_t ksteps, int64_t D) {
  return P % 2 == 0 && D % 64 == 0 && D < ((int64_t)1 << 24) && B * C * H * W * x_bytes < ((int64_t)1 << 32) && patch_lds(ksteps, 1) <= kPatchLds;
}
// chunks == 0: none.  Workgroups as high as they go, for each reads all weights, but no higher than gives every CU one, or where that takes more than
// the accumulators two (23040 x 588 -> 768 with 3 slabs 23.5 us, with 4 24.9); behind that round the chunks even out over the CUs by themselves, and the
// highest are ahead (44000 x 588 -> 768 with 4 slabs 42.7, with 3 46.8).
inline int patch_slabs(int64_t ksteps) {
  const int64_t fit = kPatchLds / patch_lds(ksteps, 1);
  return (int)(fit < kPatchSlabs ? fit : kPatchSlabs);
}
inline PatchPlan patch_plan(int64_t M, int64_t ksteps, int64_t D, int resident) {
  PatchPlan p{};
  const int64_t slabs = ceil_div(M, 16);
  const int most = patch_slabs(ksteps);
  if (most == 0) return p;
  const int64_t even = ceil_div(slabs, slabs <= (int64_t)most * resident ? resident : 2 * (int64_t)resident);
  p.slabs = (int)(even < most ? even : most);
  p.chunks = (int)ceil_div(slabs, p.slabs);
  p.units = (int)(D / 64);
  p.ksteps = (int)ksteps;
  return p;
}

}  // namespace gpusq
