// Rules of the host that a host program can check over sizes no test would launch.  Plain C++.
#pragma once
#include <stdint.h>

namespace gpusq {

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Grid (8, y, z) of prune_pairs_f32_kernel: workgroup (x, y, z) has chunks 256 y .. + 255 of the `per_rows` from (8 z + x) per_rows on.
// The second and third dimension count up to 65535.
struct PrunePairsGrid {
  int64_t per_rows, y, z;
};
inline PrunePairsGrid prune_pairs_grid(int64_t N, int64_t K) {
  const int64_t chunks = N * (K / 8);
  // by 4 rows; rows of fewer than 64 chunks, longer rows or more of them than the dimensions count: whole workgroups of consecutive chunks
  const bool by_rows = K / 2 >= 256 && K / 2 <= 256 * (int64_t)65535 && ceil_div(N, 32) <= 65535;
  const int64_t per_rows = by_rows ? K / 2 : 256 * ceil_div(chunks, (int64_t)256 * 8 * 65535);
  return PrunePairsGrid{per_rows, ceil_div(per_rows, 256), ceil_div(chunks, 8 * per_rows)};
}

struct ByteRange {
  const void* p;
  int64_t bytes;
};
inline bool overlap(const ByteRange& r, const ByteRange& q) {
  const uintptr_t a = (uintptr_t)r.p, b = (uintptr_t)q.p;
  return a < b + (uintptr_t)q.bytes && b < a + (uintptr_t)r.bytes;
}

// Whether the GEMM may quantise X (of x_bytes per value) itself.  The operands may overlap in ways in which only a GEMM behind a finished
// quantiser gives the same: Y over X (a square layer run on its own output) or over the partial maxima of a range pass (range_bytes of
// the workspace, 0 if there is none), which the GEMM that quantises reads in every workgroup, beside others that already write; and an
// out_scale that is the activation scale itself, which it would read while one workgroup writes it.
inline bool may_quantise_inside(const void* X, int x_bytes, const void* Y, int y_bytes, int64_t M, int64_t N, int64_t K, const float* scale,
                                bool scale_is_input, const float* out_scale, const void* workspace, int64_t range_bytes) {
  const ByteRange y{Y, M * N * y_bytes};
  if (overlap(ByteRange{X, M * K * x_bytes}, y)) return false;
  return scale_is_input || (out_scale != scale && (range_bytes == 0 || !overlap(ByteRange{workspace, range_bytes}, y)));
}

}  // namespace gpusq
