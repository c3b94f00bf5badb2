// INT4 operands in the pair-wise 4:8 pattern [Sec. 3.1, paragraph on the INT4 instruction]: pruning, compressed storage
// (4 kept 4-bit values + two 2-bit indices per chunk of 8) and the decode to INT8 that feeds the multiply-accumulate.
// gfx950 has no 4-bit integer matrix instruction and the pattern is not a 2:4 pattern (both kept sub-chunks of a chunk may
// lie in the same group of 4), so the product itself runs on the dense INT8 kernel over the decoded operand; what the
// format buys on this hardware is the storage: 2.5 bits per weight in HBM and on disk.
// All kernels stream their operands once (HBM-bound); one thread handles two chunks (16 dense elements).
#include "common.h"

namespace gpusq {

// ---------------------------------------------------------------------------------------------------------- prune
// Score of a sub-chunk (a, b): |a| + |b| in fp32, compared as a sign-cleared bit pattern (a total order); the two highest
// scores are kept, ties to the lower index: the rule of the 2:4 pattern applied to the four sub-chunks.
__device__ __forceinline__ unsigned pair_key(float a, float b) { return __float_as_uint(fabsf(a) + fabsf(b)) & 0x7FFFFFFFu; }

// one_per_group: of the two kept sub-chunks one lies in each group of 4 (the better of its two; ties: the lower index),
// which makes the row a 2:4 row as well: the form that the sparse matrix instructions of this hardware can consume.
// A thread per chunk.  Grid (8, S, R): S workgroups share 4 rows (`per_rows` chunks), and those of rows 4 (8z + x) .. + 3 run on XCD x (ids are
// dealt out to the XCDs in turn, x fastest), as the row quantiser's do, which comes next as a rule and then finds the pruned rows in the L2
// of its XCD.  Both, us: 3072 x 768 12.1 -> 8.4, 768 x 3072 13.0 -> 9.9, 5120 x 1280 20.1 -> 18.7.  (W read past the L2s, with the non-temporal hint: the
// pass itself 10.6 -> 12.6.)
__global__ void __launch_bounds__(256) prune_pairs_f32_kernel(const float4* __restrict__ in, float4* __restrict__ out,
                                                              uint8_t* __restrict__ mask, int one_per_group, int64_t chunks, int64_t per_rows) {
  const int64_t in_rows = (int64_t)blockIdx.y * 256 + threadIdx.x, c = ((int64_t)blockIdx.z * 8 + blockIdx.x) * per_rows + in_rows;
  if (in_rows >= per_rows || c >= chunks) return;
  const float4 lo = in[2 * c], hi = in[2 * c + 1];
  const unsigned k0 = pair_key(lo.x, lo.y), k1 = pair_key(lo.z, lo.w), k2 = pair_key(hi.x, hi.y), k3 = pair_key(hi.z, hi.w);
  const unsigned m = one_per_group ? ((k1 > k0 ? 2u : 1u) | (k3 > k2 ? 8u : 4u)) : keep_mask_of_4(k0, k1, k2, k3);
  float4 o0, o1;
  o0.x = (m & 1u) ? lo.x : 0.0f; o0.y = (m & 1u) ? lo.y : 0.0f;
  o0.z = (m & 2u) ? lo.z : 0.0f; o0.w = (m & 2u) ? lo.w : 0.0f;
  o1.x = (m & 4u) ? hi.x : 0.0f; o1.y = (m & 4u) ? hi.y : 0.0f;
  o1.z = (m & 8u) ? hi.z : 0.0f; o1.w = (m & 8u) ? hi.w : 0.0f;
  out[2 * c] = o0;
  out[2 * c + 1] = o1;
  if (mask) mask[c] = (uint8_t)m;
}

gpusq_status launch_prune_pairs(const float* Win, float* Wout, uint8_t* mask, int one_per_group, int64_t N, int64_t K, hipStream_t s) {
  const PrunePairsGrid g = prune_pairs_grid(N, K);
  const dim3 grid(8, (unsigned)g.y, (unsigned)g.z);
  prune_pairs_f32_kernel<<<grid, 256, 0, s>>>((const float4*)Win, (float4*)Wout, mask, one_per_group, N * (K / 8), g.per_rows);
  return check_launch();
}

// ---------------------------------------------------------------------------------------------------------- compress
// One chunk: 8 codes in two words (little endian) -> 16 bits of values (kept code j in nibble j) + the index nibble.
// COUNT: `bad` counts a chunk with a third non-zero sub-chunk or a code outside -8 .. 7.
template <bool COUNT>
__device__ __forceinline__ void compress_chunk(unsigned w0, unsigned w1, unsigned& vals16, unsigned& nib, int& bad) {
  // |a| + |b| of each sub-chunk: the sum of absolute differences of code + 128 and 128 over four bytes, two of them 128
  const unsigned z0 = w0 ^ 0x80808080u, z1 = w1 ^ 0x80808080u;
  auto key_of = [](unsigned pair) { return __builtin_amdgcn_sad_u8(pair, 0x80808080u, 0u); };
  const unsigned k0 = key_of((z0 & 0xFFFFu) | 0x80800000u), k1 = key_of((z0 >> 16) | 0x80800000u);
  const unsigned k2 = key_of((z1 & 0xFFFFu) | 0x80800000u), k3 = key_of((z1 >> 16) | 0x80800000u);
  // the selection rule of keep_mask_of_4 on lane masks, as KeptPair has it (through one struct for both the pass takes 4 % longer: 5120 x 1280
  // 3.36 -> 3.53 us)
  const bool c01 = k1 > k0, c02 = k2 > k0, c03 = k3 > k0, c12 = k2 > k1, c13 = k3 > k1, c23 = k3 > k2;
  auto two_of = [](bool p, bool q, bool r) { return (p & q) | (r & (p | q)); };
  const bool keep0 = !two_of(c01, c02, c03), keep1 = !two_of(!c01, c12, c13), keep2 = !two_of(!c02, !c12, c23);
  const bool keep3 = !two_of(!c03, !c13, !c23);
  const unsigned p0 = keep0 ? 0u : (keep1 ? 1u : 2u), p1 = keep3 ? 3u : (keep2 ? 2u : 1u);
  nib = p0 | (p1 << 2);
  // the two kept sub-chunks side by side, then the low nibbles of their four bytes
  const unsigned a = keep0 ? w0 : (keep1 ? w0 >> 16 : w1), b = keep3 ? w1 >> 16 : (keep2 ? w1 : w0 >> 16);
  const unsigned v = ((a & 0xFFFFu) | (b << 16)) & 0x0F0F0F0Fu, n = v | (v >> 4);
  vals16 = (n & 0xFFu) | ((n >> 8) & 0xFF00u);
  if constexpr (COUNT) {
    int out_of_range = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = (int)(int8_t)(w0 >> (8 * i)), d = (int)(int8_t)(w1 >> (8 * i));
      out_of_range |= (c < -8) | (c > 7) | (d < -8) | (d > 7);
    }
    bad += (int)((!keep0 && k0 != 0) || (!keep1 && k1 != 0) || (!keep2 && k2 != 0) || (!keep3 && k3 != 0) || out_of_range);
  }
}

__device__ __forceinline__ void add_count(int32_t* total, int bad) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) bad += __shfl_xor(bad, o, 64);
  if ((threadIdx.x & 63) == 0 && bad) atomicAdd(total, bad);
}

__global__ void __launch_bounds__(256) compress_int4_kernel(const int8_t* __restrict__ W, uint8_t* __restrict__ values,
                                                            uint8_t* __restrict__ meta, int32_t* __restrict__ violations,
                                                            int64_t N, int64_t K) {
  const int64_t chunks_per_row = K / 8;
  const int64_t mrb = (chunks_per_row + 1) / 2;
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int bad = 0;
  if (id < N * mrb) {
    const int64_t n = id / mrb, b = id % mrb;
    unsigned byte = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t c = 2 * b + h;
      if (c < chunks_per_row) {
        const uint2 w = *(const uint2*)(W + n * K + 8 * c);  // rows and chunks are 8-byte aligned (K % 8 == 0)
        unsigned vals16, nib;
        compress_chunk<true>(w.x, w.y, vals16, nib, bad);
        *(uint16_t*)(values + n * (K / 4) + 2 * c) = (uint16_t)vals16;
        byte |= nib << (4 * h);
      }
    }
    meta[n * mrb + b] = (uint8_t)byte;
  }
  if (violations) add_count(violations, bad);
}

// The same for a flat run of an even number of chunks (no row of indices ends inside a byte): two chunks per thread, one
// 16-byte load, and no division by the row length (5120 x 1280: 4.9 -> 3.4 us).
template <bool COUNT>
__global__ void __launch_bounds__(256) compress_int4_flat_kernel(const uint4* __restrict__ W, uint32_t* __restrict__ values,
                                                                 uint8_t* __restrict__ meta, int32_t* __restrict__ violations, int64_t pairs) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int bad = 0;
  if (id < pairs) {
    const uint4 w = W[id];
    unsigned v[2], nib[2];
    compress_chunk<COUNT>(w.x, w.y, v[0], nib[0], bad);
    compress_chunk<COUNT>(w.z, w.w, v[1], nib[1], bad);
    values[id] = v[0] | (v[1] << 16);
    meta[id] = (uint8_t)(nib[0] | (nib[1] << 4));
  }
  if constexpr (COUNT) add_count(violations, bad);
}

__global__ void clear_i32_kernel(int32_t* p) { *p = 0; }

gpusq_status launch_compress_int4(const int8_t* W, uint8_t* values, uint8_t* meta, int32_t* violations, int64_t N, int64_t K,
                                  hipStream_t s) {
  const int64_t mrb = (K / 8 + 1) / 2;
  if (violations) clear_i32_kernel<<<1, 1, 0, s>>>(violations);
  const int64_t pairs = N * (K / 16);
  const unsigned flat_blocks = (unsigned)ceil_div(pairs, 256);
  if (K % 16 != 0)
    compress_int4_kernel<<<(unsigned)ceil_div(N * mrb, 256), 256, 0, s>>>(W, values, meta, violations, N, K);
  else if (violations)
    compress_int4_flat_kernel<true><<<flat_blocks, 256, 0, s>>>((const uint4*)W, (uint32_t*)values, meta, violations, pairs);
  else
    compress_int4_flat_kernel<false><<<flat_blocks, 256, 0, s>>>((const uint4*)W, (uint32_t*)values, meta, nullptr, pairs);
  return check_launch();
}

// ---------------------------------------------------------------------------------------------------------- decode
__global__ void __launch_bounds__(256) decompress_int4_kernel(const uint8_t* __restrict__ values, const uint8_t* __restrict__ meta,
                                                              int8_t* __restrict__ W, int64_t N, int64_t K) {
  const int64_t chunks_per_row = K / 8;
  const int64_t mrb = (chunks_per_row + 1) / 2;
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= N * mrb) return;
  const int64_t n = id / mrb, b = id % mrb;
  const unsigned byte = meta[n * mrb + b];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int64_t c = 2 * b + h;
    if (c < chunks_per_row) {
      const unsigned nib = (byte >> (4 * h)) & 0xFu;
      const unsigned p0 = nib & 3u, p1 = nib >> 2;
      const unsigned v = *(const uint16_t*)(values + n * (K / 4) + 2 * c);
      // sign-extend the four nibbles to bytes: the two codes of a kept sub-chunk as a 16-bit pair
      auto byte_of = [](unsigned nibble) { return (unsigned)((int)(nibble << 28) >> 28) & 0xFFu; };
      const uint64_t first = byte_of(v & 0xFu) | (byte_of((v >> 4) & 0xFu) << 8);
      const uint64_t second = byte_of((v >> 8) & 0xFu) | (byte_of((v >> 12) & 0xFu) << 8);
      const uint64_t chunk = (first << (16 * p0)) | (second << (16 * p1));
      *(uint2*)(W + n * K + 8 * c) = uint2{(unsigned)chunk, (unsigned)(chunk >> 32)};
    }
  }
}

// ---------------------------------------------------------------------------------------------------------- to 2:4
// INT4 storage -> the INT8 2:4 compressed form (values [N][K/2], one metadata byte per chunk = two groups of 4), for rows
// in which no group of 4 holds two non-zero sub-chunks (what pruning with one_per_group produces).  A group keeps its
// non-zero sub-chunk (the first one if it has none); a group with two non-zero sub-chunks keeps the second and is counted.
__device__ __forceinline__ void sparse_chunk(unsigned v, unsigned nib, unsigned& vals, unsigned& meta, int& bad) {
  const unsigned p0 = nib & 3u, p1 = nib >> 2;
  auto byte_of = [](unsigned nibble) { return (unsigned)((int)(nibble << 28) >> 28) & 0xFFu; };
  const uint64_t first = byte_of(v & 0xFu) | (byte_of((v >> 4) & 0xFu) << 8);
  const uint64_t second = byte_of((v >> 8) & 0xFu) | (byte_of((v >> 12) & 0xFu) << 8);
  const uint64_t chunk = (first << (16 * p0)) | (second << (16 * p1));  // the 8 dense codes, one byte each
  vals = 0;
  meta = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const unsigned group = (unsigned)(chunk >> (32 * h));
    const unsigned pair0 = group & 0xFFFFu, pair1 = group >> 16;
    bad += (int)(pair0 != 0 && pair1 != 0);
    const unsigned local = pair1 != 0 ? 1u : 0u;
    vals |= (local ? pair1 : pair0) << (16 * h);
    meta |= ((2 * local) | ((2 * local + 1) << 2)) << (4 * h);
  }
}

__global__ void __launch_bounds__(256) int4_to_sparse_int8_kernel(const uint8_t* __restrict__ values4, const uint8_t* __restrict__ meta4,
                                                                  int8_t* __restrict__ values8, uint8_t* __restrict__ meta8,
                                                                  int32_t* __restrict__ mismatches, int64_t N, int64_t K) {
  const int64_t chunks_per_row = K / 8;
  const int64_t mrb4 = (chunks_per_row + 1) / 2;
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int bad = 0;
  if (id < N * chunks_per_row) {
    const int64_t n = id / chunks_per_row, c = id % chunks_per_row;
    const unsigned nib = (meta4[n * mrb4 + (c >> 1)] >> (4 * (c & 1))) & 0xFu;
    unsigned vals, meta;
    sparse_chunk(*(const uint16_t*)(values4 + n * (K / 4) + 2 * c), nib, vals, meta, bad);
    *(uint32_t*)(values8 + n * (K / 2) + 4 * c) = vals;
    meta8[n * chunks_per_row + c] = (uint8_t)meta;
  }
  if (mismatches) add_count(mismatches, bad);
}

// The same for a flat run of an even number of chunks (no row of indices ends inside a byte): two chunks per thread and no
// division by the row length (5120 x 1280: 4.2 -> 3.4 us).
__global__ void __launch_bounds__(256) int4_to_sparse_int8_flat_kernel(const uint32_t* __restrict__ values4, const uint8_t* __restrict__ meta4,
                                                                       uint2* __restrict__ values8, uint16_t* __restrict__ meta8,
                                                                       int32_t* __restrict__ mismatches, int64_t pairs) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int bad = 0;
  if (id < pairs) {
    const unsigned v = values4[id], ix = meta4[id];
    unsigned o[2], m[2];
    sparse_chunk(v & 0xFFFFu, ix & 0xFu, o[0], m[0], bad);
    sparse_chunk(v >> 16, ix >> 4, o[1], m[1], bad);
    values8[id] = uint2{o[0], o[1]};
    meta8[id] = (uint16_t)(m[0] | (m[1] << 8));
  }
  if (mismatches) add_count(mismatches, bad);
}

gpusq_status launch_int4_to_sparse_int8(const uint8_t* values4, const uint8_t* meta4, int8_t* values8, uint8_t* meta8,
                                        int32_t* mismatches, int64_t N, int64_t K, hipStream_t s) {
  if (mismatches) clear_i32_kernel<<<1, 1, 0, s>>>(mismatches);
  if (K % 16 == 0)
    int4_to_sparse_int8_flat_kernel<<<(unsigned)ceil_div(N * (K / 16), 256), 256, 0, s>>>((const uint32_t*)values4, meta4, (uint2*)values8,
                                                                                        (uint16_t*)meta8, mismatches, N * (K / 16));
  else
    int4_to_sparse_int8_kernel<<<(unsigned)ceil_div(N * (K / 8), 256), 256, 0, s>>>(values4, meta4, values8, meta8, mismatches, N, K);
  return check_launch();
}

gpusq_status launch_decompress_int4(const uint8_t* values, const uint8_t* meta, int8_t* W, int64_t N, int64_t K, hipStream_t s) {
  const int64_t mrb = (K / 8 + 1) / 2;
  decompress_int4_kernel<<<(unsigned)ceil_div(N * mrb, 256), 256, 0, s>>>(values, meta, W, N, K);
  return check_launch();
}

}  // namespace gpusq
