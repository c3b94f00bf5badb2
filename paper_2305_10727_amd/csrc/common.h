// Internal declarations shared by the HIP translation units of libgpusq (not part of the public ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/gpusq.h"
#include "launch_rules.h"

namespace gpusq {

// ---- geometry of the kernel-native packed weight format (written by pack.hip, read by the GEMM kernels) ----------
// K advances in steps of 128 bytes of the dense activation row (128 int8 or 64 fp16 elements), the K extent of one
// gfx950 sparse matrix instruction (v_smfmac_i32_16x16x128_i8 / v_smfmac_f32_16x16x64_f16).  Output channels are
// grouped in tiles of 256 = 4 blocks of 64 = 16 fragments of 16 rows.  The packed buffer is an array of tiles
// [ceil(N/256)][ksteps]; one tile holds, for its 256 channels and one K step,
//     16 fragments x 1024 bytes of kept values   (fragment f, lane l: 16 bytes at f*1024 + l*16)
//   + 16 fragments x 64 lanes of index bits      (4 bytes per lane for int8, 2 for fp16), starting at byte 16384
//     (see index_offset),
// so that a workgroup fetches a tile with whole 1 KB wavefront-wide copies and a wavefront reads a fragment with one
// 16-byte and one 4-byte (2-byte) access per lane.
constexpr int kRowBlock = 64;          // output channels whose fragments interleave (see packed_row_to_channel)
constexpr int kTileRows = 256;         // output channels per packed tile
constexpr int kStepBytes = 128;        // bytes of a dense activation row consumed per K step
constexpr int kFragValueBytes = 1024;  // 64 lanes x 16 bytes of kept values
constexpr int kTileValueBytes = 16 * kFragValueBytes;
constexpr int kPrepareMaxK = 16384;    // longest row that gpusq_prepare_weights takes

__host__ __device__ constexpr int step_elems(bool is_i8) { return is_i8 ? 128 : 64; }
// index bytes of one fragment: 2 bits per kept value; 16 int8 values (32 bits) or 8 fp16 values (16 bits) per lane
__host__ __device__ constexpr int frag_index_bytes(bool is_i8) { return is_i8 ? 256 : 128; }
__host__ __device__ constexpr int tile_bytes(bool is_i8) { return kTileValueBytes + 16 * frag_index_bytes(is_i8); }
// Byte offset, inside a tile, of the index word of lane l of fragment f.  The index words are grouped per half tile
// (fragments 0..7 / 8..15 = the 128 channels one wavefront of the large-tile kernel owns) and, inside a half, per
// lane: a lane finds the index words of its 8 fragments in 32 (int8) or 16 (fp16) consecutive bytes and fetches them
// with two (one) 16-byte LDS reads instead of eight small ones.
__host__ __device__ constexpr int index_offset(bool is_i8, int f, int l) {
  const int ib = is_i8 ? 4 : 2;
  return kTileValueBytes + (f >> 3) * (64 * 8 * ib) + l * (8 * ib) + (f & 7) * ib;
}


// Row r (0..15) of fragment t (0..3) inside a 64-row block holds output channel
//   n = 64*blk + 32*(t/2) + 8*(r/4) + 4*(t%2) + (r%4).
// The accumulator of a 16x16 matrix instruction gives lane l the rows 4*(l/16)..4*(l/16)+3 of its column, so with
// this permutation a lane ends up, over fragments 0 and 1, with the 8 consecutive channels 8*(l/16)..+7 of one
// activation row (16 bytes of fp16 output) and the four lane groups of a wavefront write 64 contiguous bytes of that
// row in one store; fragments 2 and 3 give the next 32 channels the same way.
__host__ __device__ inline int packed_row_to_channel(int t, int r) { return 32 * (t >> 1) + 8 * (r >> 2) + 4 * (t & 1) + (r & 3); }

__device__ __forceinline__ float scale_reciprocal(float s) { return __fdiv_rn(1.0f, s); }

// Integer code of x under the scale s: clamp(rint(x / s), -127, 127) with the IEEE fp32 division of the definition
// (not a reciprocal multiply) and round-half-even, NaN -> 0, so that the code is decided exactly as a plain CPU
// evaluation of the formula decides it -- but without paying for a division per element.  r = fl(1 / s) (correctly
// rounded, computed once per scale).  t = x * r carries two roundings, |t - x/s| <= |x/s| (2^-23 + 2^-48), and the
// correctly rounded quotient is within 2^-24 |x/s| of x/s, so the quotient lies within 0.38 |t| 2^-21 of t.  rint()
// of the two can differ only if a half-integer lies between them or on one of them, which is excluded when t is at
// least |t| 2^-21 away from every half-integer (t - floor(t) is exact in fp32).  Only the rare element inside that
// band (about 1 in 10^5 for |t| near 100) pays for the division, and |t| >= 2^20, where the test always fails.  It is written
// as "not >=", so that an infinite or NaN t divides as well: under a denormal scale r is infinite and the quotient may be small.
__device__ __forceinline__ int finish_code(float q, float qmax = 127.0f) {
  const float c = fminf(fmaxf(rintf(q), -qmax), qmax);
  return (q != q) ? 0 : (int)c;  // of a NaN, or of a quotient without a value (infinity by infinity, 0 by 0): 0
}
// N values at once: the band test of all N values of all lanes is folded into one wavefront-uniform branch, so the
// common case executes no division at all (a per-element conditional is turned into a select by the compiler, which
// then evaluates the division for every element).
template <int N>
__device__ __forceinline__ void quantize_codes(const float (&x)[N], float s, float r, int (&q)[N], float qmax = 127.0f) {
  float t[N];
  bool near_half = false;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    t[j] = x[j] * r;
    near_half |= !(fabsf(__builtin_amdgcn_fractf(t[j]) - 0.5f) >= fabsf(t[j]) * 0x1p-21f);
  }
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(near_half) != 0, 0)) {  // some element of some lane sits next to a rounding boundary
#pragma unroll
    for (int j = 0; j < N; ++j) t[j] = __fdiv_rn(x[j], s);
  }
#pragma unroll
  for (int j = 0; j < N; ++j) q[j] = finish_code(t[j], qmax);
}
// The low bytes of four words as one.  (v_perm_b32: selector bytes 0..3 take bytes of the second operand, 4..7 of the first, 0x0c zero)
__device__ __forceinline__ unsigned low_bytes(unsigned b0, unsigned b1, unsigned b2, unsigned b3) {
  return __builtin_amdgcn_perm(b1, b0, 0x0c0c0400u) | __builtin_amdgcn_perm(b3, b2, 0x04000c0cu);
}
// The same codes as bytes, four to a word: a finite t is clamped first, then rounded half to even by adding 1.5 * 2^23, whose low byte
// is the two's-complement code.
template <int N>
__device__ __forceinline__ void quantize_words(const float (&x)[N], float s, float r, unsigned (&w)[N / 4], float qmax) {
  float t[N];
  unsigned b[N];
  bool near_half = false;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    t[j] = x[j] * r;
    near_half |= !(fabsf(__builtin_amdgcn_fractf(t[j]) - 0.5f) >= fabsf(t[j]) * 0x1p-21f);
    b[j] = __float_as_uint(__builtin_amdgcn_fmed3f(t[j], -qmax, qmax) + 12582912.0f);
  }
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(near_half) != 0, 0)) {
#pragma unroll
    for (int j = 0; j < N; ++j) b[j] = (unsigned)finish_code(__fdiv_rn(x[j], s), qmax);
  }
#pragma unroll
  for (int j = 0; j < N; j += 4) w[j / 4] = low_bytes(b[j], b[j + 1], b[j + 2], b[j + 3]);
}
// The codes of 8 values as bytes, the same ones as quantize_codes, with less arithmetic in the common case, for epilogues that are
// bound by the vector ALU.  In units of 2^-16: u = x (65536 r) + 32769 as a whole number, whose upper half is the code, floor(x / s +
// 1/2), and whose lower half says how far the quotient is from a boundary between codes.
//   * |u - (65536 x / s + 32769)| < 1.75 for |x / s| <= 127 (beyond, both clamp to the same code): half a unit from r (2^-24 of 127 2^16),
//     a quarter from the rounding of the fused multiply-add below 2^23, less than one from the conversion, which drops the fraction.
//     The quotient rounded to fp32 is within a quarter of a unit of x / s.  So a lower half of 3 or more puts it strictly between the
//     two boundaries of that code: 3 - 1.75 - 1 >= 1/4 above the lower one, 65535 + 1.75 - 1 <= 65536 - 1/4 below the upper one.  Other
//     values go to the division: 3 lower halves in 65536.
//   * The conversion saturates: +infinity to a lower half of 65535 and the code 127, -infinity and NaN (0) to a lower half of 0, that
//     is to the division.  A reciprocal that leaves no room for the factor 65536 (|s| below 2^-111) or is not finite sends every value
//     there.
// Four and a half vector instructions a value with the question, the clamp and the packing.
struct ByteQuantiser {
  float s, r16;
  __device__ __forceinline__ ByteQuantiser(float scale, float r) : s(scale), r16(fabsf(r) < 0x1p111f ? r * 65536.0f : __builtin_nanf("")) {
    asm("" : "+v"(r16));  // (the choice is made once, not for every value)
  }
  static constexpr unsigned short kNear = 3;  // a lower half below it: near a boundary
  __device__ __forceinline__ void units(float x, int& u) const {
    const float t = __fmaf_rn(x, r16, 32769.0f);
    asm("v_cvt_i32_f32 %0, %1" : "=v"(u) : "v"(t));  // (saturates, NaN gives 0: a C++ cast would promise neither)
  }
  __device__ __forceinline__ void units(const float (&x)[8], int (&u)[8]) const {
#pragma unroll
    for (int j = 0; j < 8; ++j) units(x[j], u[j]);
  }
  static __device__ __forceinline__ bool some_near(const int (&u)[8]) {  // wavefront-uniform
    unsigned m;  // of the lower halves the least (16-bit operations: the upper halves do not matter)
    asm("v_min3_u16 %0, %1, %2, %3" : "=v"(m) : "v"(u[0]), "v"(u[1]), "v"(u[2]));
    asm("v_min3_u16 %0, %0, %1, %2" : "+v"(m) : "v"(u[3]), "v"(u[4]));
    asm("v_min3_u16 %0, %0, %1, %2" : "+v"(m) : "v"(u[5]), "v"(u[6]));
    asm("v_min_u16 %0, %0, %1" : "+v"(m) : "v"(u[7]));
    return __builtin_amdgcn_ballot_w64((unsigned short)m < kNear) != 0;
  }
  // Each lane divides one of its values that ask for it at a time (a second one in a lane is rare, but where all of them do).  Marked
  // as unlikely, so that it stands behind the epilogue's own code: eight IEEE divisions in line, jumped over 15 times out of 16, and two
  // instructions more for every value took 49 us for 25216 x 768 -> 2304 where this takes 46, 31.6 for 50432 x 192 -> 768 + GELU (29.0),
  // 10.5 for 6304 x 384 -> 1000 (8.6).
  __device__ __forceinline__ void settle(const float (&x)[8], int (&u)[8]) const {
    if (__builtin_expect(some_near(u), 0)) {
      do {
        int which = 8;
        float xv = 0.0f;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const bool near = (unsigned short)u[j] < kNear;
          which = near ? j : which;
          xv = near ? x[j] : xv;
        }
        const int code = finish_code(__fdiv_rn(xv, s)) * 65536 + 32768;
#pragma unroll
        for (int j = 0; j < 8; ++j) u[j] = which == j ? code : u[j];
      } while (some_near(u));
    }
  }
  // value 0 in the low byte of `lo`
  static __device__ __forceinline__ void pack(const int (&u)[8], unsigned& lo, unsigned& hi) {
    unsigned c[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int least_code = -127 * 65536, most_code = 127 * 65536 + 65535;
      const int v = u[j] < least_code ? least_code : u[j];
      c[j] = (unsigned)(v > most_code ? most_code : v);
    }
    // byte 2 of each (v_perm_b32: selector bytes 0..3 take bytes of the second operand, 4..7 of the first, 0x0c zero)
    lo = __builtin_amdgcn_perm(c[1], c[0], 0x0c0c0602u) | __builtin_amdgcn_perm(c[3], c[2], 0x06020c0cu);
    hi = __builtin_amdgcn_perm(c[5], c[4], 0x0c0c0602u) | __builtin_amdgcn_perm(c[7], c[6], 0x06020c0cu);
  }
};
__device__ __forceinline__ void quantize_bytes8(const float (&x)[8], float s, float r, unsigned& lo, unsigned& hi) {
  const ByteQuantiser q(s, r);
  int u[8];
  q.units(x, u);
  q.settle(x, u);
  q.pack(u, lo, hi);
}
__device__ __forceinline__ int quantize_code(float x, float s, float r, float qmax = 127.0f) {
  const float xs[1] = {x};
  int q[1];
  quantize_codes<1>(xs, s, r, q, qmax);
  return q[0];
}

// The same codes for fp16 input with less arithmetic: one fused multiply-add per value, x * r + 1.5 * 2^23 (the exact product,
// rounded once, half to even, to a whole number), whose low byte is the code.  Whether that decides every code as
// rint(x / s) does depends on s alone and is checked once per scale and workgroup: both are monotone in x, so they agree on
// every fp16 x if they agree on the two fp16 neighbours of each code boundary (c + 0.5) * s, 254 values, one per thread; any
// other x lies at least one fp16 spacing, 2^-11 of it, from every boundary, thousands of times the rounding errors of either.
// r is the correctly rounded 1 / s or one of the two floats next to it, whichever agrees: the scale of a tensor's own range,
// amax / 127, puts x = amax / 2, an fp16 number, on the boundary 63.5 but for the roundings of s, and there the rounded
// reciprocal decides the other way for two scales in five.
// Where none agrees (one such scale in 250), the workgroup refines every product to the correctly rounded quotient first (t = x r,
// then t + r times the exact remainder x - t s: Markstein's division with a correctly rounded reciprocal), which takes four more
// operations: t is held within +-1024, far beyond every code, so that the remainder of an infinite x is infinite and not infinity
// less infinity.  (The few rows of 333 x 1040 -> 520 under a given scale take 5.0 us without and 6.1 with them.)
// A negative scale decides like its magnitude: the quotient and the product change their signs together, and the rounding is
// symmetric.  A magnitude outside 2^-100 .. 2^100 (denormal, 0, infinite, NaN) needs neither: every quotient is then far beyond
// the largest code or rounds to 0, or is NaN, and so is the product.
struct Fp16Quantiser {
  typedef _Float16 h8 __attribute__((ext_vector_type(8)));
  typedef _Float16 h2 __attribute__((ext_vector_type(2)));
  typedef int i4 __attribute__((ext_vector_type(4)));
  float s, r;
  bool refine;

  static __device__ __forceinline__ float neighbour(float r, int step) { return __uint_as_float(__float_as_uint(r) + (unsigned)step); }
  // The check of thread `tid` of a workgroup of 256 or more: bit c of the result is set if reciprocal c (0: the rounded one, 1, 2: its
  // neighbours above and below in magnitude) disagrees; the same in every lane of a wavefront.
  __device__ __forceinline__ unsigned prepare(float scale, int tid) {
    s = scale;
    r = scale_reciprocal(scale);
    const float mag = fabsf(scale), rmag = fabsf(r);
    bool bad[3] = {false, false, false};
    if (mag >= 0x1p-100f && mag <= 0x1p100f && tid < 254) {
      const float boundary = ((float)(tid >> 1) + 0.5f) * mag;
      const h2 down = __builtin_bit_cast(h2, __builtin_amdgcn_cvt_pkrtz(boundary, 0.0f));
      const unsigned short bits = (unsigned short)(__builtin_bit_cast(unsigned short, down[0]) + (tid & 1));
      if (bits < 0x7C00) {  // else no finite fp16 number there
        const float x = (float)__builtin_bit_cast(_Float16, bits);
        // (Markstein's quotient is not the rounded one under a scale one unit below a power of two, x = s / 2: a division)
        const float exact = fminf(rintf(__fdiv_rn(x, mag)), 127.0f);
#pragma unroll
        for (int c = 0; c < 3; ++c)
          bad[c] = fminf(__fmaf_rn(x, neighbour(rmag, c == 2 ? -1 : c), 12582912.0f) - 12582912.0f, 127.0f) != exact;
      }
    }
    unsigned votes = 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) votes |= __builtin_amdgcn_ballot_w64(bad[c]) != 0 ? 1u << c : 0u;
    return votes;
  }
  // With the votes of all threads.
  __device__ __forceinline__ void decide(unsigned votes) {
    refine = (votes & 7u) == 7u;
    if ((votes & 1u) != 0 && !refine) r = neighbour(r, (votes & 2u) == 0 ? 1 : -1);
  }
  // Wavefront-uniform: some lane's 8 N values need `odd` codes: a NaN is among them (or infinities of both signs, which lose nothing
  // there), or the reciprocal is one whose product with 0 or infinity is NaN; there the quotient is NaN as well, or 0 by a denormal.
  template <int N>
  __device__ __forceinline__ bool odd(const i4 (&raw)[N]) const {
    h2 sum = h2(0);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const h8 x = __builtin_bit_cast(h8, raw[j]);
      sum += (h2{x[0], x[1]} + h2{x[2], x[3]}) + (h2{x[4], x[5]} + h2{x[6], x[7]});
    }
    const _Float16 all = sum[0] + sum[1];
    return __builtin_amdgcn_ballot_w64(!(all == all)) != 0 || !(fabsf(r) > 0.0f && fabsf(r) <= 3.4028234663852886e38f);
  }
  // Codes of 8 values as bytes.  CLAMP: values may exceed 127 s (a given scale; with the scale of the data's own range no
  // quotient reaches 127.5).  The code of a NaN is 0.
  template <bool CLAMP>
  __device__ __forceinline__ void codes(i4 raw, bool odd, unsigned& lo, unsigned& hi) const {
    const h8 x = __builtin_bit_cast(h8, raw);
    float y[8];
    if (__builtin_expect(refine, 0)) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float t = __builtin_amdgcn_fmed3f((float)x[j] * r, -1024.0f, 1024.0f);
        y[j] = __builtin_fmaf(__builtin_fmaf(-t, s, (float)x[j]), r, t) + 12582912.0f;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) y[j] = __builtin_fmaf((float)x[j], r, 12582912.0f);
    }
    if (__builtin_expect(odd, 0)) {
#pragma unroll
      for (int j = 0; j < 8; ++j) y[j] = y[j] == y[j] ? y[j] : 12582912.0f;
    }
    if constexpr (CLAMP) {
#pragma unroll
      for (int j = 0; j < 8; ++j) y[j] = __builtin_amdgcn_fmed3f(y[j], 12582912.0f - 127.0f, 12582912.0f + 127.0f);
    }
    unsigned b[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) b[j] = __float_as_uint(y[j]);
    lo = low_bytes(b[0], b[1], b[2], b[3]);
    hi = low_bytes(b[4], b[5], b[6], b[7]);
  }
  // The codes of N vectors: one question for all of them, and what is rare stands out of line (a wavefront alone on its SIMD pays for every
  // branch it meets).
  template <bool CLAMP, int N>
  __device__ __forceinline__ void codes_of(const i4 (&raw)[N], unsigned (&c)[N][2]) const {
    const bool some_odd = odd(raw);
    if (__builtin_expect(some_odd || refine, 0)) {
#pragma unroll
      for (int j = 0; j < N; ++j) {
        i4 x = raw[j];
        asm volatile("" : "+v"(x));  // (nothing of it is shared with the other branch, and computed in front of both)
        codes<CLAMP>(x, some_odd, c[j][0], c[j][1]);
      }
    } else {
      const Fp16Quantiser plain{s, r, false};
#pragma unroll
      for (int j = 0; j < N; ++j) plain.codes<CLAMP>(raw[j], false, c[j][0], c[j][1]);
    }
  }
};

// The largest of a wavefront's values, none of them negative or NaN (their bit patterns then compare as they do): data-parallel
// primitives instead of six trips through the LDS crossbar.
__device__ __forceinline__ float wave_max_magnitude(float v) {
  unsigned m = __float_as_uint(v);
#define GPUSQ_MAX_DPP(CTRL, ROWS) \
  {                               \
    const unsigned o = (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, CTRL, ROWS, 0xF, false); \
    m = m > o ? m : o;            \
  }
  GPUSQ_MAX_DPP(0x111, 0xF)  // row_shr 1, 2, 4, 8: the last lane of each row of 16 has the row's
  GPUSQ_MAX_DPP(0x112, 0xF)
  GPUSQ_MAX_DPP(0x114, 0xF)
  GPUSQ_MAX_DPP(0x118, 0xF)
  GPUSQ_MAX_DPP(0x142, 0xA)  // row_bcast 15 to rows 1 and 3, row_bcast 31 to rows 2 and 3: lane 63 has the wavefront's
  GPUSQ_MAX_DPP(0x143, 0xC)
#undef GPUSQ_MAX_DPP
  return __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)m, 63));
}

// Largest magnitude (NaN aside) of this thread's share of n fp16 values, n % 8 == 0 and n / 8 below 2^27: 16-byte loads, eight of
// them in flight.  Magnitudes are compared as whole numbers; a thread that meets a NaN, the largest of these, goes over its share
// again with the comparison that ignores it.
__device__ __forceinline__ float range_of_fp16(const uint8_t* X, int64_t n, int tid, int threads) {
  typedef _Float16 h8 __attribute__((ext_vector_type(8)));
  typedef unsigned short us8 __attribute__((ext_vector_type(8)));
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  const int vecs = (int)(n / 8);
  auto at = [&](int i) { return *(const u4*)(X + 16u * (uint32_t)i) & 0x7fff7fffu; };
  us8 m = us8(0);
  for (int i = tid; i < vecs; i += 8 * threads) {
    u4 v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = at(i + j * threads < vecs ? i + j * threads : vecs - 1);
#pragma unroll
    for (int j = 0; j < 8; ++j) m = __builtin_elementwise_max(m, __builtin_bit_cast(us8, v[j]));
  }
  unsigned top = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) top = m[j] > top ? m[j] : top;
  if (top > 0x7C00u) {
    h8 f = h8(0);
    for (int i = tid; i < vecs; i += threads) f = __builtin_elementwise_max(f, __builtin_bit_cast(h8, at(i)));
    float amax = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) amax = fmaxf(amax, (float)f[j]);
    return amax;
  }
  return (float)__builtin_bit_cast(_Float16, (unsigned short)top);
}

// The same of fp32 values, n % 4 == 0.
__device__ __forceinline__ float range_of_fp32(const float* X, int64_t n, int tid, int threads) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  const int vecs = (int)(n / 4);
  float amax = 0.0f;
  for (int i = tid; i < vecs; i += 8 * threads) {
    f4 v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = ((const f4*)X)[i + j * threads < vecs ? i + j * threads : vecs - 1];
#pragma unroll
    for (int j = 0; j < 8; ++j) amax = fmaxf(fmaxf(amax, fmaxf(fabsf(v[j][0]), fabsf(v[j][1]))), fmaxf(fabsf(v[j][2]), fabsf(v[j][3])));
  }
  return amax;
}

// Selection rule inside one group of 4 [Sec. 3.1: two of every four contiguous elements are zero; the rule is this
// library's reading]: element i is kept iff fewer than two elements beat it, where j beats i when |w_j| > |w_i|, or
// |w_j| == |w_i| and j < i.  Magnitudes are compared as sign-cleared bit patterns (a total order).
// Returns the 4-bit keep mask (exactly two bits set).
__device__ __forceinline__ unsigned keep_mask_of_4(unsigned k0, unsigned k1, unsigned k2, unsigned k3) {
  const unsigned r0 = (k1 > k0) + (k2 > k0) + (k3 > k0);
  const unsigned r1 = (k0 >= k1) + (k2 > k1) + (k3 > k1);
  const unsigned r2 = (k0 >= k2) + (k1 >= k2) + (k3 > k2);
  const unsigned r3 = (k0 >= k3) + (k1 >= k3) + (k2 >= k3);
  return (r0 < 2u) | ((r1 < 2u) << 1) | ((r2 < 2u) << 2) | ((r3 < 2u) << 3);
}

// positions of the two set bits of a keep mask, packed as the metadata nibble p0 | p1 << 2 (p0 < p1)
__device__ __forceinline__ unsigned nibble_of_mask(unsigned m) {
  const unsigned p0 = __builtin_ctz(m);
  const unsigned p1 = 31u - __builtin_clz(m);
  return p0 | (p1 << 2);
}

void set_last_hip_error(hipError_t e);

struct GemmArgs {
  const void* X;
  const void* W;  // packed (sparse) or dense [N][K]
  const float* act_scale;
  const float* w_scale;
  const float* bias;
  const float* out_scale;
  void* Y;
  int M, N, K;
  int epilogue;
  int out_dt;
  // Patch-embedding mode (patch_P != 0): X is an image batch [B][C][H][W] and row m = (b, py, px) of the X operand is
  // patch (py, px) of image b, column (c*P + i)*P + j its pixel (py*P + i, px*P + j) of channel c; M = B*(H/P)*(W/P),
  // K = C*P*P.  The tile kernel then fetches its X slabs from the image directly (no flattened-patch buffer).
  int patch_P = 0, patch_C = 0, patch_H = 0, patch_W = 0;
  // INT8 path, small kernels only: X holds fp16 (1) activations, quantised inside the kernel with the static act_scale; in the kernel
  // for few rows fp32 (2) as well
  int x_f16 = 0;
  // ... or, in the kernel for few rows, with the scale of X's own range: that of the `npartial` partial maxima a range pass
  // left behind, or of all of X, read by every workgroup; the scale goes to scale_out, the codes to xq_out (if not NULL)
  int range_mode = 0, npartial = 0;
  const float* partial = nullptr;
  float* scale_out = nullptr;
  int8_t* xq_out = nullptr;
  // INT8 path, fp16 output without GELU: the codes of that output as well, under out_scale (not NULL then)
  int8_t* codes_out = nullptr;
};
// What a kernel writes where its template says so: a gpusq_dtype, or fp16 and its codes (GemmArgs::codes_out)
constexpr int kOutF16Codes = 16;
__host__ __device__ constexpr bool is_f16_out(int out) { return out == GPUSQ_F16 || out == kOutF16Codes; }
enum { kRangeGiven = 0, kRangePartials = 1, kRangeHere = 2 };

gpusq_status launch_spgemm(bool is_i8, const GemmArgs& a, hipStream_t s);
gpusq_status launch_dense(bool is_i8, const GemmArgs& a, hipStream_t s);
// the sparse GEMM for few rows (fewrows.hip)
bool fewrows_supports(const GemmArgs& a);
bool fewrows_folds_quantiser(int64_t M, int64_t N, int64_t K, int resident, bool fp32);
gpusq_status launch_fewrows(bool is_i8, const GemmArgs& a, int resident, hipStream_t s);
// the sparse INT8 GEMM on whole rows that it quantises (wide.hip)
struct WidePlan;
gpusq_status launch_wide(const GemmArgs& a, const WidePlan& p, hipStream_t s);
// the layers behind attention on calibrated scales (mlp.hip): attention's codes Xq [M][D]; proj's output P and its codes Hq [M][D], the codes G [M][H]
// of fc1's GELU, fc2's output Y [M][D]
struct MlpArgs {
  const int8_t* Xq;
  const void *Wp, *W1, *W2;
  const float *s_attn, *s_h, *s_g;
  const float *ws_proj, *ws_fc1, *ws_fc2, *b_proj, *b_fc1, *b_fc2;
  void* P;
  int8_t *Hq, *G;
  void* Y;
  int M, D, H;
};
bool mlp_in_one_launch(const MlpArgs& a);
int mlp_launches(int64_t M, int64_t D, int64_t H, int cus);
gpusq_status launch_mlp(const MlpArgs& a, hipStream_t s);
// a patch embedding on fp16 images in one launch (patches.hip), or by flattened patches in a.X and the GEMM
gpusq_status launch_patch_embed_f16(GemmArgs a, const void* img, int64_t B, int64_t C, int64_t H, int64_t W, int64_t P, hipStream_t s);
int patch_embed_f16_launches(int64_t B, int64_t C, int64_t H, int64_t W, int64_t P, int64_t K_pad, int64_t D, int epilogue, int cus);
// 16 x 16 patches, few of them, on the kernel for whole rows behind a range pass (a: with the fields of a patch embedding)
bool few_patches_take_whole_rows(int64_t M, int64_t N, int64_t K, int epilogue, gpusq_dtype dt, int cus);
gpusq_status launch_few_patches(const GemmArgs& a, gpusq_dtype dt, int8_t* img_q, float* scale, void* workspace, hipStream_t s);
// the int8 one: range pass and the same kernel, or quantiser, flattened patches in a.X and the GEMM
gpusq_status launch_patch_embed_i8(GemmArgs a, const void* img, gpusq_dtype dt, int8_t* img_q, float* scale, void* workspace, int64_t B, int64_t C, int64_t H,
                                   int64_t W, int64_t P, hipStream_t s);
int patch_embed_i8_launches(gpusq_dtype dt, int64_t B, int64_t C, int64_t H, int64_t W, int64_t P, int64_t K_pad, int64_t D, int epilogue, int cus);
int num_cus();                      // of the current device
// quantise (dt of X, workspace as for launch_quantize) and multiply: one, two or three launches
gpusq_status launch_linear_int8(GemmArgs a, gpusq_dtype dt, int8_t* Xq, float* scale, int scale_is_input, void* workspace, hipStream_t s);
int linear_int8_launches(const GemmArgs& a, gpusq_dtype dt, int scale_is_input, int cus);
int linear_int8_quantiser(const GemmArgs& a, gpusq_dtype dt, int scale_is_input, int cus);
// the same for a patch embedding (GemmArgs::patch_P): images of dt, their codes
gpusq_status launch_patch_embed_int8(GemmArgs a, gpusq_dtype dt, int8_t* img_q, float* scale, void* workspace, hipStream_t s);
// the range pass of the per-tensor quantiser alone; returns the number of partial maxima it leaves in the workspace
int launch_amax(const void* X, gpusq_dtype dt, int64_t n, void* workspace, hipStream_t s);
int forced_kernel();                // -1 when none is forced
int set_forced_kernel(int kernel);  // testing aid, see gpusq_force_kernel; returns the previous value
gpusq_status plan_spgemm(bool is_i8, int64_t M, int64_t N, int64_t K, int epilogue, int cus, int32_t* out);

gpusq_status launch_prune(const void* Win, void* Wout, uint8_t* mask, gpusq_dtype dt, int64_t N, int64_t K, hipStream_t s);
gpusq_status launch_prune_n_of_m(const float* Win, float* Wout, int n_keep, int m, int64_t N, int64_t K, hipStream_t s);
gpusq_status launch_cast_f16(const float* in, void* out, int64_t n, hipStream_t s);
gpusq_status launch_im2col_patches(const void* img, void* X, gpusq_dtype dt, int64_t B, int64_t C, int64_t H, int64_t W, int64_t P,
                                   int64_t K_pad, hipStream_t s);
gpusq_status launch_quantize(const void* X, gpusq_dtype dt, int8_t* Xq, float* scale, int mode, int scale_is_input,
                             int64_t rows, int64_t cols, void* workspace, hipStream_t s);
gpusq_status launch_quantize_tensor_static(const void* X, gpusq_dtype dt, int8_t* Xq, float* scale, int scale_is_input,
                                           int64_t rows, int64_t cols, hipStream_t s);
gpusq_status launch_quantize_rows_int4(const void* X, gpusq_dtype dt, int8_t* Xq, float* scale, int scale_is_input, int64_t rows,
                                       int64_t cols, hipStream_t s);
gpusq_status launch_prune_pairs(const float* Win, float* Wout, uint8_t* mask, int one_per_group, int64_t N, int64_t K, hipStream_t s);
gpusq_status launch_int4_to_sparse_int8(const uint8_t* values4, const uint8_t* meta4, int8_t* values8, uint8_t* meta8,
                                        int32_t* mismatches, int64_t N, int64_t K, hipStream_t s);
gpusq_status launch_compress_int4(const int8_t* W, uint8_t* values, uint8_t* meta, int32_t* violations, int64_t N, int64_t K,
                                  hipStream_t s);
gpusq_status launch_decompress_int4(const uint8_t* values, const uint8_t* meta, int8_t* W, int64_t N, int64_t K, hipStream_t s);
gpusq_status launch_count_violations(const void* W, gpusq_dtype dt, int32_t* violations, int64_t N, int64_t K, hipStream_t s);
gpusq_status launch_compress(const void* W, void* values, uint8_t* meta, int32_t* violations, gpusq_dtype dt,
                             int64_t N, int64_t K, hipStream_t s);
gpusq_status launch_decompress(const void* values, const uint8_t* meta, void* W, gpusq_dtype dt, int64_t N, int64_t K,
                               hipStream_t s);
gpusq_status launch_pack(const void* values, const uint8_t* meta, void* packed, gpusq_dtype dt, int64_t N, int64_t K,
                         hipStream_t s);

gpusq_status launch_prepare_weights(const float* W, gpusq_dtype dt, float* Wp, void* Wlow, float* w_scale, void* values,
                                    uint8_t* meta, void* packed, int64_t N, int64_t K, hipStream_t s);

inline gpusq_status check_launch() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_last_hip_error(e);
    return GPUSQ_ERR_HIP;
  }
  return GPUSQ_OK;
}

}  // namespace gpusq
