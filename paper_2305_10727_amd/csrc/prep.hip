// Weight / activation preparation kernels: 2:4 pruning, symmetric INT8 quantisation, compression to kept values +
// 2-bit metadata, decompression, and re-tiling into the kernel-native packed format.
// All of them stream their operands once and are bound by HBM bandwidth; work is laid out wavefront-parallel over
// groups of 4 (one lane per group or per pair of groups), with 16-byte accesses where the layout allows.
#include <atomic>
#include <type_traits>

#include "common.h"

namespace gpusq {

// ------------------------------------------------------------------------------------------------------------ prune
__global__ void __launch_bounds__(256) prune_f32_kernel(const float4* __restrict__ in, float4* __restrict__ out,
                                                        uint8_t* __restrict__ mask, int64_t groups) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= groups) return;
  const float4 w = in[g];
  const unsigned m = keep_mask_of_4(__float_as_uint(w.x) & 0x7FFFFFFFu, __float_as_uint(w.y) & 0x7FFFFFFFu,
                                    __float_as_uint(w.z) & 0x7FFFFFFFu, __float_as_uint(w.w) & 0x7FFFFFFFu);
  float4 o;
  o.x = (m & 1u) ? w.x : 0.0f;
  o.y = (m & 2u) ? w.y : 0.0f;
  o.z = (m & 4u) ? w.z : 0.0f;
  o.w = (m & 8u) ? w.w : 0.0f;
  out[g] = o;
  if (mask) mask[g] = (uint8_t)m;
}

__global__ void __launch_bounds__(256) prune_f16_kernel(const uint2* __restrict__ in, uint2* __restrict__ out,
                                                        uint8_t* __restrict__ mask, int64_t groups) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= groups) return;
  const uint2 w = in[g];
  const unsigned h0 = w.x & 0xFFFFu, h1 = w.x >> 16, h2 = w.y & 0xFFFFu, h3 = w.y >> 16;
  const unsigned m = keep_mask_of_4(h0 & 0x7FFFu, h1 & 0x7FFFu, h2 & 0x7FFFu, h3 & 0x7FFFu);
  uint2 o;
  o.x = ((m & 1u) ? h0 : 0u) | (((m & 2u) ? h1 : 0u) << 16);
  o.y = ((m & 4u) ? h2 : 0u) | (((m & 8u) ? h3 : 0u) << 16);
  out[g] = o;
  if (mask) mask[g] = (uint8_t)m;
}

gpusq_status launch_prune(const void* Win, void* Wout, uint8_t* mask, gpusq_dtype dt, int64_t N, int64_t K, hipStream_t s) {
  const int64_t groups = N * K / 4;
  const unsigned blocks = (unsigned)ceil_div(groups, 256);
  if (dt == GPUSQ_F32)
    prune_f32_kernel<<<blocks, 256, 0, s>>>((const float4*)Win, (float4*)Wout, mask, groups);
  else
    prune_f16_kernel<<<blocks, 256, 0, s>>>((const uint2*)Win, (uint2*)Wout, mask, groups);
  return check_launch();
}

// ------------------------------------------------------------------------------------------------------------ cast
__global__ void __launch_bounds__(256) cast_f16_kernel(const float* __restrict__ in, _Float16* __restrict__ out, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x * 4;
  for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4; i < n; i += stride) {
    if (i + 3 < n) {
      const float4 v = *(const float4*)(in + i);
      typedef _Float16 h4 __attribute__((ext_vector_type(4)));
      *(h4*)(out + i) = h4{(_Float16)v.x, (_Float16)v.y, (_Float16)v.z, (_Float16)v.w};
    } else {
      for (int64_t j = i; j < n; ++j) out[j] = (_Float16)in[j];
    }
  }
}

// ---- patch embedding: images [B][C][H][W] -> flattened patches X [B*(H/P)*(W/P)][K_pad] (Sec. 3.3) ------------------------
// Row m = (b, py, px) of X holds patch (py, px) of image b, column k = (c*P + i)*P + j holds pixel (py*P + i, px*P + j) of
// channel c (the order of a convolution weight [D][C][P][P] flattened along its last three axes); columns C*P*P..K_pad-1
// are zero.  One thread moves VEC consecutive columns, which lie in one image row when P % VEC == 0.
template <typename T, int VEC>
__global__ void __launch_bounds__(256) im2col_patches_kernel(const T* __restrict__ img, T* __restrict__ X, int C, int H, int W, int P,
                                                             int K, int K_pad, int64_t units) {
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  const int kv = K_pad / VEC, px_n = W / P, py_n = H / P;
  for (int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x; u < units; u += (int64_t)gridDim.x * 256) {
    const int64_t m = u / kv;
    const int k0 = (int)(u - m * kv) * VEC;
    vec_t v = vec_t(0);
    if (k0 < K) {
      const int c = k0 / (P * P), r = k0 - c * P * P, i = r / P, j = r - i * P;
      const int px = (int)(m % px_n), py = (int)((m / px_n) % py_n);
      const int64_t b = m / ((int64_t)px_n * py_n);
      const T* src = img + ((b * C + c) * H + (int64_t)py * P + i) * W + (int64_t)px * P + j;
      if constexpr (VEC == 1)
        v = vec_t(*src);
      else
        v = *(const vec_t*)src;
    }
    *(vec_t*)(X + m * K_pad + k0) = v;
  }
}

// The same for patch sizes whose rows are not multiples of 16 bytes (P = 14): one workgroup per (image, row of patches).  The
// rows of X it makes are one contiguous run of W/P * K_pad elements, written with 16-byte stores; what they hold, the P image
// rows of every channel, is read into LDS whole, several words in flight per thread.  A thread writes the same 16-byte column chunk
// of every (third, ...) patch: where its pieces of U bytes (the largest power of two that divides a patch row) lie in a patch is
// worked out once, and a store costs it 16/U LDS reads and no division.
// Memory-bound: 256 x 3 x 224 x 224 fp16, P = 14, cold: 65 us with a workgroup per channel that wrote runs of P*P columns 4 bytes at
// a time, 32 us so (77 MB read, 84 MB written: 5.0 TB/s).  With few workgroups it is latency: with one word in flight per thread and
// two divisions per piece instead of two per chunk, 18 x 3 x 280 x 308 int8 (4-byte words) took 7.3 us, 6.1 so, and 256 x 3 x 224 x 224
// int8 22.9, 19.0 so.
// Needs K_pad * sizeof(T) % 16 == 0, plane and strip sizes in whole 4-byte words and the strips of all channels in 64 KB.
constexpr size_t kStripBytes = 64 * 1024;
template <typename T, int U>
__global__ void __launch_bounds__(256) im2col_rows_kernel(const T* __restrict__ img, T* __restrict__ X, int C, int H, int W, int P, int K,
                                                          int K_pad) {
  extern __shared__ __attribute__((aligned(16))) uint8_t strip[];
  typedef typename std::conditional<U == 1, uint8_t, typename std::conditional<U == 2, uint16_t, typename std::conditional<U == 4, uint32_t, uint64_t>::type>::type>::type piece_t;
  constexpr int ES = (int)sizeof(T), PIECES = 16 / U;
  const int py_n = H / P, px_n = W / P;
  const int py = blockIdx.x % py_n, b = blockIdx.x / py_n, tid = threadIdx.x;
  const int span = P * W * ES;  // bytes of a channel's strip
  const int64_t plane = (int64_t)H * W * ES;
  const uint8_t* src = (const uint8_t*)img + (int64_t)b * C * plane + (int64_t)py * span;
  // (the strips' words, several requested before the first is stored)
  auto fill = [&](auto word) {
    typedef decltype(word) word_t;
    constexpr int S = (int)sizeof(word_t), B = S == 16 ? 4 : 8;
    const int per = span / S, all = C * per;
    for (int base = tid; base < all; base += 256 * B) {
      word_t v[B];
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int i = base + 256 * u < all ? base + 256 * u : tid, c = i / per;
        v[u] = *(const word_t*)(src + c * plane + S * (i - c * per));
      }
#pragma unroll
      for (int u = 0; u < B; ++u)
        if (base + 256 * u < all) *(word_t*)(strip + S * (base + 256 * u)) = v[u];
    }
  };
  if (((span | (int)(plane & 15)) & 15) == 0)
    fill(uint4{});
  else
    fill(uint32_t{});
  __syncthreads();
  const int chunks = K_pad * ES / 16;                    // of a row of X
  const int side = chunks < 256 ? 256 / chunks : 1;      // patches side by side
  uint8_t* dst = (uint8_t*)X + ((int64_t)b * py_n + py) * px_n * K_pad * ES;
  for (int kc = tid; kc < side * chunks; kc += 256) {
    const int px0 = kc / chunks, chunk = kc - px0 * chunks;
    int at[PIECES];  // LDS offset of each piece in patch 0; < 0: a padding column
    int k = chunk * (16 / ES);
    int c = k / (P * P), i = (k - c * P * P) / P, j = k - (c * P + i) * P;
#pragma unroll
    for (int e = 0; e < PIECES; ++e) {
      at[e] = k < K ? ((c * P + i) * W + j) * ES : -1;
      k += U / ES;
      j += U / ES;
      if (j == P) {  // (a piece never crosses a patch row)
        j = 0;
        if (++i == P) i = 0, ++c;
      }
    }
    for (int px = px0; px < px_n; px += side) {
      union {
        piece_t piece[PIECES];
        uint4 v;
      } o;
#pragma unroll
      for (int e = 0; e < PIECES; ++e) {
        const piece_t x = *(const piece_t*)(strip + (at[e] < 0 ? 0 : at[e] + px * P * ES));
        o.piece[e] = at[e] < 0 ? (piece_t)0 : x;
      }
      *(uint4*)(dst + ((int64_t)px * chunks + chunk) * 16) = o.v;
    }
  }
}

// The same where the strips of all channels do not fit into LDS or a row of X is no whole number of 16-byte chunks: one workgroup
// per (image, channel, row of patches).  The P image rows of that strip are one contiguous span of P*W elements: it is read into LDS with 4-byte
// loads, and written out as W/P runs of P*P consecutive columns (one per patch), 4 bytes per thread and store, each word
// gathered from LDS.  The workgroups of channel 0 also zero the padding columns of their rows.
// Needs (W * sizeof(T)) % 4 == 0, (P*P * sizeof(T)) % 4 == 0, (K_pad * sizeof(T)) % 4 == 0 and a span of at most 48 KB.
template <typename T>
__global__ void __launch_bounds__(256) im2col_strip_kernel(const T* __restrict__ img, T* __restrict__ X, int C, int H, int W, int P,
                                                           int K, int K_pad) {
  extern __shared__ __attribute__((aligned(16))) uint8_t strip_raw[];
  T* strip = (T*)strip_raw;
  constexpr int EPW = 4 / (int)sizeof(T);  // elements per 4-byte word
  const int py_n = H / P, px_n = W / P;
  const int py = blockIdx.x % py_n, c = (blockIdx.x / py_n) % C;
  const int64_t b = blockIdx.x / (py_n * C);
  const int span_words = P * W / EPW;
  const uint32_t* src = (const uint32_t*)(img + ((b * C + c) * H + (int64_t)py * P) * W);
  for (int q = threadIdx.x; q < span_words; q += 256) ((uint32_t*)strip)[q] = src[q];
  __syncthreads();
  const int wpr = P * P / EPW;  // words per run
  const int64_t m0 = (b * py_n + py) * px_n;
  for (int q = threadIdx.x; q < span_words; q += 256) {
    const int px = q / wpr, rq = q - px * wpr;
    T e[EPW];
#pragma unroll
    for (int t = 0; t < EPW; ++t) {
      const int r = rq * EPW + t, i = r / P, j = r - i * P;
      e[t] = strip[i * W + px * P + j];
    }
    uint32_t word;
    __builtin_memcpy(&word, e, 4);
    *(uint32_t*)(X + (m0 + px) * K_pad + (int64_t)c * P * P + rq * EPW) = word;
  }
  if (c == 0) {
    const int pad_words = (K_pad - K) / EPW;
    for (int q = threadIdx.x; q < pad_words * px_n; q += 256) {
      const int px = q / pad_words, w = q - px * pad_words;
      *(uint32_t*)(X + (m0 + px) * K_pad + K + w * EPW) = 0u;
    }
  }
}

template <typename T>
static gpusq_status launch_im2col_typed(const T* img, T* X, int64_t B, int64_t C, int64_t H, int64_t W, int64_t P, int64_t K_pad,
                                        hipStream_t s) {
  const int64_t M = B * (H / P) * (W / P);
  const int K = (int)(C * P * P);
  // the widest power-of-two move (up to 16 bytes) for which every source and destination address is aligned: it must
  // divide P (a move stays inside one image row and pixel offsets are multiples of it), W and K_pad
  int vec = 16 / (int)sizeof(T);
  while (vec > 1 && (P % vec != 0 || W % vec != 0 || K_pad % vec != 0)) vec >>= 1;
  const int64_t span_bytes = P * W * (int64_t)sizeof(T);
  const bool ragged = vec * sizeof(T) < 16;
  const bool strips = ragged && (W * sizeof(T)) % 4 == 0 && (P * P * sizeof(T)) % 4 == 0 && (K_pad * sizeof(T)) % 4 == 0 &&
                      (K * sizeof(T)) % 4 == 0 && span_bytes <= 48 * 1024 && B * C * (H / P) <= INT32_MAX;
  int u = 8;  // bytes of the pieces a patch row is made of
  while ((P * (int)sizeof(T)) % u != 0 || (W * (int)sizeof(T)) % u != 0) u >>= 1;
  // Pieces of 1 or 2 bytes and up to 256 strips (4 images of 224 x 224, P = 14): the kernels with more workgroups, each with less of a
  // chain (int8, P = 14, 1 image: 3.5 us against 3.8; 8 images 4.1 against 4.0; P = 7, 1 image: 3.3 against 4.2; pieces of 4 bytes, fp16,
  // P = 14, 1 image: 4.2 against 4.1)
  const bool few = u <= 2 && B * C * (H / P) <= 256;
  if (ragged && !few && (K_pad * sizeof(T)) % 16 == 0 && span_bytes % 4 == 0 && (H * W * sizeof(T)) % 4 == 0 &&
      C * span_bytes <= (int64_t)kStripBytes && B * (H / P) <= INT32_MAX) {
    const unsigned grid = (unsigned)(B * (H / P));
#define GPUSQ_IM2COL_ROWS(U) im2col_rows_kernel<T, U><<<grid, 256, (size_t)(C * span_bytes), s>>>(img, X, (int)C, (int)H, (int)W, (int)P, K, (int)K_pad)
    if (u >= 8) GPUSQ_IM2COL_ROWS(8);
    else if (u == 4) GPUSQ_IM2COL_ROWS(4);
    else if (u == 2) GPUSQ_IM2COL_ROWS(2);
    else GPUSQ_IM2COL_ROWS(sizeof(T));
#undef GPUSQ_IM2COL_ROWS
    return check_launch();
  }
  if (strips) {
    im2col_strip_kernel<T><<<(unsigned)(B * C * (H / P)), 256, (size_t)span_bytes, s>>>(img, X, (int)C, (int)H, (int)W, (int)P, K, (int)K_pad);
    return check_launch();
  }
  const int64_t units = M * (K_pad / vec);
  const int64_t want = ceil_div(units, 256);
  const unsigned grid = (unsigned)(want < 16384 ? want : 16384);
#define GPUSQ_IM2COL_CASE(V) \
  case V:                    \
    im2col_patches_kernel<T, V><<<grid, 256, 0, s>>>(img, X, (int)C, (int)H, (int)W, (int)P, K, (int)K_pad, units); \
    break;
  switch (vec) {
    GPUSQ_IM2COL_CASE(16)
    GPUSQ_IM2COL_CASE(8)
    GPUSQ_IM2COL_CASE(4)
    GPUSQ_IM2COL_CASE(2)
    default:
      im2col_patches_kernel<T, 1><<<grid, 256, 0, s>>>(img, X, (int)C, (int)H, (int)W, (int)P, K, (int)K_pad, units);
      break;
  }
#undef GPUSQ_IM2COL_CASE
  return check_launch();
}

gpusq_status launch_im2col_patches(const void* img, void* X, gpusq_dtype dt, int64_t B, int64_t C, int64_t H, int64_t W, int64_t P,
                                   int64_t K_pad, hipStream_t s) {
  if (dt == GPUSQ_I8) return launch_im2col_typed<int8_t>((const int8_t*)img, (int8_t*)X, B, C, H, W, P, K_pad, s);
  return launch_im2col_typed<_Float16>((const _Float16*)img, (_Float16*)X, B, C, H, W, P, K_pad, s);
}

gpusq_status launch_cast_f16(const float* in, void* out, int64_t n, hipStream_t s) {
  const int64_t want = ceil_div(n, 256 * 4);
  cast_f16_kernel<<<(unsigned)(want < 8192 ? want : 8192), 256, 0, s>>>(in, (_Float16*)out, n);
  return check_launch();
}

// n:m pruning [Sec. 5, limitation paragraph: 1:4, 2:16]: the n largest magnitudes of every M contiguous elements are kept
// (ties: the lower index).  One thread per group; an element is kept iff fewer than n elements beat it.
template <int M>
__global__ void __launch_bounds__(256) prune_n_of_m_kernel(const float4* __restrict__ in, float4* __restrict__ out, int n_keep,
                                                           int64_t groups) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= groups) return;
  float v[M];
#pragma unroll
  for (int q = 0; q < M / 4; ++q) {
    const float4 w = in[g * (M / 4) + q];
    v[4 * q] = w.x; v[4 * q + 1] = w.y; v[4 * q + 2] = w.z; v[4 * q + 3] = w.w;
  }
  unsigned key[M];
#pragma unroll
  for (int i = 0; i < M; ++i) key[i] = __float_as_uint(v[i]) & 0x7FFFFFFFu;
#pragma unroll
  for (int i = 0; i < M; ++i) {
    int beaten = 0;
#pragma unroll
    for (int j = 0; j < M; ++j)
      if (j != i) beaten += (j < i) ? (key[j] >= key[i]) : (key[j] > key[i]);
    if (beaten >= n_keep) v[i] = 0.0f;
  }
#pragma unroll
  for (int q = 0; q < M / 4; ++q) out[g * (M / 4) + q] = float4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
}

gpusq_status launch_prune_n_of_m(const float* Win, float* Wout, int n_keep, int m, int64_t N, int64_t K, hipStream_t s) {
  const int64_t groups = N * (K / m);
  const unsigned blocks = (unsigned)ceil_div(groups, 256);
  if (m == 4)
    prune_n_of_m_kernel<4><<<blocks, 256, 0, s>>>((const float4*)Win, (float4*)Wout, n_keep, groups);
  else if (m == 8)
    prune_n_of_m_kernel<8><<<blocks, 256, 0, s>>>((const float4*)Win, (float4*)Wout, n_keep, groups);
  else
    prune_n_of_m_kernel<16><<<blocks, 256, 0, s>>>((const float4*)Win, (float4*)Wout, n_keep, groups);
  return check_launch();
}

// ------------------------------------------------------------------------------------------------------------ quantise
__device__ __forceinline__ float load_as_f32(const float* p, int64_t i) { return p[i]; }
__device__ __forceinline__ float load_as_f32(const _Float16* p, int64_t i) { return (float)p[i]; }

// One wavefront per row (= per output channel), 4 rows per workgroup.
// Rows of whole vectors of VEC elements: a batch of kRowBatch vectors per lane is requested before the first is used, and a row of
// one batch stays in registers between the range and the codes; a longer one is read again.
// A load per loop turn, and two turns over the row, took a trip to memory each: 768 x 3072 fp32 11.0 us, 5.3 so.
template <typename T, int VEC, int kRowBatch, int QMAX>
__global__ void __launch_bounds__(256) quantize_rows_kernel(const T* __restrict__ X, int8_t* __restrict__ Q,
                                                            float* __restrict__ scale, int scale_is_input,
                                                            int64_t rows, int64_t cols) {
  constexpr float qmax = (float)QMAX;
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const T* x = X + row * cols;
  int8_t* q = Q + row * cols;
  float s;
  if (cols % VEC == 0) {
    const int64_t vecs = cols / VEC;
    vec_t v[kRowBatch];
    auto load = [&](int64_t base) {
#pragma unroll
      for (int j = 0; j < kRowBatch; ++j) {
        const int64_t i = base + j * 64 + lane;
        v[j] = i < vecs ? *(const vec_t*)(x + i * VEC) : vec_t(0);
      }
    };
    load(0);
    if (scale_is_input) {
      s = scale[row];
    } else {
      float amax = 0.0f;
      for (int64_t base = 0;;) {
#pragma unroll
        for (int j = 0; j < kRowBatch; ++j)
#pragma unroll
          for (int e = 0; e < VEC; ++e) amax = fmaxf(amax, fabsf((float)v[j][e]));
        base += kRowBatch * 64;
        if (base >= vecs) break;
        load(base);
      }
      amax = wave_max_magnitude(amax);
      s = (amax == 0.0f) ? 1.0f : __fdiv_rn(amax, qmax);
      if (lane == 0) scale[row] = s;
      if (vecs > kRowBatch * 64) load(0);
    }
    const float rs = scale_reciprocal(s);
    for (int64_t base = 0;;) {
#pragma unroll
      for (int j = 0; j < kRowBatch; ++j) {
        const int64_t i = base + j * 64 + lane;
        if (base + j * 64 >= vecs) break;  // wavefront-uniform
        float xs[VEC];
        unsigned w[VEC / 4];
#pragma unroll
        for (int e = 0; e < VEC; ++e) xs[e] = (float)v[j][e];
        quantize_words<VEC>(xs, s, rs, w, qmax);
        if (i < vecs) {
#pragma unroll
          for (int e = 0; e < VEC; e += 4) *(uint32_t*)(q + i * VEC + e) = w[e / 4];
        }
      }
      base += kRowBatch * 64;
      if (base >= vecs) break;
      load(base);
    }
    return;
  }
  if (scale_is_input) {
    s = scale[row];
  } else {
    float amax = 0.0f;
    for (int64_t c = lane; c < cols; c += 64) amax = fmaxf(amax, fabsf(load_as_f32(x, c)));
    amax = wave_max_magnitude(amax);
    s = (amax == 0.0f) ? 1.0f : __fdiv_rn(amax, qmax);
    if (lane == 0) scale[row] = s;
  }
  const float rs = scale_reciprocal(s);
  for (int64_t c = lane; c < cols; c += 64) q[c] = (int8_t)quantize_code(load_as_f32(x, c), s, rs, qmax);
}

// kRowBatch: the fewest of 1, 2, 4, 8 and 20 that hold a row (a batch of 8 for every short row: 12608 x 768 fp32 11.9 us, 10.2 so;
// 100000 x 64 41, 22), 8 for the longest.  With given scales there is no range to keep the row for, and more wavefronts
// hide the trips: 8 at most (4096 x 4096 fp32 20.0 us with 20, 14.7 so), 4 of the vectors of 8 (fp16 13.3 with 8, 12.8 so).
template <typename T, int VEC, int QMAX>
static void launch_quantize_rows_vec(const T* X, int8_t* Xq, float* scale, int scale_is_input, int64_t rows, int64_t cols, hipStream_t s) {
  const unsigned blocks = (unsigned)ceil_div(rows, 4);
  const int64_t per_lane = ceil_div(cols, VEC * 64);
#define GPUSQ_QUANTIZE_ROWS(B) quantize_rows_kernel<T, VEC, B, QMAX><<<blocks, 256, 0, s>>>(X, Xq, scale, scale_is_input, rows, cols)
  if (per_lane <= 1 || cols % VEC != 0) GPUSQ_QUANTIZE_ROWS(1);
  else if (per_lane <= 2) GPUSQ_QUANTIZE_ROWS(2);
  else if (per_lane <= 4 || (scale_is_input && VEC > 4)) GPUSQ_QUANTIZE_ROWS(4);
  else if (per_lane > 8 && per_lane <= 20 && !scale_is_input) GPUSQ_QUANTIZE_ROWS(20);
  else GPUSQ_QUANTIZE_ROWS(8);
#undef GPUSQ_QUANTIZE_ROWS
}
// Vectors of 16 bytes, or of 4 fp16 values where those leave fewer of a wavefront's lanes idle: what a vector costs is the arithmetic
// of its codes (100000 x 64 fp16 33 us with 8 values, 24 with 4; 12608 x 768 11.5 and 9.5).
template <typename T, int QMAX>
static gpusq_status launch_quantize_rows(const T* X, int8_t* Xq, float* scale, int scale_is_input, int64_t rows, int64_t cols, hipStream_t s) {
  constexpr int WIDE = 16 / (int)sizeof(T);
  if (WIDE > 4 && cols % WIDE == 0 && ceil_div(cols, 4 * 64) * 4 < ceil_div(cols, WIDE * 64) * WIDE)
    launch_quantize_rows_vec<T, 4, QMAX>(X, Xq, scale, scale_is_input, rows, cols, s);
  else
    launch_quantize_rows_vec<T, WIDE, QMAX>(X, Xq, scale, scale_is_input, rows, cols, s);
  return check_launch();
}

__global__ void fill_u32_kernel(uint32_t* p, uint32_t v) { *p = v; }

constexpr int kAmaxMaxBlocks = 1024;  // per-block partial maxima kept in the caller's workspace (4 KB)

__device__ __forceinline__ float block_max(float v) {
  __shared__ float part[4];
  v = wave_max_magnitude(v);
  __syncthreads();  // a previous use of part[] has been read
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
}

// The two passes of the per-tensor quantiser: the range, then the codes.  A workgroup takes blocks of 256 x 2 consecutive 16-byte
// vectors, every gridDim.x-th one, two vectors in flight per thread; both passes have the same grid, so that a workgroup id,
// and with it an XCD, meets the same blocks in both, and the second pass goes over them backwards: what the first one read last is
// still in that XCD's L2 (4 MB each, read at 12 TB/s where HBM and the memory-side cache give 6 to 7).
// Memory-bound, up to some 20 MB by what a workgroup does before its first code: fold the partial maxima, check its reciprocal
// (Fp16Quantiser).  So X is asked for before that, and there are no more than 1024 workgroups.  With the grids apart, the second pass
// forwards on 2048 workgroups and X waited for in front of the scale, both passes, us: 1576 x 768 fp16 5.9, now 5.2; 12544 x 512 10.3, 8.4;
// 12608 x 768 fp16 12.2, 10.0, fp32 16.9, 14.4; 25216 x 3072 fp16 70, 68, fp32 126, 116; a given scale: 12544 x 512 6.1, 5.1, 12608 x 768 7.4,
// 6.3.  (Four vectors in flight, 512 or 2048 workgroups: within 3 % or behind.)
constexpr int kQuantVecs = 2, kQuantBlock = 256 * kQuantVecs;

__device__ __forceinline__ float range_of_vec(const float4& v) { return fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))); }

// Per-tensor max |x|: one partial maximum per workgroup into the workspace; the second pass folds them (no atomics, nothing to
// clear beforehand).
template <typename T>
__global__ void __launch_bounds__(256) tensor_amax_kernel(const T* __restrict__ X, int64_t n, float* __restrict__ partial) {
  constexpr int VEC = 16 / (int)sizeof(T), U = kQuantVecs;
  typedef _Float16 h8 __attribute__((ext_vector_type(8)));
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  const int64_t vecs = n / VEC;
  float amax = 0.0f;
  h8 m = h8(0);
  const int64_t stride = (int64_t)gridDim.x * kQuantBlock;
  for (int64_t i = (int64_t)blockIdx.x * kQuantBlock + threadIdx.x; i < vecs; i += stride) {
    u4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = ((const u4*)X)[i + 256 * u < vecs ? i + 256 * u : i];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (VEC == 8)
        m = __builtin_elementwise_max(m, __builtin_bit_cast(h8, v[u] & 0x7fff7fffu));
      else
        amax = fmaxf(amax, range_of_vec(__builtin_bit_cast(float4, v[u])));
    }
  }
  if constexpr (VEC == 8) {
#pragma unroll
    for (int j = 0; j < 8; ++j) amax = fmaxf(amax, (float)m[j]);
  }
  if (blockIdx.x == 0 && vecs * VEC + threadIdx.x < n) amax = fmaxf(amax, fabsf(load_as_f32(X, vecs * VEC + threadIdx.x)));
  amax = block_max(amax);
  if (threadIdx.x == 0) partial[blockIdx.x] = amax;
}

// The codes, with the scale of the partial maxima (OWN) or a given one.  A workgroup has blocks_each blocks, the first blocks_over
// workgroups one more.
// (Stored with the non-temporal hint the two passes take 60 us instead of 69 on 25216 x 3072 fp16, but the GEMM behind them
// then finds its codes in HBM instead of the memory-side cache and loses more: 65792 x 1280 -> 5120 both together 394 -> 419.)
template <typename T, bool OWN>
__global__ void __launch_bounds__(256) quantize_tensor_kernel(const T* __restrict__ X, int8_t* __restrict__ Q,
                                                              float* __restrict__ scale, const float* __restrict__ partial,
                                                              int npartial, int64_t n, int blocks_each, int blocks_over,
                                                              bool backwards) {
  constexpr int VEC = 16 / (int)sizeof(T), U = kQuantVecs;
  typedef int i4 __attribute__((ext_vector_type(4)));
  constexpr int P = kAmaxMaxBlocks / 256;
  float known[P];
  auto ask = [&]() {
    if constexpr (OWN) {
#pragma unroll
      for (int j = 0; j < P; ++j) known[j] = partial[(int)threadIdx.x + 256 * j < npartial ? threadIdx.x + 256 * j : 0];
    } else {
      known[0] = scale[0];
    }
  };
  auto scale_of_known = [&]() {
    if constexpr (!OWN) return known[0];
    float amax = known[0];
#pragma unroll
    for (int j = 1; j < P; ++j) amax = fmaxf(amax, known[j]);
    amax = block_max(amax);
    const float s = (amax == 0.0f) ? 1.0f : __fdiv_rn(amax, 127.0f);
    if (blockIdx.x == 0 && threadIdx.x == 0) scale[0] = s;
    return s;
  };
  const int64_t vecs = n / VEC, stride = (int64_t)gridDim.x * kQuantBlock;
  auto tail = [&](float s, float rs) {
    if (blockIdx.x == 0 && vecs * VEC + threadIdx.x < n)
      Q[vecs * VEC + threadIdx.x] = (int8_t)quantize_code(load_as_f32(X, vecs * VEC + threadIdx.x), s, rs);
  };
  if (vecs == 0) {  // fewer values than a vector, one workgroup
    ask();
    const float s = scale_of_known();
    tail(s, scale_reciprocal(s));
    return;
  }
  // The partial maxima or the scale are asked for first and the first vectors of X right behind them, without a condition: the scale
  // and what is derived from it then take their time while X is on its way.
  ask();
  int left = blocks_each + ((int)blockIdx.x < blocks_over ? 1 : 0);  // this workgroup's blocks, at least one
  const int64_t step = backwards ? -stride : stride;
  int64_t at = (int64_t)blockIdx.x * kQuantBlock + (backwards ? (left - 1) * stride : 0) + threadIdx.x;
  i4 v[U];
  auto load = [&](int64_t i) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (OWN)
        v[u] = ((const i4*)X)[i + 256 * u < vecs ? i + 256 * u : vecs - 1];
      else if (i + 256 * u < vecs)
        v[u] = ((const i4*)X)[i + 256 * u];
    }
  };
  load(at);
  const float s = scale_of_known();
  const float rs = scale_reciprocal(s);
  Fp16Quantiser qz;
  if constexpr (VEC == 8) {
    __shared__ unsigned votes[4];
    const unsigned wave_votes = qz.prepare(s, threadIdx.x);
    if ((threadIdx.x & 63) == 0) votes[threadIdx.x >> 6] = wave_votes;
    __syncthreads();
    qz.decide((unsigned)__builtin_amdgcn_readfirstlane((int)(votes[0] | votes[1] | votes[2] | votes[3])));
  }
  while (left > 0) {
    unsigned q[U][2];
    if constexpr (VEC == 8) {
      const bool odd = qz.odd(v);
#pragma unroll
      for (int u = 0; u < U; ++u) qz.codes<!OWN>(v[u], odd, q[u][0], q[u][1]);
    } else {
#pragma unroll
      for (int u = 0; u < U; u += 2) {
        const float4 a = __builtin_bit_cast(float4, v[u]), b = __builtin_bit_cast(float4, v[u + 1]);
        const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        quantize_bytes8(x, s, rs, q[u][0], q[u + 1][0]);
      }
    }
    const int64_t here = at;
    at += step;
    if (--left > 0) load(at);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = here + 256 * u;
      if (i < vecs) {
        if constexpr (VEC == 8)
          ((uint2*)Q)[i] = uint2{q[u][0], q[u][1]};
        else
          ((uint32_t*)Q)[i] = q[u][0];
      }
    }
  }
  tail(s, rs);
}

// Workgroups of either pass for a tensor of that many bytes (no more than the workspace holds partial maxima).
static int quantize_grid(int64_t bytes) {
  const int64_t blocks = ceil_div(bytes / 16, kQuantBlock);
  return (int)(blocks < 1 ? 1 : (blocks < kAmaxMaxBlocks ? blocks : kAmaxMaxBlocks));
}

template <typename T>
static int launch_amax_typed(const T* X, int64_t n, float* partial, hipStream_t s) {
  const int grid = quantize_grid(n * (int64_t)sizeof(T));
  tensor_amax_kernel<T><<<(unsigned)grid, 256, 0, s>>>(X, n, partial);
  return grid;
}

int launch_amax(const void* X, gpusq_dtype dt, int64_t n, void* workspace, hipStream_t s) {
  return dt == GPUSQ_F32 ? launch_amax_typed((const float*)X, n, (float*)workspace, s)
                         : launch_amax_typed((const _Float16*)X, n, (float*)workspace, s);
}

template <typename T>
static gpusq_status quantize_typed(const T* X, int8_t* Xq, float* scale, int mode, int scale_is_input, int64_t rows,
                                   int64_t cols, void* workspace, hipStream_t s) {
  if (mode == GPUSQ_PER_ROW) {
    return launch_quantize_rows<T, 127>(X, Xq, scale, scale_is_input, rows, cols, s);
  }
  const int64_t n = rows * cols, bytes = n * (int64_t)sizeof(T);
  const int grid = quantize_grid(bytes);
  const int64_t blocks = ceil_div(bytes / 16, kQuantBlock);
  const int each = (int)(blocks / grid), over = (int)(blocks % grid);
  if (scale_is_input) {
    quantize_tensor_kernel<T, false><<<(unsigned)grid, 256, 0, s>>>(X, Xq, scale, nullptr, 0, n, each, over, false);
    return check_launch();
  }
  // (large fp16 tensors, of which little is left in the L2s, forwards: as fast, and the GEMM behind them 2 % faster)
  const bool backwards = sizeof(T) == 4 || bytes <= ((int64_t)96 << 20);
  launch_amax_typed<T>(X, n, (float*)workspace, s);
  quantize_tensor_kernel<T, true><<<(unsigned)grid, 256, 0, s>>>(X, Xq, scale, (const float*)workspace, grid, n, each, over, backwards);
  return check_launch();
}

gpusq_status launch_quantize(const void* X, gpusq_dtype dt, int8_t* Xq, float* scale, int mode, int scale_is_input,
                             int64_t rows, int64_t cols, void* workspace, hipStream_t s) {
  if (dt == GPUSQ_F32) return quantize_typed<float>((const float*)X, Xq, scale, mode, scale_is_input, rows, cols, workspace, s);
  return quantize_typed<_Float16>((const _Float16*)X, Xq, scale, mode, scale_is_input, rows, cols, workspace, s);
}

// ---- per-tensor quantiser for callers that cannot allocate -------------------------------------------------------
// The per-workgroup partial maxima of the range pass live in this file-scope device array instead of a caller's
// workspace.  Every GPU the library runs on holds its own copy until the process ends; its address on a device is
// looked up once per device (hipGetSymbolAddress with that device current) and kept.  The array's name is only a
// host-side handle: host code passes the looked-up pointer to the kernels, never the name.
static __device__ __align__(256) float g_amax_scratch[kAmaxMaxBlocks];

static float* amax_scratch_of_current_device(gpusq_status* st) {
  constexpr int kMaxDevices = 64;
  static std::atomic<float*> ptrs[kMaxDevices];
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    if (e != hipSuccess) set_last_hip_error(e);
    *st = e != hipSuccess ? GPUSQ_ERR_HIP : GPUSQ_ERR_UNSUPPORTED;
    return nullptr;
  }
  float* p = ptrs[dev].load(std::memory_order_acquire);
  if (!p) {
    void* sym = nullptr;
    e = hipGetSymbolAddress(&sym, HIP_SYMBOL(g_amax_scratch));
    if (e != hipSuccess || !sym) {
      set_last_hip_error(e);
      *st = GPUSQ_ERR_HIP;
      return nullptr;
    }
    p = (float*)sym;
    ptrs[dev].store(p, std::memory_order_release);  // (a racing first call looks up the same address)
  }
  *st = GPUSQ_OK;
  return p;
}

gpusq_status launch_quantize_tensor_static(const void* X, gpusq_dtype dt, int8_t* Xq, float* scale, int scale_is_input,
                                           int64_t rows, int64_t cols, hipStream_t s) {
  float* scratch = nullptr;
  if (!scale_is_input) {  // a given scale needs no range pass and no scratch
    gpusq_status st;
    scratch = amax_scratch_of_current_device(&st);
    if (!scratch) return st;
  }
  // Nothing has to be cleared: the range pass overwrites the partial maxima the quantising pass reads (the same
  // number of them in both launches), whatever an earlier call left behind.
  return launch_quantize(X, dt, Xq, scale, GPUSQ_PER_TENSOR, scale_is_input, rows, cols, scratch, s);
}

// The same per-row quantiser with the 4-bit range: codes -7..7 in int8 containers, scale = max|row| / 7.
gpusq_status launch_quantize_rows_int4(const void* X, gpusq_dtype dt, int8_t* Xq, float* scale, int scale_is_input, int64_t rows,
                                       int64_t cols, hipStream_t s) {
  if (dt == GPUSQ_F32) return launch_quantize_rows<float, 7>((const float*)X, Xq, scale, scale_is_input, rows, cols, s);
  return launch_quantize_rows<_Float16, 7>((const _Float16*)X, Xq, scale, scale_is_input, rows, cols, s);
}

// ------------------------------------------------------------------------------------------------------------ compress
// One lane per metadata byte = per pair of groups (the last byte of a row holds one group when K/4 is odd).
template <typename T>
__device__ __forceinline__ unsigned magnitude_key(T v);
template <>
__device__ __forceinline__ unsigned magnitude_key<uint32_t>(uint32_t v) { return v & 0x7FFFFFFFu; }
template <>
__device__ __forceinline__ unsigned magnitude_key<uint16_t>(uint16_t v) { return v & 0x7FFFu; }
template <>
__device__ __forceinline__ unsigned magnitude_key<int8_t>(int8_t v) { return (unsigned)(v < 0 ? -(int)v : (int)v); }

template <typename T>
__global__ void __launch_bounds__(256) compress_kernel(const T* __restrict__ W, T* __restrict__ values,
                                                       uint8_t* __restrict__ meta, int32_t* __restrict__ violations,
                                                       int64_t N, int64_t K) {
  const int64_t groups_per_row = K / 4;
  const int64_t mrb = (groups_per_row + 1) / 2;
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int bad = 0;
  if (id < N * mrb) {
    const int64_t n = id / mrb, b = id % mrb;
    unsigned byte = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t g = 2 * b + h;
      if (g < groups_per_row) {
        const T* w = W + n * K + 4 * g;
        const T w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3];
        const unsigned k0 = magnitude_key<T>(w0), k1 = magnitude_key<T>(w1), k2 = magnitude_key<T>(w2), k3 = magnitude_key<T>(w3);
        const unsigned m = keep_mask_of_4(k0, k1, k2, k3);
        const unsigned nib = nibble_of_mask(m);
        const unsigned p0 = nib & 3u, p1 = nib >> 2;
        const T v0 = p0 == 0 ? w0 : (p0 == 1 ? w1 : w2);
        const T v1 = p1 == 1 ? w1 : (p1 == 2 ? w2 : w3);
        values[n * (K / 2) + 2 * g] = v0;
        values[n * (K / 2) + 2 * g + 1] = v1;
        byte |= nib << (4 * h);
        bad += (int)(((m & 1u) == 0 && k0 != 0) || ((m & 2u) == 0 && k1 != 0) || ((m & 4u) == 0 && k2 != 0) ||
                     ((m & 8u) == 0 && k3 != 0));
      }
    }
    meta[n * mrb + b] = (uint8_t)byte;
  }
  if (violations) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) bad += __shfl_xor(bad, o, 64);
    if ((threadIdx.x & 63) == 0 && bad) atomicAdd(violations, bad);
  }
}

gpusq_status launch_compress(const void* W, void* values, uint8_t* meta, int32_t* violations, gpusq_dtype dt,
                             int64_t N, int64_t K, hipStream_t s) {
  const int64_t mrb = (K / 4 + 1) / 2;
  const unsigned blocks = (unsigned)ceil_div(N * mrb, 256);
  if (violations) fill_u32_kernel<<<1, 1, 0, s>>>((uint32_t*)violations, 0u);
  if (dt == GPUSQ_F16)
    compress_kernel<uint16_t><<<blocks, 256, 0, s>>>((const uint16_t*)W, (uint16_t*)values, meta, violations, N, K);
  else
    compress_kernel<int8_t><<<blocks, 256, 0, s>>>((const int8_t*)W, (int8_t*)values, meta, violations, N, K);
  return check_launch();
}

// Groups of 4 along K with more than two non-zero elements (Sec. 3.1: a 2:4 tensor keeps at most two of every four).
// One thread per 16 bytes of a row (4 groups of fp32 ... 16 of int8: K % 4 == 0 makes rows whole groups, the pointer is
// 16-byte aligned, and the tail of the tensor that does not fill 16 bytes goes element by element); -0 counts as zero.
template <typename T>
__global__ void __launch_bounds__(256) count_violations_kernel(const T* __restrict__ W, int32_t* __restrict__ violations, int64_t elems) {
  constexpr int PER = 16 / (int)sizeof(T);  // elements per 16-byte piece: whole groups
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t e0 = id * PER;
  int bad = 0;
  if (e0 < elems) {
    alignas(16) T w[PER];
    if (e0 + PER <= elems) {
      *(uint4*)w = *(const uint4*)(W + e0);
    } else {
      for (int i = 0; i < PER; ++i) w[i] = e0 + i < elems ? W[e0 + i] : (T)0;
    }
#pragma unroll
    for (int g = 0; g < PER / 4; ++g) {
      int nz = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) nz += (int)(magnitude_key<T>(w[4 * g + i]) != 0u);
      bad += (int)(nz > 2);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) bad += __shfl_xor(bad, o, 64);
  if ((threadIdx.x & 63) == 0 && bad) atomicAdd(violations, bad);
}

gpusq_status launch_count_violations(const void* W, gpusq_dtype dt, int32_t* violations, int64_t N, int64_t K, hipStream_t s) {
  const int64_t elems = N * K;
  fill_u32_kernel<<<1, 1, 0, s>>>((uint32_t*)violations, 0u);
  if (dt == GPUSQ_F32)
    count_violations_kernel<uint32_t><<<(unsigned)ceil_div(ceil_div(elems, 4), 256), 256, 0, s>>>((const uint32_t*)W, violations, elems);
  else if (dt == GPUSQ_F16)
    count_violations_kernel<uint16_t><<<(unsigned)ceil_div(ceil_div(elems, 8), 256), 256, 0, s>>>((const uint16_t*)W, violations, elems);
  else
    count_violations_kernel<int8_t><<<(unsigned)ceil_div(ceil_div(elems, 16), 256), 256, 0, s>>>((const int8_t*)W, violations, elems);
  return check_launch();
}

template <typename T>
__global__ void __launch_bounds__(256) decompress_kernel(const T* __restrict__ values, const uint8_t* __restrict__ meta,
                                                         T* __restrict__ W, int64_t N, int64_t K) {
  const int64_t groups_per_row = K / 4;
  const int64_t mrb = (groups_per_row + 1) / 2;
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= N * mrb) return;
  const int64_t n = id / mrb, b = id % mrb;
  const unsigned byte = meta[n * mrb + b];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int64_t g = 2 * b + h;
    if (g < groups_per_row) {
      const unsigned nib = (byte >> (4 * h)) & 0xFu;
      const unsigned p0 = nib & 3u, p1 = nib >> 2;
      const T v0 = values[n * (K / 2) + 2 * g], v1 = values[n * (K / 2) + 2 * g + 1];
      T* w = W + n * K + 4 * g;
#pragma unroll
      for (unsigned i = 0; i < 4; ++i) w[i] = (i == p0) ? v0 : ((i == p1) ? v1 : (T)0);
    }
  }
}

gpusq_status launch_decompress(const void* values, const uint8_t* meta, void* W, gpusq_dtype dt, int64_t N, int64_t K,
                               hipStream_t s) {
  const int64_t mrb = (K / 4 + 1) / 2;
  const unsigned blocks = (unsigned)ceil_div(N * mrb, 256);
  if (dt == GPUSQ_F16)
    decompress_kernel<uint16_t><<<blocks, 256, 0, s>>>((const uint16_t*)values, meta, (uint16_t*)W, N, K);
  else
    decompress_kernel<int8_t><<<blocks, 256, 0, s>>>((const int8_t*)values, meta, (int8_t*)W, N, K);
  return check_launch();
}

// ------------------------------------------------------------------------------------------------------------ pack
// Re-tiles the canonical (values, meta) arrays into the packed tile format described in common.h.
// Lane l of fragment f (0..15) of tile (nb, ks) serves output channel nb*256 + 64*(f/4) + packed_row_to_channel(f%4,
// l%16) and the dense K range [ks*E + (l/16)*E/4, +E/4) with E = elements per step; the sparse matrix instruction
// wants, per lane, the kept values of that range in order (16 bytes) and their 2-bit positions in order starting at
// bit 0 of the index register.  Both are contiguous byte runs of the canonical arrays:
// values[n][k0/2 .. k0/2 + kept) and meta[n][k0/8 ..).  Rows >= N and K beyond the row end are zero-filled.
// WHOLE: K is a multiple of a lane's range (32 int8, 16 fp16 elements), so a run is one 16-byte and one 4-byte (2-byte) load;
// byte by byte the 5120 x 1280 int8 operand took 11.6 us.
template <bool IS_I8, bool WHOLE>
__global__ void __launch_bounds__(256) pack_kernel(const uint8_t* __restrict__ values, const uint8_t* __restrict__ meta,
                                                   uint8_t* __restrict__ packed, int64_t N, int64_t K, int ksteps,
                                                   int64_t total_lanes) {
  constexpr int E = step_elems(IS_I8);  // dense elements per step
  constexpr int ES = IS_I8 ? 1 : 2;     // element size
  constexpr int KL = E / 4;             // dense elements per lane
  constexpr int IB = IS_I8 ? 4 : 2;     // index bytes per lane
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= total_lanes) return;
  const int lane = (int)(id & 63);
  const int f = (int)((id >> 6) & 15);
  const int64_t tile = id >> 10;
  const int64_t nb = (unsigned)tile / (unsigned)ksteps, ks = (unsigned)tile - (unsigned)nb * (unsigned)ksteps;  // (fewer than 2^32 tiles)
  const int64_t n = nb * kTileRows + (f >> 2) * kRowBlock + packed_row_to_channel(f & 3, lane & 15);
  const int64_t k0 = ks * E + (int64_t)(lane >> 4) * KL;  // first dense element of this lane
  const int64_t mrb = (K / 4 + 1) / 2;
  uint8_t* t = packed + tile * tile_bytes(IS_I8);
  uint8_t* ip = t + index_offset(IS_I8, f, lane);
  if (WHOLE) {  // every lane's run lies inside a row or past its end, and is aligned
    uint4 vv = uint4{0, 0, 0, 0};
    uint32_t ix = 0;
    if (n < N && k0 < K) {
      vv = *(const uint4*)(values + (n * (K / 2) + k0 / 2) * ES);
      if constexpr (IS_I8)
        ix = *(const uint32_t*)(meta + n * (K / 8) + k0 / 8);
      else
        ix = *(const uint16_t*)(meta + n * (K / 8) + k0 / 8);
    }
    *(uint4*)(t + f * kFragValueBytes + lane * 16) = vv;
    if constexpr (IS_I8)
      *(uint32_t*)ip = ix;
    else
      *(uint16_t*)ip = (uint16_t)ix;
    return;
  }
  uint8_t v[16];
  uint8_t ix[IB];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int64_t byte = (k0 / 2) * ES + i;  // byte offset inside the row of kept values
    v[i] = (n < N && byte < (K / 2) * ES) ? values[n * (K / 2) * ES + byte] : (uint8_t)0;
  }
#pragma unroll
  for (int i = 0; i < IB; ++i) {
    const int64_t byte = k0 / 8 + i;
    // padding (rows >= N, K beyond the row end) carries zero values; its positions are irrelevant
    ix[i] = (n < N && byte < mrb) ? meta[n * mrb + byte] : (uint8_t)0;
  }
  uint4 vv;
  vv.x = v[0] | (v[1] << 8) | (v[2] << 16) | ((uint32_t)v[3] << 24);
  vv.y = v[4] | (v[5] << 8) | (v[6] << 16) | ((uint32_t)v[7] << 24);
  vv.z = v[8] | (v[9] << 8) | (v[10] << 16) | ((uint32_t)v[11] << 24);
  vv.w = v[12] | (v[13] << 8) | (v[14] << 16) | ((uint32_t)v[15] << 24);
  *(uint4*)(t + f * kFragValueBytes + lane * 16) = vv;
  if constexpr (IS_I8)
    *(uint32_t*)ip = ix[0] | (ix[1] << 8) | (ix[2] << 16) | ((uint32_t)ix[3] << 24);
  else
    *(uint16_t*)ip = (uint16_t)(ix[0] | (ix[1] << 8));
}

gpusq_status launch_pack(const void* values, const uint8_t* meta, void* packed, gpusq_dtype dt, int64_t N, int64_t K,
                         hipStream_t s) {
  const bool is_i8 = dt == GPUSQ_I8;
  const int64_t ksteps = ceil_div(K, step_elems(is_i8));
  const int64_t tiles = ceil_div(N, kTileRows) * ksteps;
  const int64_t total_lanes = tiles * 16 * 64;
  const unsigned blocks = (unsigned)ceil_div(total_lanes, 256);
  const bool whole = K % (step_elems(is_i8) / 4) == 0;
#define GPUSQ_PACK(I8, WH) pack_kernel<I8, WH><<<blocks, 256, 0, s>>>((const uint8_t*)values, meta, (uint8_t*)packed, N, K, (int)ksteps, total_lanes)
  if (is_i8 && whole) GPUSQ_PACK(true, true);
  else if (is_i8) GPUSQ_PACK(true, false);
  else if (whole) GPUSQ_PACK(false, true);
  else GPUSQ_PACK(false, false);
#undef GPUSQ_PACK
  return check_launch();
}

// ------------------------------------------------------------------------------------------------------------ fused
// The two kept elements of a group of 4 and their positions: the selection rule of keep_mask_of_4 on lane masks (element i is dropped iff two
// or more of the others beat it, where of a pair the second beats the first iff it is larger: six comparisons, the rest is scalar logic).
struct KeptPair {
  float first, second;
  unsigned p0, p1;
  bool keep[4];
  __device__ __forceinline__ explicit KeptPair(const float4& x) {
    const unsigned k0 = __float_as_uint(x.x) & 0x7FFFFFFFu, k1 = __float_as_uint(x.y) & 0x7FFFFFFFu;
    const unsigned k2 = __float_as_uint(x.z) & 0x7FFFFFFFu, k3 = __float_as_uint(x.w) & 0x7FFFFFFFu;
    const bool c01 = k1 > k0, c02 = k2 > k0, c03 = k3 > k0, c12 = k2 > k1, c13 = k3 > k1, c23 = k3 > k2;
    auto two_of = [](bool p, bool q, bool r) { return (p & q) | (r & (p | q)); };
    keep[0] = !two_of(c01, c02, c03);
    keep[1] = !two_of(!c01, c12, c13);
    keep[2] = !two_of(!c02, !c12, c23);
    keep[3] = !two_of(!c03, !c13, !c23);
    p0 = keep[0] ? 0u : (keep[1] ? 1u : 2u);
    p1 = keep[3] ? 3u : (keep[2] ? 2u : 1u);
    first = keep[0] ? x.x : (keep[1] ? x.y : x.z);
    second = keep[3] ? x.w : (keep[2] ? x.z : x.y);
  }
};
// The positions recorded are those of the rule applied to the low-precision group (kept: its two values), which differ from the
// fp32 group's only where a kept value became zero: then zeros are kept from the lowest index on.
template <bool IS_I8>
__device__ __forceinline__ void low_precision_positions(unsigned& kept, unsigned& p0, unsigned& p1) {
  constexpr int BITS = IS_I8 ? 8 : 16;
  constexpr unsigned ONE = (1u << BITS) - 1u, MAGNITUDE = IS_I8 ? 0xFFu : 0x7FFFu;
  const uint64_t group = ((uint64_t)(kept & ONE) << (BITS * p0)) | ((uint64_t)(kept >> BITS) << (BITS * p1));
  unsigned nz = 0;  // the non-zero elements of the low-precision group: at most two, and they come first
#pragma unroll
  for (int i = 0; i < 4; ++i) nz |= (unsigned)(((unsigned)(group >> (BITS * i)) & MAGNITUDE) != 0) << i;
  const unsigned nib = nibble_of_mask(keep_mask_of_4(nz & 1u, (nz >> 1) & 1u, (nz >> 2) & 1u, (nz >> 3) & 1u));
  p0 = nib & 3u;
  p1 = nib >> 2;
  kept = ((unsigned)(group >> (BITS * p0)) & ONE) | (((unsigned)(group >> (BITS * p1)) & ONE) << BITS);
}
// The positions of a packed lane's GU (4 or 8) groups, the first group's in the low nibble: exchanged inside its lanes
// (quad_perm 1,0,3,2 = 0xB1, quad_perm 2,3,0,1 = 0x4E, row_half_mirror = 0x141)
template <int GU>
__device__ __forceinline__ unsigned lane_positions(unsigned nib, int lane) {
  unsigned ix = nib << (4 * (lane & (GU - 1)));
  ix |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)ix, 0xB1, 0xF, 0xF, true);
  ix |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)ix, 0x4E, 0xF, 0xF, true);
  if constexpr (GU == 8) ix |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)ix, 0x141, 0xF, 0xF, true);
  return ix;
}
// Workgroup id -> (64-channel block, fragment t of it, ROWS of its 16 rows), the last varying fastest; the ids that share a
// line (8 rows) go to workgroups 8 apart, which the dispatcher places on one XCD.
template <int ROWS>
__device__ __forceinline__ int prepare_place() {
  constexpr int SHARE = 8 / ROWS;
  const int id = (int)blockIdx.x;
  return (id & ~(8 * SHARE - 1)) | ((id & 7) * SHARE) | ((id >> 3) & (SHARE - 1));
}

// prune -> (INT8: per-output-channel quantise | FP16: round) -> compress -> pack for one weight matrix in one launch.
// One wavefront per output channel, one lane per group of 4: a lane prunes its group, quantises or rounds it, applies the
// compression rule to the low-precision group and writes its two kept values and its positions to every requested output.
// All arithmetic is the same sequence of operations as the separate kernels above, so the results are bit-identical to running
// them in turn.  (Pruning never removes the row maximum, so the maximum of the row is that of the pruned row.)
// What bounds it is latency: the row, its maximum, the codes.  So a row's groups are requested in batches of kPrepBatch per
// lane, all before the first is used, and a row of one batch stays in registers (a longer one is read twice, the second time
// from the L2); the maximum takes data-parallel primitives (wave_max_magnitude).  Rows of more than 2048 elements are dealt out over WPR = 4 wavefronts
// (768 x 3072: with one wavefront per row the chip has fewer wavefronts than SIMDs).  A workgroup takes 4 (WPR = 4: 1) rows of
// a fragment, and the workgroups whose packed lanes share 128-byte lines run on one XCD.  The rows of the packed
// tiles past N and the K range past the row end are written (zero) by the wavefronts that own them.
// With a thread per 32 elements, LDS for the rows and one load in flight per thread, int8: 3072 x 768 9.8 us, 6.0 so; 768 x
// 3072 10.0, 6.1 so; 5120 x 1280 17.3, 12.2 so.  Workgroups of 256 threads: with 512 and 1024 the 1280 x 5120 take 16 and 20
// us instead of 13 (their last round is thin), and WPR = 4 at K = 768 12 instead of 6 (one row per workgroup).
constexpr int kPrepBatch = 8;
template <bool IS_I8, int WPR>
__global__ void __launch_bounds__(256) prepare_weights_kernel(const float* __restrict__ W, float* __restrict__ Wp,
                                                              uint8_t* __restrict__ Wlow, float* __restrict__ w_scale,
                                                              uint8_t* __restrict__ values, uint8_t* __restrict__ meta,
                                                              uint8_t* __restrict__ packed, int64_t N, int64_t K, int ksteps) {
  constexpr int GS = step_elems(IS_I8) / 4;   // groups per K step
  constexpr int GU = GS / 4;                  // groups per packed lane
  constexpr int GB = 16 / GU;                 // bytes of kept values per group
  constexpr int B = kPrepBatch;
  constexpr int ROWS = 4 / WPR, STRIDE = 64 * WPR;  // rows of a workgroup; groups between a lane's consecutive ones
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int id = prepare_place<ROWS>();
  constexpr int PER_FRAG = 16 / ROWS;
  const int blk = id / (4 * PER_FRAG), t = (id / PER_FRAG) & 3, r = ROWS * (id % PER_FRAG) + wave / WPR;
  const int64_t n = (int64_t)blk * kRowBlock + packed_row_to_channel(t, r);
  const bool live = n < N;  // wavefront-uniform
  const int groups = live ? (int)(K / 4) : 0, padded = ksteps * GS;
  const int start = (wave % WPR) * 64;  // this wavefront's first group
  const float4* row = (const float4*)(W + (live ? n : 0) * K);
  float4 v[B];
  auto load = [&](int base) {
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const int g = base + j * STRIDE + lane;
      v[j] = g < groups ? row[g] : float4{0.0f, 0.0f, 0.0f, 0.0f};
    }
  };
  load(start);
  float s = 1.0f;
  if constexpr (IS_I8) {
    float amax = 0.0f;
    for (int base = start;;) {
#pragma unroll
      for (int j = 0; j < B; ++j) amax = fmaxf(fmaxf(amax, fmaxf(fabsf(v[j].x), fabsf(v[j].y))), fmaxf(fabsf(v[j].z), fabsf(v[j].w)));
      base += B * STRIDE;
      if (base >= groups) break;
      load(base);
    }
    amax = wave_max_magnitude(amax);
    if constexpr (WPR > 1) {
      __shared__ float part[ROWS * WPR];
      if (lane == 0) part[wave] = amax;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < WPR; ++w) amax = fmaxf(amax, part[wave / WPR * WPR + w]);
    }
    s = (amax == 0.0f) ? 1.0f : __fdiv_rn(amax, 127.0f);
    if (live && start == 0 && lane == 0) w_scale[n] = s;
    if (start + B * STRIDE < groups) load(start);
  }
  const float rs = scale_reciprocal(s);
  const int64_t mrb = (K / 4 + 1) / 2;
  const int f = (blk & 3) * 4 + t;  // fragment of the packed tile
  uint8_t* column = packed + (n / kTileRows) * ksteps * tile_bytes(IS_I8);
  for (int base = start; base < padded;) {
#pragma unroll
    for (int j = 0; j < B; ++j) {
      if (base + j * STRIDE >= padded) break;  // wavefront-uniform
      const int g = base + j * STRIDE + lane;
      const float4 x = v[j];
      const KeptPair two(x);
      const bool keep0 = two.keep[0], keep1 = two.keep[1], keep2 = two.keep[2], keep3 = two.keep[3];
      const float first = two.first, second = two.second;
      unsigned p0 = two.p0, p1 = two.p1;
      const bool in_row = g < groups;
      if (Wp && in_row) *(float4*)(Wp + n * K + 4 * g) = float4{keep0 ? x.x : 0.0f, keep1 ? x.y : 0.0f, keep2 ? x.z : 0.0f, keep3 ? x.w : 0.0f};
      // the two kept values in low precision
      unsigned kept;
      bool zero;
      if constexpr (IS_I8) {
        const float xs[2] = {first, second};
        int q[2];
        quantize_codes<2>(xs, s, rs, q);
        kept = (unsigned)(q[0] & 0xFF) | ((unsigned)(q[1] & 0xFF) << 8);
        zero = q[0] == 0 || q[1] == 0;
      } else {
        const unsigned h0 = __builtin_bit_cast(unsigned short, (_Float16)first), h1 = __builtin_bit_cast(unsigned short, (_Float16)second);
        kept = h0 | (h1 << 16);
        zero = (h0 & 0x7FFFu) == 0 || (h1 & 0x7FFFu) == 0;
      }
      if (Wlow && in_row) {
        if constexpr (IS_I8)
          *(uint32_t*)(Wlow + n * K + 4 * g) = ((kept & 0xFFu) << (8 * p0)) | ((kept >> 8) << (8 * p1));
        else
          *(uint64_t*)(Wlow + (n * K + 4 * g) * 2) = ((uint64_t)(kept & 0xFFFFu) << (16 * p0)) | ((uint64_t)(kept >> 16) << (16 * p1));
      }
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(zero) != 0, 0)) low_precision_positions<IS_I8>(kept, p0, p1);
      const unsigned nib = in_row ? p0 | (p1 << 2) : 0u;
      const unsigned ix = lane_positions<GU>(nib, lane);
      if (in_row) {
        if (values) {
          if constexpr (IS_I8)
            *(uint16_t*)(values + n * (K / 2) + 2 * g) = (uint16_t)kept;
          else
            *(uint32_t*)(values + (n * (K / 2) + 2 * g) * 2) = kept;
        }
        if (meta && (g & 1) == 0) meta[n * mrb + (g >> 1)] = (uint8_t)(ix >> (4 * (lane & (GU - 1))));
      }
      if (g < padded) {
        const int ks = g / GS, q4 = (g & (GS - 1)) / GU, in_lane = g & (GU - 1);
        uint8_t* tp = column + (int64_t)ks * tile_bytes(IS_I8);
        uint8_t* vp = tp + f * kFragValueBytes + (r + 16 * q4) * 16 + in_lane * GB;
        if constexpr (IS_I8)
          *(uint16_t*)vp = (uint16_t)kept;
        else
          *(uint32_t*)vp = kept;
        if (in_lane == 0) {
          uint8_t* ip = tp + index_offset(IS_I8, f, r + 16 * q4);
          if constexpr (IS_I8)
            *(uint32_t*)ip = ix;
          else
            *(uint16_t*)ip = (uint16_t)ix;
        }
      }
    }
    base += B * STRIDE;
    if (base < padded) load(base);
  }
}

// The same where only what the sparse GEMM reads is asked for (packed operand, scales): a row stays in B registers of 16 bytes per
// lane (B = 8: or comes in batches of 8), loads and stores have a wavefront's address and a 32-bit lane offset that grows by a constant,
// an int8 code takes some four operations (see ByteQuantiser), and what few wavefronts run stands behind.  Some 45 vector instructions for a
// group of 4 where the kernel above takes 130; with its 114 registers it also leaves a fifth of the wavefronts of 5120 x 1280 to a
// second round.  5120 x 1280 int8 12.3 us, 9.2 so; fp16 10.5, 9.3; 3072 x 768 int8 6.6, 4.8; 768 x 192 3.4, 2.5.  What is left is one burst: all
// rows are asked for at once and come at some 6 TB/s.
// The 32-bit offsets inside a row and inside a column of packed tiles hold K up to kPrepareMaxK with much to spare.
template <bool IS_I8, int WPR, int B>
__global__ void __launch_bounds__(256) prepare_packed_kernel(const float* __restrict__ W, float* __restrict__ w_scale,
                                                             uint8_t* __restrict__ packed, int64_t N, int K, int ksteps) {
  constexpr int GS = step_elems(IS_I8) / 4;  // groups per K step
  constexpr int GU = GS / 4;                 // groups per packed lane
  constexpr int GB = 16 / GU;                // bytes of kept values per group
  constexpr int ROWS = 4 / WPR, STRIDE = 64 * WPR, PER_FRAG = 16 / ROWS;
  constexpr bool ONE_BATCH = B < kPrepBatch;
  static_assert(STRIDE % GS == 0, "a lane's groups lie at the same place of their K steps");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int id = prepare_place<ROWS>(), blk = id / (4 * PER_FRAG), t = (id / PER_FRAG) & 3, r = ROWS * (id % PER_FRAG) + wave / WPR;
  const int64_t n = (int64_t)blk * kRowBlock + packed_row_to_channel(t, r);
  const bool live = n < N;  // wavefront-uniform, as all that follows from the wavefront's number
  const int groups = live ? K / 4 : 0, last = live ? K / 4 - 1 : 0, padded = ksteps * GS, start = (wave % WPR) * 64;
  const uint8_t* row = (const uint8_t*)(W + (live ? n : 0) * K);
  float4 v[B];
  auto load = [&](int base) {  // (groups past the end re-read the last one; they count as zeros below)
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const int g = base + j * STRIDE + lane;
      v[j] = *(const float4*)(row + 16u * (uint32_t)(g < last ? g : last));
    }
  };
  load(start);
  float s = 1.0f;
  if constexpr (IS_I8) {
    float amax = 0.0f;
    for (int base = start;;) {
#pragma unroll
      for (int j = 0; j < B; ++j) amax = fmaxf(fmaxf(amax, fmaxf(fabsf(v[j].x), fabsf(v[j].y))), fmaxf(fabsf(v[j].z), fabsf(v[j].w)));
      base += B * STRIDE;
      if (ONE_BATCH || base >= groups) break;
      load(base);
    }
    amax = wave_max_magnitude(amax);
    if constexpr (WPR > 1) {
      __shared__ float part[ROWS * WPR];
      if (lane == 0) part[wave] = amax;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < WPR; ++w) amax = fmaxf(amax, part[wave / WPR * WPR + w]);
    }
    s = (amax == 0.0f) ? 1.0f : __fdiv_rn(amax, 127.0f);
    if (live && start == 0 && lane == 0) w_scale[n] = s;
    if (!ONE_BATCH && start + B * STRIDE < groups) load(start);
  }
  const ByteQuantiser bq(s, IS_I8 ? scale_reciprocal(s) : 1.0f);
  const int f = (blk & 3) * 4 + t;  // fragment of the packed tile
  uint8_t* column = packed + (n / kTileRows) * ksteps * tile_bytes(IS_I8);
  const int q4 = (lane & (GS - 1)) / GU, in_lane = lane & (GU - 1);
  const uint32_t first_step = (uint32_t)((start + lane) / GS) * tile_bytes(IS_I8);
  uint32_t value_at = first_step + f * kFragValueBytes + (r + 16 * q4) * 16 + in_lane * GB, index_at = first_step + index_offset(IS_I8, f, r + 16 * q4);
  for (int base = start; base < padded;) {
#pragma unroll
    for (int j = 0; j < B; ++j) {
      if (base + j * STRIDE >= padded) break;  // wavefront-uniform
      const int g = base + j * STRIDE + lane;
      KeptPair two(v[j]);
      unsigned kept;
      bool zero;
      if constexpr (IS_I8) {
        int u[2];
        bq.units(two.first, u[0]);
        bq.units(two.second, u[1]);
        const unsigned short l0 = (unsigned short)u[0], l1 = (unsigned short)u[1];
        if (__builtin_expect(__builtin_amdgcn_ballot_w64((l0 < l1 ? l0 : l1) < ByteQuantiser::kNear) != 0, 0)) {
          u[0] = finish_code(__fdiv_rn(two.first, s)) * 65536;
          u[1] = finish_code(__fdiv_rn(two.second, s)) * 65536;
        }
        kept = __builtin_amdgcn_perm((unsigned)u[1], (unsigned)u[0], 0x0c0c0602u);  // (no quotient reaches 127.5 here)
        zero = (kept & 0xFFu) == 0 || kept < 0x100u;
      } else {
        const unsigned h0 = __builtin_bit_cast(unsigned short, (_Float16)two.first), h1 = __builtin_bit_cast(unsigned short, (_Float16)two.second);
        kept = h0 | (h1 << 16);
        zero = (h0 & 0x7FFFu) == 0 || (h1 & 0x7FFFu) == 0;
      }
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(zero) != 0, 0)) low_precision_positions<IS_I8>(kept, two.p0, two.p1);
      const bool in_row = g < groups;
      kept = in_row ? kept : 0u;
      const unsigned ix = lane_positions<GU>(in_row ? two.p0 | (two.p1 << 2) : 0u, lane);
      if (g < padded) {
        if constexpr (IS_I8)
          *(uint16_t*)(column + value_at) = (uint16_t)kept;
        else
          *(uint32_t*)(column + value_at) = kept;
        if (in_lane == 0) {
          if constexpr (IS_I8)
            *(uint32_t*)(column + index_at) = ix;
          else
            *(uint16_t*)(column + index_at) = (uint16_t)ix;
        }
      }
      value_at += STRIDE / GS * tile_bytes(IS_I8);
      index_at += STRIDE / GS * tile_bytes(IS_I8);
    }
    base += B * STRIDE;
    if (ONE_BATCH) break;
    if (base < padded) load(base);
  }
}

template <bool IS_I8, int WPR>
static void launch_prepare_packed(const float* W, float* w_scale, uint8_t* packed, int64_t N, int64_t K, int ksteps, unsigned tiles, hipStream_t s) {
#define GPUSQ_PREPARE_PACKED(B) \
  prepare_packed_kernel<IS_I8, WPR, B><<<tiles * (kTileRows * WPR / 4), 256, 0, s>>>(W, w_scale, packed, N, (int)K, ksteps)
  const int64_t per_lane = ceil_div((int64_t)ksteps * (step_elems(IS_I8) / 4), 64 * WPR);  // groups, the padding's too
  if (per_lane <= 1) GPUSQ_PREPARE_PACKED(1);
  else if (per_lane == 2) GPUSQ_PREPARE_PACKED(2);
  else if (per_lane == 3) GPUSQ_PREPARE_PACKED(3);
  else if (per_lane == 4) GPUSQ_PREPARE_PACKED(4);
  else if (per_lane == 5) GPUSQ_PREPARE_PACKED(5);
  else if (per_lane == 6) GPUSQ_PREPARE_PACKED(6);
  else GPUSQ_PREPARE_PACKED(8);
#undef GPUSQ_PREPARE_PACKED
}

gpusq_status launch_prepare_weights(const float* W, gpusq_dtype dt, float* Wp, void* Wlow, float* w_scale, void* values,
                                    uint8_t* meta, void* packed, int64_t N, int64_t K, hipStream_t s) {
  const bool is_i8 = dt == GPUSQ_I8;
  const int ksteps = (int)ceil_div(K, step_elems(is_i8));
  const unsigned tiles = (unsigned)ceil_div(N, kTileRows);  // the padding rows of the last tile have their workgroups as well
  if (!Wp && !Wlow && !values && !meta) {
    if (is_i8 && K > 2048) launch_prepare_packed<true, 4>(W, w_scale, (uint8_t*)packed, N, K, ksteps, tiles, s);
    else if (is_i8) launch_prepare_packed<true, 1>(W, w_scale, (uint8_t*)packed, N, K, ksteps, tiles, s);
    else if (K > 2048) launch_prepare_packed<false, 4>(W, w_scale, (uint8_t*)packed, N, K, ksteps, tiles, s);
    else launch_prepare_packed<false, 1>(W, w_scale, (uint8_t*)packed, N, K, ksteps, tiles, s);
    return check_launch();
  }
#define GPUSQ_PREPARE(I8, WPR, ROWS)                                                                                                  \
  prepare_weights_kernel<I8, WPR><<<tiles * (kTileRows / ROWS), 64 * WPR * ROWS, 0, s>>>(W, Wp, (uint8_t*)Wlow, w_scale, (uint8_t*)values, \
                                                                                          meta, (uint8_t*)packed, N, K, ksteps)
  if (is_i8 && K > 2048) GPUSQ_PREPARE(true, 4, 1);
  else if (is_i8) GPUSQ_PREPARE(true, 1, 4);
  else if (K > 2048) GPUSQ_PREPARE(false, 4, 1);
  else GPUSQ_PREPARE(false, 1, 4);
#undef GPUSQ_PREPARE
  return check_launch();
}

}  // namespace gpusq
