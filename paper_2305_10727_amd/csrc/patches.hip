// Patch embedding from the images to the tokens in one launch: the patches are cut, and on the int8 path quantised behind a range pass, in LDS.
//
// Flattened patches in memory are written and read again, 84 MB each way for 256 images of 224 x 224 in patches of 14 x 14, and a GEMM over column
// tiles reads them once for each.  Here a workgroup takes 16 to 64 whole patches, all their values in LDS (75 KB of 64 x 588), and multiplies them by all weights.
//   - A patch row (28 bytes) has no alignment but that of a pair of pixels: a thread moves the same pair of every row, 4 bytes at a time, the next 14 loads on
//     their way while these are put where the fragment reads look for them (one address a pair; divisions once a patch).
//   - The weights go from the packed buffer (in lane order) straight into registers, a wavefront's units of 64 channels one behind the other, two K steps
//     ahead (three, 0 to 2 % slower); B fragments one step ahead (82.6 us, read in the step itself 89.1).
//   - Two workgroups of four wavefronts to a CU: one cuts or stores while the other multiplies.  One of 128 patches and eight wavefronts reads the weights half as often,
//     but nothing runs beside its cutting: 93.8.
// What bounds it: the board's power limit (1.39 of 1.4 kW, 1.85 GHz); of 82 us for 65536 x 588 -> 1280 the matrix instructions alone are 38 (their pipes are 31 % busy), with their
// weights from the L2 (64 bytes a clock and CU) 50, the 168 MB of output 34 alone, the images 15.  Flattened patches and GEMM / here, us: 65536 x 588 -> 1280 113 / 82, 44000 x 588 -> 768
// 61 / 42.7, 16384 x 588 -> 768 25.4 / 18.1, 4096 x 588 -> 320 13.2 / 9.9, 36936 x 144 -> 320 21.1 / 14.2.  (Output through the L2 instead of past it: 101 us.)
// int8, quantiser's two launches, flattened patches and GEMM / range pass and here: 62400 x 588 -> 576 89.5 / 63.2, 16200 x 588 -> 192 28.4 / 18.0, 2048 x 588 -> 192 15.7 / 11.0, from
// fp32 images 57600 x 588 -> 1216 126.6 / 107.5.  What bounds that: the codes go to the images' and to LDS two at a time, 74 stores of each for a thread and 64 patches.
#include "patches_plan.h"
#include "tile_common.h"

namespace gpusq {

typedef __attribute__((address_space(1))) v4i patch_global_v4;
typedef __attribute__((address_space(1))) ep_v2i patch_global_v2;
typedef __attribute__((address_space(1))) ep_v4f patch_global_f4;
typedef __attribute__((address_space(1))) uint16_t patch_global_codes;
typedef float patch_v2f __attribute__((ext_vector_type(2)));

// IN: GPUSQ_I32 for the fp16 product; GPUSQ_F16 or GPUSQ_F32 for the int8 one, which quantises images of that type.
constexpr int kPatchesF16 = GPUSQ_I32;
template <int S, int IN>
__global__ void __launch_bounds__(kPatchThreads, 2) patch_kernel(const GemmArgs a, const PatchPlan p) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  constexpr int T = kPatchThreads, WAVES = T / 64, R = 3;  // R: K steps of weights in registers, the one in hand and those on their way
  constexpr int panel = 16 * S * kPatchPanelBytes;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t m0 = (int64_t)blockIdx.x * (16 * S);
  const int rows = a.M - m0 < 16 * S ? (int)(a.M - m0) : 16 * S;
  const int units = p.units, ksteps = p.ksteps;
  constexpr bool I8 = IN != kPatchesF16, FP32 = IN == GPUSQ_F32;
  constexpr int ES = I8 ? 1 : 2, XS = FP32 ? 4 : 2;  // bytes of a value in LDS, of a pixel

  // ---- weights: a wavefront's units, one behind the other
  struct Step {
    v4i f[4];
    typename std::conditional<I8, v4i, ep_v2i>::type ix;
  } ring[R];
  const global_u8* W = uniform_ptr(a.W);
  auto first_tile = [&](int unit) __attribute__((always_inline)) { return W + (uint64_t)((uint32_t)(unit >> 2) * (uint32_t)ksteps) * (uint32_t)tile_bytes(I8); };
  int next_unit = w < units ? w : units - 1, next_ks = 0;
  const global_u8* next_tile = first_tile(next_unit);
  auto fetch = [&](Step& h) __attribute__((always_inline)) {
    const int f0 = (next_unit & 3) * 4;
    const global_u8 *av = next_tile + f0 * kFragValueBytes, *iv = next_tile + index_offset(I8, f0, 0);
    asm("" : "+s"(av));
    asm("" : "+s"(iv));
    uint32_t off = (uint32_t)lane * 16, ix_off = (uint32_t)lane * (I8 ? 32 : 16);
    asm volatile("" : "+v"(off), "+v"(ix_off));  // (widened here: scalar-base addressing)
#pragma unroll
    for (int f = 0; f < 4; ++f) h.f[f] = *(const patch_global_v4*)(av + off + f * kFragValueBytes);
    if constexpr (I8)
      h.ix = *(const patch_global_v4*)(iv + ix_off);
    else
      h.ix = *(const patch_global_v2*)(iv + ix_off);
    next_tile += tile_bytes(I8);
    if (++next_ks == ksteps) {  // (behind the last unit: that one again)
      next_ks = 0;
      next_unit = next_unit + WAVES < units ? next_unit + WAVES : next_unit;
      next_tile = first_tile(next_unit);
    }
  };
#pragma unroll
  for (int j = 0; j + 1 < R; ++j) fetch(ring[j]);
  __builtin_amdgcn_sched_barrier(0);

  // ---- the scale of all images, from the partial maxima of the range pass
  float s_a = 1.0f, r_a = 1.0f;
  Fp16Quantiser qz{};
  auto find_scale = [&]() __attribute__((always_inline)) {
    float* part = (float*)lds;
    unsigned* votes = (unsigned*)lds + WAVES;
    float v[4];  // (none is below 0; a range pass leaves at most 1024)
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = a.partial[tid + j * T < a.npartial ? tid + j * T : 0];
    const float mine = wave_max_magnitude(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])));
    if (lane == 0) part[w] = mine;
    __syncthreads();
    const float amax = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
    s_a = amax == 0.0f ? 1.0f : __fdiv_rn(amax, 127.0f);
    if (blockIdx.x == 0 && tid == 0) a.scale_out[0] = s_a;
    if constexpr (FP32) {
      r_a = scale_reciprocal(s_a);
    } else {
      const unsigned wave_votes = qz.prepare(s_a, tid);
      if (lane == 0) votes[w] = wave_votes;
      __syncthreads();
      qz.decide((unsigned)__builtin_amdgcn_readfirstlane((int)(votes[0] | votes[1] | votes[2] | votes[3])));
    }
    __syncthreads();  // (the patches go where these stand)
  };

  // ---- the patches: a thread takes the same pair of pixels of every row of IT patches; U rows at a time, the next ones on their way.  A row past
  // the last of a patch, and a patch past the last, is the last again: written once more to where it stands already.
  {
    constexpr int IT = S > 2 ? 2 : 1, U = 14 / IT;
    typedef typename std::conditional<FP32, patch_v2f, uint32_t>::type pair_t;
    typedef __attribute__((address_space(1))) pair_t global_pair;
    const int P = a.patch_P, pairs = P / 2, items = 16 * S * pairs, batches = a.patch_C * ((P + U - 1) / U);
    const global_u8* img = uniform_ptr(a.X);
    global_u8* codes = uniform_ptr(a.xq_out);
    const uint32_t image_row = (uint32_t)a.patch_W, plane = (uint32_t)a.patch_H * image_row;  // pixels
    const uint32_t px_n = (uint32_t)(a.patch_W / P), py_n = (uint32_t)(a.patch_H / P);
    for (int i0 = 0; i0 < items; i0 += IT * T) {
      uint32_t off[IT], kx[IT], swizzle[IT];
      int row[IT];
#pragma unroll
      for (int n = 0; n < IT; ++n) {
        const int i = i0 + n * T + tid < items ? i0 + n * T + tid : items - 1, r = i / pairs, x = i - r * pairs;
        const uint32_t m = (uint32_t)m0 + (uint32_t)(r < rows ? r : rows - 1);
        const uint32_t prow = m / px_n, px = m - prow * px_n, b = prow / py_n, py = prow - b * py_n;
        off[n] = b * (uint32_t)a.patch_C * plane + py * (uint32_t)P * image_row + px * (uint32_t)P + 2u * (uint32_t)x;
        kx[n] = (uint32_t)(2 * ES) * (uint32_t)x;
        swizzle[n] = patch_swizzle(r);
        row[n] = r;
      }
      struct Where {
        int c, y0;
      };
      auto forward = [&](Where& h) __attribute__((always_inline)) {
        h.y0 += U;
        if (h.y0 >= P) h.y0 = 0, ++h.c;
      };
      auto row_of = [&](const Where& h, int j) __attribute__((always_inline)) { return h.y0 + j < P ? h.y0 + j : P - 1; };
      auto row_at = [&](const Where& h, int j) __attribute__((always_inline)) { return (uint64_t)(uint32_t)h.c * plane + (uint64_t)(uint32_t)row_of(h, j) * image_row; };
      auto load = [&](const Where& h, pair_t (&v)[IT][U]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const global_u8* g = img + row_at(h, j) * XS;
          asm("" : "+s"(g));
#pragma unroll
          for (int n = 0; n < IT; ++n) {
            uint32_t o = off[n] * XS;
            asm volatile("" : "+v"(o));
            v[n][j] = *(const global_pair*)(g + o);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      auto lds_of = [&](const Where& h, int j, int n) __attribute__((always_inline)) {
        return lds + patch_lds_at((uint32_t)((h.c * P + row_of(h, j)) * P * ES) + kx[n], row[n], swizzle[n], S);
      };
      auto put = [&](const Where& h, const pair_t (&v)[IT][U]) __attribute__((always_inline)) {
        if constexpr (!I8) {
#pragma unroll
          for (int j = 0; j < U; ++j)
#pragma unroll
            for (int n = 0; n < IT; ++n) *(uint32_t*)lds_of(h, j, n) = v[n][j];
        } else {
#pragma unroll
          for (int j0 = 0; j0 < U; j0 += 4)
#pragma unroll
            for (int n = 0; n < IT; ++n) {
              unsigned c[2];
              if constexpr (FP32) {
                float x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = v[n][j0 + e / 2 < U ? j0 + e / 2 : U - 1][e & 1];
                quantize_bytes8(x, s_a, r_a, c[0], c[1]);
              } else {
                Fp16Quantiser::i4 raw;
#pragma unroll
                for (int e = 0; e < 4; ++e) raw[e] = (int)v[n][j0 + e < U ? j0 + e : U - 1];
                if (__builtin_expect(qz.refine, 0)) {
                  const Fp16Quantiser::i4 raws[1] = {raw};
                  qz.codes<true>(raw, qz.odd(raws), c[0], c[1]);
                } else {
                  const Fp16Quantiser plain{qz.s, qz.r, false};
                  plain.codes<false>(raw, false, c[0], c[1]);
                }
              }
#pragma unroll
              for (int e = 0; e < 4 && j0 + e < U; ++e) {
                const uint16_t code = (uint16_t)(c[e >> 1] >> (e & 1) * 16);
                *(uint16_t*)lds_of(h, j0 + e, n) = code;
                global_u8* q = codes + row_at(h, j0 + e);
                asm("" : "+s"(q));
                uint32_t o = off[n];
                asm volatile("" : "+v"(o));
                *(patch_global_codes*)(q + o) = code;
              }
            }
        }
      };
      pair_t v0[IT][U], v1[IT][U];
      Where asked{0, 0}, here{0, 0};
      load(asked, v0);
      if (I8 && i0 == 0) find_scale();
      int left = batches - 1;
#pragma nounroll
      for (; left >= 2; left -= 2) {
        forward(asked);
        load(asked, v1);
        put(here, v0);
        forward(here);
        forward(asked);
        load(asked, v0);
        put(here, v1);
        forward(here);
      }
      if (left == 1) {
        forward(asked);
        load(asked, v1);
        put(here, v0);
        forward(here);
        put(here, v1);
      } else {
        put(here, v0);
      }
    }
    const int first = a.patch_C * P * P * ES / 4, pad = ksteps * 32 - first;  // by 4 bytes; zeros behind the last value
    for (int i = tid; i < pad * 16 * S; i += T) {
      const int r = i % (16 * S);
      *(uint32_t*)(lds + patch_lds_at((uint32_t)(first + i / (16 * S)) * 4, r, patch_swizzle(r), S)) = 0;
    }
  }
  __syncthreads();
  if (w >= units) return;

  // ---- the product
  const uint32_t b_lo = (uint32_t)((lane & 15) * 128 + (((lane >> 4) ^ ((lane & 15) >> 1)) << 4)), b_hi = b_lo ^ 64u;
  auto read_b = [&](const uint8_t* s, int mt) __attribute__((always_inline)) {
    const v4i lo = *(const v4i*)(s + b_lo + mt * 2048), hi = *(const v4i*)(s + b_hi + mt * 2048);
    return v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  };
  typedef typename AccT<I8>::type acc_t;
  acc_t acc[4][S];
  ep_v4f factor[2][2], bias[2][2];  // of a lane's 8 channels of each 32 of a unit
  auto start = [&](int unit) __attribute__((always_inline)) {
    uint32_t off = (uint32_t)(lane >> 4) * 32;
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        factor[g][j] = bias[g][j] = ep_v4f{0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (I8) factor[g][j] = *(const patch_global_f4*)(uniform_ptr(a.w_scale + unit * kRowBlock) + off + g * 128 + j * 16);
        if (a.epilogue & GPUSQ_EPI_BIAS) bias[g][j] = *(const patch_global_f4*)(uniform_ptr(a.bias + unit * kRowBlock) + off + g * 128 + j * 16);
      }
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
      for (int mt = 0; mt < S; ++mt) acc[f][mt] = acc_t{0, 0, 0, 0};
  };
  auto store = [&](int unit) __attribute__((always_inline)) {
    int l = lane;
    asm volatile("" : "+v"(l));  // (what follows from the lane is computed here, not kept across the product)
    const int c16 = l & 15, q = l >> 4, row_bytes = a.N * 2;
    global_u8* y = uniform_ptr((uint8_t*)a.Y + m0 * row_bytes + unit * (2 * kRowBlock));
#pragma unroll
    for (int mt = 0; mt < S; ++mt) {
      ep_v4i h[2];
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const auto x = acc[2 * g + (j >> 2)][mt][j & 3];
          v[j] = I8 ? epilogue_value<true>((int)x, 0.0f, s_a * factor[g][j >> 2][j & 3], bias[g][j >> 2][j & 3]) : epilogue_value<false>(0, (float)x, 1.0f, bias[g][j >> 2][j & 3]);
        }
        pin8(v);
        ep_v8h x;
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = (_Float16)v[j];
        h[g] = __builtin_bit_cast(ep_v4i, x);
      }
      const int r = mt * 16 + (c16 & 7);
      store_line_pair(h[0], h[1], y, (uint32_t)(r * row_bytes + (c16 >> 3) * 64 + q * 16), 8 * row_bytes, r < rows, r + 8 < rows);
    }
  };
  v8i b[S];
#pragma unroll
  for (int mt = 0; mt < S; ++mt) b[mt] = read_b(lds, mt);
  int unit = w, ks = 0;
  start(unit);
  for (;;) {
#pragma unroll
    for (int slot = 0; slot < R; ++slot) {
      fetch(ring[(slot + R - 1) % R]);
      __builtin_amdgcn_sched_barrier(0);
      const Step& h = ring[slot];
      const uint8_t* coming = lds + (ks + 1 == ksteps ? 0 : ks + 1) * panel;
#pragma unroll
      for (int mt = 0; mt < S; ++mt) {
        if constexpr (I8) {
#pragma unroll
          for (int f = 0; f < 4; ++f) acc[f][mt] = smfmac<true>(h.f[f], b[mt], acc[f][mt], h.ix[f]);
        } else {
          acc[0][mt] = smfmac<false, 0>(h.f[0], b[mt], acc[0][mt], h.ix[0]);
          acc[1][mt] = smfmac<false, 1>(h.f[1], b[mt], acc[1][mt], h.ix[0]);
          acc[2][mt] = smfmac<false, 0>(h.f[2], b[mt], acc[2][mt], h.ix[1]);
          acc[3][mt] = smfmac<false, 1>(h.f[3], b[mt], acc[3][mt], h.ix[1]);
        }
        b[mt] = read_b(coming, mt);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (++ks == ksteps) {
        store(unit);
        unit += WAVES;
        if (unit >= units) return;
        start(unit);
        ks = 0;
      }
    }
  }
}

template <int IN>
static gpusq_status launch_patches(GemmArgs a, const PatchPlan& p, const void* img, int64_t C, int64_t H, int64_t W, int64_t P, hipStream_t s) {
  a.X = img;
  a.patch_P = (int)P;
  a.patch_C = (int)C;
  a.patch_H = (int)H;
  a.patch_W = (int)W;
  const size_t lds = (size_t)patch_lds(p.ksteps, p.slabs);
  const unsigned grid = (unsigned)p.chunks;
  switch (p.slabs) {
    case 1: patch_kernel<1, IN><<<grid, kPatchThreads, lds, s>>>(a, p); break;
    case 2: patch_kernel<2, IN><<<grid, kPatchThreads, lds, s>>>(a, p); break;
    case 3: patch_kernel<3, IN><<<grid, kPatchThreads, lds, s>>>(a, p); break;
    case 4: patch_kernel<4, IN><<<grid, kPatchThreads, lds, s>>>(a, p); break;
    default: return GPUSQ_ERR_UNSUPPORTED;
  }
  return check_launch();
}

// The plan of one launch; chunks == 0: flattened patches in memory and the GEMM.  Every workgroup reads all weights, so it takes patches enough for them and LDS for
// at least two slabs (8192 x 588 -> 192 14.1 / 8.9 us, 2048 x 588 -> 768 12.6 / 11.8, 16384 x 588 -> 1280 33.2 / 25.7; slower 1105 x 588 -> 1280 12.7 / 15.1, 8192 x 588 -> 3072 35.7 / 38.4,
// with one slab 42390 x 1600 -> 448 124 / 137).  What it costs is not the patches' values but their rows: a patch is cut in batches of 7 or 14 rows of one channel of the image, full
// or not, so many channels of few rows are slow, 2420 x 1280 -> 64 of 320 channels of 2 x 2 12.0 / 212.9, 9000 x 512 of 32 channels of 4 x 4 three times as slow; up to four channels are taken.
// Of 10538 sizes timed (600 to 80000 patches of 2 x 2 to 28 x 28, 1 to 320 channels, 64 to 3072 channels out, calls in turn on three buffers) it takes 6551, 1.48 times as fast in one
// launch, 10 of them slower by 3 to 8 %; of 46400 others that it takes, up to 400000 patches, 1.76 times, 147 slower by more than 3 % (17 % at the most).  16 x 16 patches, whose 16-byte pieces need no cutting, have gpusq_patch_embed16_fp16 (25088 x 768 -> 768 28.3, here 43.1) or, few of them, the
// two launches (832 x 768 -> 256 7.8, here 8.1).
static bool patch_f16_ahead(int64_t M, int64_t C, int64_t P, int64_t ksteps, int64_t D, const PatchPlan& p, int resident) {
  const int fit = patch_slabs(ksteps);
  if (P == 16 || C > 4 || fit < 2) return false;
  // workgroups just past what `n` of them fill: the CUs wait for the few that are left (two slabs, 16720 x 972 -> 384 29.1 / 34.6)
  auto just_past = [&](int64_t n) { return p.chunks > n && 4 * (int64_t)p.chunks <= 5 * n; };
  if (fit == 2) return M >= 2048 && D <= 512 && !just_past(resident / 2) && !just_past(resident) && !just_past(2 * (int64_t)resident);
  if (D <= 512) return M >= (C == 4 && D > 256 ? 800 : 640);  // (660 x 256 -> 384 of four channels 5.7 / 6.5)
  // three slabs at the most: all of them (5244 x 648 -> 1152 with two 17.4 / 21.1, 1008 x 800 -> 576 with one 9.7 / 11.2)
  if (fit == 3) return p.slabs == 3 && D <= 1408 && !just_past(2 * (int64_t)resident);
  if (D <= 1408) return M >= 12 * (D - 512) + 512;  // (760 x 576 -> 576 7.0 / 8.2, 1280 x 256 -> 640 7.1 / 7.6)
  // more channels out: a K of 8 steps, else the output decides (34632 x 64 -> 2752 41.2 / 54.0)
  return ksteps >= 8 && M >= 10 * (D - 512) && !just_past(2 * (int64_t)resident);
}
// int8: two launches instead of four, so for fewer patches too (98 x 588 -> 256 15.6 / 10.6, 896 x 588 -> 1088 20.9 / 16.2; 672 x 588 -> 1024 14.2 / 14.9); from fp32 images, which cost more
// registers and loads, four times as many (1000 x 192 -> 960 12.0 / 13.2).  Codes move two at a time, so up to three channels (3 us of 12 behind with a fourth and few patches), and where
// a workgroup has more than two slabs, rows of 2, 4 or 8 pixels, which leave half of a batch of 7 empty, only with one or two batches (50160 x 192 -> 256 fp32 29.9 / 36.6, 75776 x 48 -> 192
// fp32 23.7 / 27.6); 14 rows leave nothing empty, the others are behind just past a round of workgroups (33120 x 300 -> 1088 40.5 / 45.3).  Patches of more than 14 rows are 28 rows of work
// (4464 x 972 -> 896 24.0 / 30.4).  Of 21715 sizes timed (16 to 80000 patches of 2 x 2 to 14 x 14, 1 to 320 channels, 64 to 3072 channels out, fp16 and fp32) it takes 13337, 1.42 times as fast,
// 8 of them slower by more than 3 %; of 51691 others that it takes, up to 400000 patches, 1.41 times, 194 slower (17 % at the most).
static bool patch_i8_ahead(int64_t M, int64_t C, int64_t P, int64_t ksteps, int64_t D, bool fp32, const PatchPlan& p, int resident) {
  if (P > 14 || C > 3 || patch_slabs(ksteps) < 3 || D > 1408 || M < (fp32 ? 8 : 2) * (D - 512)) return false;
  if (p.slabs <= 2 || P == 14) return true;
  if ((P <= 4 || P == 8) && (fp32 || C * ceil_div(P, 7) > 2)) return false;
  return p.chunks <= 2 * (int64_t)resident || 4 * (int64_t)p.chunks > 5 * 2 * (int64_t)resident;
}
static PatchPlan patch_plan_where_ahead(bool is_i8, int x_bytes, int64_t B, int64_t C, int64_t H, int64_t W, int64_t P, int64_t ksteps, int64_t D, int epilogue, int resident) {
  const int forced = forced_kernel();
  if ((forced >= 0 && forced < 5) || (epilogue & GPUSQ_EPI_GELU) || !patch_takes_sizes(x_bytes, B, C, H, W, P, ksteps, D)) return PatchPlan{};
  const int64_t M = B * (H / P) * (W / P);
  if (M > INT32_MAX) return PatchPlan{};
  const PatchPlan p = patch_plan(M, ksteps, D, resident);
  if (forced == 6 || (is_i8 ? patch_i8_ahead(M, C, P, ksteps, D, x_bytes == 4, p, resident) : patch_f16_ahead(M, C, P, ksteps, D, p, resident))) return p;
  return PatchPlan{};
}

int patch_embed_f16_launches(int64_t B, int64_t C, int64_t H, int64_t W, int64_t P, int64_t K_pad, int64_t D, int epilogue, int cus) {
  return patch_plan_where_ahead(false, 2, B, C, H, W, P, ceil_div(K_pad, 64), D, epilogue, cus > 0 ? cus : num_cus()).chunks > 0 ? 1 : 2;
}

gpusq_status launch_patch_embed_f16(GemmArgs a, const void* img, int64_t B, int64_t C, int64_t H, int64_t W, int64_t P, hipStream_t s) {
  const PatchPlan p = patch_plan_where_ahead(false, 2, B, C, H, W, P, ceil_div(a.K, 64), a.N, a.epilogue, num_cus());
  // (a workgroup would write what another still reads)
  if (p.chunks == 0 || overlap(ByteRange{img, B * C * H * W * 2}, ByteRange{a.Y, (int64_t)a.M * a.N * 2})) {
    const gpusq_status st = launch_im2col_patches(img, const_cast<void*>(a.X), GPUSQ_F16, B, C, H, W, P, a.K, s);
    return st != GPUSQ_OK ? st : launch_spgemm(false, a, s);
  }
  return launch_patches<kPatchesF16>(a, p, img, C, H, W, P, s);
}

int patch_embed_i8_launches(gpusq_dtype dt, int64_t B, int64_t C, int64_t H, int64_t W, int64_t P, int64_t K_pad, int64_t D, int epilogue, int cus) {
  const int resident = cus > 0 ? cus : num_cus();
  if (P == 16 && K_pad == C * 256 && few_patches_take_whole_rows(B * (H / P) * (W / P), D, K_pad, epilogue, dt, resident)) return 2;
  return patch_plan_where_ahead(true, dt == GPUSQ_F32 ? 4 : 2, B, C, H, W, P, ceil_div(K_pad, 128), D, epilogue, resident).chunks > 0 ? 2 : 4;
}

gpusq_status launch_patch_embed_i8(GemmArgs a, const void* img, gpusq_dtype dt, int8_t* img_q, float* scale, void* workspace, int64_t B, int64_t C, int64_t H,
                                   int64_t W, int64_t P, hipStream_t s) {
  const int64_t pixels = B * C * H * W;
  const int x_bytes = dt == GPUSQ_F32 ? 4 : 2;
  const int resident = num_cus();
  const bool whole_rows = P == 16 && a.K == C * 256 && few_patches_take_whole_rows(a.M, a.N, a.K, a.epilogue, dt, resident);
  const PatchPlan p = patch_plan_where_ahead(true, x_bytes, B, C, H, W, P, ceil_div(a.K, 128), a.N, a.epilogue, resident);
  const ByteRange in{img, pixels * x_bytes}, codes{img_q, pixels}, y{a.Y, (int64_t)a.M * a.N * 2};
  const ByteRange range{workspace, (int64_t)gpusq_quantize_workspace_bytes(GPUSQ_PER_TENSOR, 1, pixels)};
  a.act_scale = scale;
  if ((!whole_rows && p.chunks == 0) || overlap(in, y) || overlap(in, codes) || overlap(codes, y) || overlap(range, y) || overlap(range, codes)) {
    gpusq_status st = launch_quantize(img, dt, img_q, scale, GPUSQ_PER_TENSOR, 0, 1, pixels, workspace, s);
    if (st != GPUSQ_OK) return st;
    st = launch_im2col_patches(img_q, const_cast<void*>(a.X), GPUSQ_I8, B, C, H, W, P, a.K, s);
    return st != GPUSQ_OK ? st : launch_spgemm(true, a, s);
  }
  if (whole_rows) {
    a.X = img;
    a.patch_P = (int)P;
    a.patch_C = (int)C;
    a.patch_H = (int)H;
    a.patch_W = (int)W;
    return launch_few_patches(a, dt, img_q, scale, workspace, s);
  }
  a.xq_out = img_q;
  a.scale_out = scale;
  a.npartial = launch_amax(img, dt, pixels, workspace, s);
  a.partial = (const float*)workspace;
  return dt == GPUSQ_F32 ? launch_patches<GPUSQ_F32>(a, p, img, C, H, W, P, s) : launch_patches<GPUSQ_F16>(a, p, img, C, H, W, P, s);
}

}  // namespace gpusq
