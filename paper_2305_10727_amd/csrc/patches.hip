// Patch embedding of fp16 images, from the images to the tokens in one launch: the patches are cut in LDS.
//
// Flattened patches in memory are written and read again, 84 MB each way for 256 images of 224 x 224 in patches of 14 x 14, and a GEMM over column
// tiles reads them once for each.  Here a workgroup takes 16 to 64 whole patches, all their values in LDS (75 KB of 64 x 588), and multiplies them by all weights.
//   - A patch row (28 bytes) has no alignment but that of a pair of pixels: a thread moves the same pair of every row, 4 bytes at a time, the next 14 loads on
//     their way while these are put where the fragment reads look for them (one address a pair; divisions once a patch).
//   - The weights go from the packed buffer (in lane order) straight into registers, a wavefront's units of 64 channels one behind the other, two K steps
//     ahead (three, 0 to 2 % slower); B fragments one step ahead (82.6 us, read in the step itself 89.1).
//   - Two workgroups of four wavefronts to a CU: one cuts or stores while the other multiplies.  One of 128 patches and eight wavefronts reads the weights half as often,
//     but nothing runs beside its cutting: 93.8.
// What bounds it: the matrix instructions at the board's power limit, 38 us of 82 for 65536 x 588 -> 1280, with their weights from the L2 (64 bytes a clock and CU) 50, the
// 168 MB of output 34 alone, the images 15.  Flattened patches and GEMM / here, us: 65536 x 588 -> 1280 113 / 82, 44000 x 588 -> 768 61 / 42.7, 16384 x 588 -> 768 25.4 / 18.1, 4096 x 588
// -> 320 13.2 / 9.9, 36936 x 144 -> 320 21.1 / 14.2.  (Output through the L2 instead of past it: 101 us.)
#include "patches_plan.h"
#include "tile_common.h"

namespace gpusq {

typedef __attribute__((address_space(1))) v4i patch_global_v4;
typedef __attribute__((address_space(1))) ep_v2i patch_global_v2;
typedef __attribute__((address_space(1))) ep_v4f patch_global_f4;
typedef __attribute__((address_space(1))) uint32_t patch_global_pair;

template <int S>
__global__ void __launch_bounds__(kPatchThreads, 2) patch_kernel(const GemmArgs a, const PatchPlan p) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  constexpr int T = kPatchThreads, WAVES = T / 64, R = 3;  // R: K steps of weights in registers, the one in hand and those on their way
  constexpr int panel = 16 * S * kPatchPanelBytes;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t m0 = (int64_t)blockIdx.x * (16 * S);
  const int rows = a.M - m0 < 16 * S ? (int)(a.M - m0) : 16 * S;
  const int units = p.units, ksteps = p.ksteps;

  // ---- weights: a wavefront's units, one behind the other
  struct Step {
    v4i f[4];
    ep_v2i ix;
  } ring[R];
  const global_u8* W = uniform_ptr(a.W);
  auto first_tile = [&](int unit) __attribute__((always_inline)) { return W + (uint64_t)((uint32_t)(unit >> 2) * (uint32_t)ksteps) * (uint32_t)tile_bytes(false); };
  int next_unit = w < units ? w : units - 1, next_ks = 0;
  const global_u8* next_tile = first_tile(next_unit);
  auto fetch = [&](Step& h) __attribute__((always_inline)) {
    const int f0 = (next_unit & 3) * 4;
    const global_u8 *av = next_tile + f0 * kFragValueBytes, *iv = next_tile + index_offset(false, f0, 0);
    asm("" : "+s"(av));
    asm("" : "+s"(iv));
    uint32_t off = (uint32_t)lane * 16;
    asm volatile("" : "+v"(off));  // (widened here: scalar-base addressing)
#pragma unroll
    for (int f = 0; f < 4; ++f) h.f[f] = *(const patch_global_v4*)(av + off + f * kFragValueBytes);
    h.ix = *(const patch_global_v2*)(iv + off);
    next_tile += tile_bytes(false);
    if (++next_ks == ksteps) {  // (behind the last unit: that one again)
      next_ks = 0;
      next_unit = next_unit + WAVES < units ? next_unit + WAVES : next_unit;
      next_tile = first_tile(next_unit);
    }
  };
#pragma unroll
  for (int j = 0; j + 1 < R; ++j) fetch(ring[j]);
  __builtin_amdgcn_sched_barrier(0);

  // ---- the patches: a thread takes the same pair of pixels of every row of IT patches; U rows at a time, the next ones on their way.  A row past
  // the last of a patch, and a patch past the last, is the last again: written once more to where it stands already.
  {
    constexpr int IT = S > 2 ? 2 : 1, U = 14 / IT;
    const int P = a.patch_P, pairs = P / 2, items = 16 * S * pairs, batches = a.patch_C * ((P + U - 1) / U);
    const global_u8* img = uniform_ptr(a.X);
    const uint32_t image_row = (uint32_t)a.patch_W * 2, plane = (uint32_t)a.patch_H * image_row;
    const uint32_t px_n = (uint32_t)(a.patch_W / P), py_n = (uint32_t)(a.patch_H / P);
    for (int i0 = 0; i0 < items; i0 += IT * T) {
      uint32_t off[IT], kx[IT], swizzle[IT];
      int row[IT];
#pragma unroll
      for (int n = 0; n < IT; ++n) {
        const int i = i0 + n * T + tid < items ? i0 + n * T + tid : items - 1, r = i / pairs, x = i - r * pairs;
        const uint32_t m = (uint32_t)m0 + (uint32_t)(r < rows ? r : rows - 1);
        const uint32_t prow = m / px_n, px = m - prow * px_n, b = prow / py_n, py = prow - b * py_n;
        off[n] = b * (uint32_t)a.patch_C * plane + py * (uint32_t)P * image_row + px * (uint32_t)(2 * P) + 4u * (uint32_t)x;
        kx[n] = 4u * (uint32_t)x;
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
      auto load = [&](const Where& h, uint32_t (&v)[IT][U]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const global_u8* g = img + ((uint64_t)(uint32_t)h.c * plane + (uint64_t)(uint32_t)row_of(h, j) * image_row);
          asm("" : "+s"(g));
#pragma unroll
          for (int n = 0; n < IT; ++n) {
            uint32_t o = off[n];
            asm volatile("" : "+v"(o));
            v[n][j] = *(const patch_global_pair*)(g + o);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      auto put = [&](const Where& h, const uint32_t (&v)[IT][U]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < U; ++j)
#pragma unroll
          for (int n = 0; n < IT; ++n)
            *(uint32_t*)(lds + patch_lds_at((uint32_t)((h.c * P + row_of(h, j)) * P * 2) + kx[n], row[n], swizzle[n], S)) = v[n][j];
      };
      uint32_t v0[IT][U], v1[IT][U];
      Where asked{0, 0}, here{0, 0};
      load(asked, v0);
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
    const int first = a.patch_C * P * P / 2, pad = ksteps * 32 - first;  // pairs; zeros behind the last value
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
  v4f acc[4][S];
  ep_v4f bias[2][2];  // of a lane's 8 channels of each 32 of a unit
  auto start = [&](int unit) __attribute__((always_inline)) {
    uint32_t off = (uint32_t)(lane >> 4) * 32;
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        bias[g][j] = ep_v4f{0.0f, 0.0f, 0.0f, 0.0f};
        if (a.epilogue & GPUSQ_EPI_BIAS) bias[g][j] = *(const patch_global_f4*)(uniform_ptr(a.bias + unit * kRowBlock) + off + g * 128 + j * 16);
      }
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
      for (int mt = 0; mt < S; ++mt) acc[f][mt] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
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
        for (int j = 0; j < 8; ++j) v[j] = epilogue_value<false>(0, j < 4 ? acc[2 * g][mt][j] : acc[2 * g + 1][mt][j - 4], 1.0f, bias[g][j >> 2][j & 3]);
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
        acc[0][mt] = smfmac<false, 0>(h.f[0], b[mt], acc[0][mt], h.ix[0]);
        acc[1][mt] = smfmac<false, 1>(h.f[1], b[mt], acc[1][mt], h.ix[0]);
        acc[2][mt] = smfmac<false, 0>(h.f[2], b[mt], acc[2][mt], h.ix[1]);
        acc[3][mt] = smfmac<false, 1>(h.f[3], b[mt], acc[3][mt], h.ix[1]);
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

// The plan of one launch; chunks == 0: flattened patches in memory and the GEMM.  Every workgroup reads all weights, so it takes patches enough for them and LDS for
// at least two slabs.  Of 540 sizes timed (650 to 66000 patches of 2 x 2 to 28 x 28, 1 to 4 channels, 128 to 1408 channels out, calls in turn on three buffers) these are 1.5
// times as fast in one launch (8192 x 588 -> 192 14.1 / 8.9 us, 2048 x 588 -> 768 12.6 / 11.8, 16384 x 588 -> 1280 33.2 / 25.7), 2 of 226 slower by 3 %; of the others 1105 x 588
// -> 1280 12.7 / 15.1, 8192 x 588 -> 3072 35.7 / 38.4, with two slabs (972 to 1280 values) 2160 x 1200 -> 1152 24.0 / 24.7, with one 42390 x 1600 -> 448 124 / 137.  16 x 16 patches of more
// than 2^18 outputs have gpusq_patch_embed16_fp16, whose 16-byte pieces need no cutting (25088 x 768 -> 768 28.3, here 43.1).
static PatchPlan patch_plan_where_ahead(int64_t B, int64_t C, int64_t H, int64_t W, int64_t P, int64_t K_pad, int64_t D, int epilogue, int resident) {
  const int forced = forced_kernel();
  if ((forced >= 0 && forced < 5) || (epilogue & GPUSQ_EPI_GELU) || !patch_takes_sizes(B, C, H, W, P, K_pad, D)) return PatchPlan{};
  const int64_t M = B * (H / P) * (W / P);
  if (M > INT32_MAX) return PatchPlan{};
  if (forced != 6) {
    const int slabs = patch_slabs(ceil_div(K_pad, 64));
    if ((P == 16 && M * D > 256 * 1024) || slabs < 2 || (slabs == 2 ? M < 2048 || D > 512 : M < 640 || M < 6 * (D - 512))) return PatchPlan{};
  }
  return patch_plan(M, K_pad, D, resident);
}

int patch_embed_f16_launches(int64_t B, int64_t C, int64_t H, int64_t W, int64_t P, int64_t K_pad, int64_t D, int epilogue, int cus) {
  return patch_plan_where_ahead(B, C, H, W, P, K_pad, D, epilogue, cus > 0 ? cus : num_cus()).chunks > 0 ? 1 : 2;
}

gpusq_status launch_patch_embed_f16(GemmArgs a, const void* img, int64_t B, int64_t C, int64_t H, int64_t W, int64_t P, hipStream_t s) {
  PatchPlan p = patch_plan_where_ahead(B, C, H, W, P, a.K, a.N, a.epilogue, num_cus());
  // (a workgroup would write what another still reads)
  if (p.chunks == 0 || overlap(ByteRange{img, B * C * H * W * 2}, ByteRange{a.Y, (int64_t)a.M * a.N * 2})) {
    const gpusq_status st = launch_im2col_patches(img, const_cast<void*>(a.X), GPUSQ_F16, B, C, H, W, P, a.K, s);
    return st != GPUSQ_OK ? st : launch_spgemm(false, a, s);
  }
  a.X = img;
  a.patch_P = (int)P;
  a.patch_C = (int)C;
  a.patch_H = (int)H;
  a.patch_W = (int)W;
  const size_t lds = (size_t)patch_lds(p.ksteps, p.slabs);
  const unsigned grid = (unsigned)p.chunks;
  switch (p.slabs) {
    case 1: patch_kernel<1><<<grid, kPatchThreads, lds, s>>>(a, p); break;
    case 2: patch_kernel<2><<<grid, kPatchThreads, lds, s>>>(a, p); break;
    case 3: patch_kernel<3><<<grid, kPatchThreads, lds, s>>>(a, p); break;
    case 4: patch_kernel<4><<<grid, kPatchThreads, lds, s>>>(a, p); break;
    default: return GPUSQ_ERR_UNSUPPORTED;
  }
  return check_launch();
}

}  // namespace gpusq
