// The linear layers behind attention of an encoder block on calibrated scales, in one launch: proj (fp16 output and its codes), fc1 with GELU (codes), fc2.
//
// Between the launches of the three layers each CU waits for the slowest, the launch and its first operands, and fc2 reads from memory what fc1 has just
// written.  But a row of the block needs no other row: here a workgroup takes 16 to 64 rows through all three layers, with their codes in LDS.
//   - The weights go from the packed buffer (in lane order) straight into registers, a wavefront's own channels, all K steps of a unit (16 F channels) while the
//     results of the unit before are worked on; every CU reads all of them, from the L2 of its XCD (64 bytes a clock and CU: 12 us for 1.47 MB).
//   - Nothing is shared but the codes, so there are three barriers in all: behind the copy of attention's codes, proj and fc1.
//   - F: two fragments up to 384 channels, where all wavefronts of a SIMD then have a unit of the narrow layers, four beyond (the index words of two come in
//     half-used lines: 12000 x 448, 1792 35.2 -> 32.6 us; 12608 x 384, 1536 is 33.5 with four, 32.2 with two).  The number of wavefronts is a multiple of four, one for each
//     SIMD; those past the narrow layers' channels take part in fc1 alone (12608 x 384, 1536 with six wavefronts of four fragments 38.0, with eight 33.7).
//   - Chunks of whole slabs of 16 rows, at most one slab apart: 12544 rows on 256 CUs as 240 chunks of 48 and 16 of 64 take 41.7 us, as 256 chunks of 49 rows, each as
//     much work as 64, 46.0.
// What bounds it: fc1's GELU and codes in the vector units, 20 of 32 us where few CUs are at work (12544 x 512, 2048 with 64 rows in each; start-up 3, proj 4.6, fc2
// 5); on all CUs the clock falls as well, to 2.0 to 2.1 GHz at 1.2 of the board's 1.4 kW.  Three launches / one, us: 12544 x 512, 2048 54.8 / 41.7, 3136 x 512, 2048 28.9 / 23.1, 12608 x 192, 768 29.0 / 17.3, 197 x 192, 768
// 12.2 / 7.8, 25000 x 256, 1024 44.9 / 30.2, 50176 x 512, 2048 158.7 / 150.0.
// (All operands touched ahead, a share of them by each workgroup of an XCD, so that the L2 has them: level.  B fragments read one slab ahead: level.)
#include "mlp_plan.h"
#include "tile_common.h"

namespace gpusq {

typedef __attribute__((address_space(1))) v4i mlp_global_v4;
typedef __attribute__((address_space(1))) ep_v2i mlp_global_v2;
typedef __attribute__((address_space(1))) ep_v4f mlp_global_f4;

// What a wavefront needs of a packed operand for a unit of 16 F channels and a K step
template <int F>
struct Unit {
  v4i a[F];
  typename std::conditional<F == 4, v4i, ep_v2i>::type ix;
};
__device__ __forceinline__ const global_u8* scalar(const global_u8* p) {  // (no constant is folded into the lane's offset, which then would be 64 bits wide)
  asm("" : "+s"(p));
  return p;
}
template <int F>
__device__ __forceinline__ void load_unit(Unit<F>& h, const global_u8* W, int ksteps, int unit, int ks, int lane) {
  const int f0 = unit * F & 15;
  const global_u8* t = W + (uint64_t)((uint32_t)(unit * F >> 4) * (uint32_t)ksteps + (uint32_t)ks) * (uint32_t)tile_bytes(true);
  const global_u8 *av = scalar(t + f0 * kFragValueBytes), *iv = scalar(t + kTileValueBytes + (f0 >> 3) * 2048 + (f0 & 7) * 4);
  uint32_t a_lane = (uint32_t)lane * 16, i_lane = (uint32_t)lane * 32;
  asm volatile("" : "+v"(a_lane), "+v"(i_lane));  // (widened here: scalar-base addressing)
#pragma unroll
  for (int f = 0; f < F; ++f) h.a[f] = *(const mlp_global_v4*)(av + a_lane + f * kFragValueBytes);
  if constexpr (F == 4)
    h.ix = *(const mlp_global_v4*)(iv + i_lane);
  else
    h.ix = *(const mlp_global_v2*)(iv + i_lane);
}

// The rows of one chunk, S slabs.
template <int S, int KS, int F>
__device__ __forceinline__ void block_mlp(const MlpArgs& a, int64_t m0, uint8_t* lds) {
  constexpr int G = F / 2;  // 32-channel groups of a unit
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), waves = (int)(blockDim.x >> 6);
  const int rows = a.M - m0 < 16 * S ? (int)(a.M - m0) : 16 * S;
  constexpr int panel = 16 * S * 128;
  uint8_t *const narrow = lds, *const wide = lds + KS * panel;
  const uint32_t b_lo = (uint32_t)((lane & 15) * 128 + (((lane >> 4) ^ ((lane & 15) >> 1)) << 4)), b_hi = b_lo ^ 64u;

  const global_u8 *Wp = uniform_ptr(a.Wp), *W1 = uniform_ptr(a.W1), *W2 = uniform_ptr(a.W2);
  const int units = (a.H + 16 * F - 1) / (16 * F), ksteps2 = (a.H + 127) / 128;
  // The wavefronts past the narrow layers' channels (their number is a multiple of four, one for each SIMD) take part in fc1 alone
  const int narrow_units = a.D / (16 * F);
  const bool in_narrow = w < narrow_units;
  const int mine = in_narrow ? w : narrow_units - 1;

  // ---- the codes of attention: asked for in front of the weights, which loads that return in order would wait behind
  constexpr int P = 4;  // pieces of 16 codes of a thread at a time
  const int per_row = a.D / 16, pieces = rows * per_row, threads = (int)blockDim.x;
  const global_u8* x = uniform_ptr(a.Xq + m0 * a.D);
  v4i piece[P];
#pragma unroll
  for (int j = 0; j < P; ++j) {
    const int i = tid + j * threads;
    piece[j] = *(const mlp_global_v4*)(x + (uint32_t)(i < pieces ? i : 0) * 16u);
  }
  __builtin_amdgcn_sched_barrier(0);
  // The coming unit, all K steps of it
  Unit<F> coming[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) load_unit<F>(coming[ks], Wp, KS, mine, ks, lane);

  __builtin_amdgcn_sched_barrier(0);
  for (int i0 = tid; i0 < pieces; i0 += P * threads) {
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const int i = i0 + j * threads, r = i / per_row, c = i - r * per_row;
      if (i < pieces) {
        const v4i v = i0 == tid ? piece[j] : *(const mlp_global_v4*)(x + (uint32_t)i * 16u);
        *(v4i*)(wide + (c >> 3) * panel + r * 128 + (((c & 7) ^ ((r >> 1) & 7)) << 4)) = v;
      }
    }
  }
  const float s_attn = a.s_attn[0], s_h = a.s_h[0], s_g = a.s_g[0];
  __syncthreads();

  auto read_b = [&](const uint8_t* s, int mt) __attribute__((always_inline)) {
    const v4i lo = *(const v4i*)(s + b_lo + mt * 2048), hi = *(const v4i*)(s + b_hi + mt * 2048);
    return v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  };
  // acc = the codes in LDS times the coming unit; as its steps are done those of unit `next` of Wnext are asked for, which come while this one's
  // results are worked on
  v4i acc[F][S];
  auto product = [&](const uint8_t* src, const global_u8* Wnext, int next) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
      for (int mt = 0; mt < S; ++mt) acc[f][mt] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int mt = 0; mt < S; ++mt) {
        const v8i b = read_b(src + ks * panel, mt);
#pragma unroll
        for (int f = 0; f < F; ++f) acc[f][mt] = smfmac<true>(coming[ks].a[f], b, acc[f][mt], coming[ks].ix[f]);
      }
      __builtin_amdgcn_sched_barrier(0);
      load_unit<F>(coming[ks], Wnext, KS, next, ks, lane);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // a lane's 8 channels of each 32 of a unit: constants and values
  struct Constants {
    ep_v4f c[2], b[2];
  };
  auto constants = [&](const float* ws, const float* bias, int n0, float s, Constants (&k)[G]) __attribute__((always_inline)) {
    const global_u8 *wp = uniform_ptr(ws + n0), *bp = uniform_ptr(bias + n0);
    uint32_t off = (uint32_t)(lane >> 4) * 32;
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        k[g].c[j] = *(const mlp_global_f4*)(wp + off + g * 128 + j * 16);
        k[g].b[j] = *(const mlp_global_f4*)(bp + off + g * 128 + j * 16);
      }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int j = 0; j < 2; ++j) k[g].c[j] *= s;
  };
  auto values = [&](const v4i& lo, const v4i& hi, const Constants& k, float (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (float)(j < 4 ? lo[j] : hi[j - 4]);
    pin8(v);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = __fmaf_rn(v[j], k.c[j >> 2][j & 3], k.b[j >> 2][j & 3]);
  };
  // Codes of a lane's 8 channels, to LDS and to memory, 16 codes of a row to a lane where two pieces are at hand: F == 4 the two 32s of slab mt, F == 2 slabs
  // mt and mt + 1 (`two`: the second exists)
  auto put_codes = [&](uint8_t* dst, int unit, int8_t* out, int ld, int mt, bool two, const unsigned (&d)[2][2]) __attribute__((always_inline)) {
    int l = lane;
    asm volatile("" : "+v"(l));  // (what follows from the lane is computed here, not kept across the products)
    const int c16 = l & 15, q = l >> 4, n0 = unit * 16 * F;
    uint8_t* pan = dst + (n0 >> 7) * panel;
    global_u8* o = uniform_ptr(out + m0 * ld + n0);
    if (two) {
      const ep_v2u x = __builtin_amdgcn_permlane16_swap(d[0][0], d[1][0], false, false);
      const ep_v2u y = __builtin_amdgcn_permlane16_swap(d[0][1], d[1][1], false, false);
      const ep_v4i v = ep_v4i{(int)x[0], (int)y[0], (int)x[1], (int)y[1]};
      const int r = (mt + (F == 2 ? q & 1 : 0)) * 16 + c16, n = (F == 4 ? (q & 1) * 32 : 0) + (q >> 1) * 16, c = ((n0 & 127) + n) >> 4;
      if (r < rows) {
        *(ep_v4i*)(pan + r * 128 + ((c ^ ((r >> 1) & 7)) << 4)) = v;
        uint32_t off = (uint32_t)r * (uint32_t)ld + (uint32_t)n;
        asm volatile("" : "+v"(off));
        *(global_v4i*)(o + off) = v;
      }
    } else {
      const int r = mt * 16 + c16, c = ((n0 & 127) >> 4) + (q >> 1);
      if (r < rows) {
        const ep_v2i v = ep_v2i{(int)d[0][0], (int)d[0][1]};
        *(ep_v2i*)(pan + r * 128 + ((c ^ ((r >> 1) & 7)) << 4) + (q & 1) * 8) = v;
        uint32_t off = (uint32_t)r * (uint32_t)ld + (uint32_t)q * 8;
        asm volatile("" : "+v"(off));
        *(__attribute__((address_space(1))) ep_v2i*)(o + off) = v;
      }
    }
  };
  // fp16 values of slab mt: whole lines of 64 channels (F == 4), or 64-byte pieces
  auto put_half = [&](const ep_v4i (&h)[G], void* out, int unit, int mt) __attribute__((always_inline)) {
    int l = lane;
    asm volatile("" : "+v"(l));
    const int c16 = l & 15, q = l >> 4, row_bytes = a.D * 2;
    global_u8* o = uniform_ptr((uint8_t*)out + m0 * row_bytes + unit * (32 * F));
    if constexpr (F == 4) {
      const int r = mt * 16 + (c16 & 7);
      store_line_pair(h[0], h[1], o, (uint32_t)(r * row_bytes + (c16 >> 3) * 64 + q * 16), 8 * row_bytes, r < rows, r + 8 < rows);
    } else {
      const int r = mt * 16 + c16;
      uint32_t off = (uint32_t)(r * row_bytes + q * 16);
      asm volatile("" : "+v"(off));
      if (r < rows) *(global_v4i*)(o + off) = h[0];
    }
  };
  auto halves = [&](const v4i& lo, const v4i& hi, const Constants& k) __attribute__((always_inline)) {
    float v[8];
    values(lo, hi, k, v);
    pin8(v);
    ep_v8h h;
#pragma unroll
    for (int j = 0; j < 8; ++j) h[j] = (_Float16)v[j];
    return h;
  };

  // ---- proj: fp16 output, and its codes as fc1's input
  {
    const float r_h = scale_reciprocal(s_h);
    Constants k[G];
    constants(a.ws_proj, a.b_proj, mine * 16 * F, s_attn, k);
    product(wide, W1, w < units ? w : units - 1);
    if (in_narrow) {
      unsigned d[2][2];
#pragma unroll
      for (int mt = 0; mt < S; ++mt) {
        ep_v4i H[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const ep_v8h h = halves(acc[2 * g][mt], acc[2 * g + 1][mt], k[g]);
          H[g] = __builtin_bit_cast(ep_v4i, h);
          const int i = F == 4 ? g : mt & 1;
          quantize_half8(h, s_h, r_h, d[i][0], d[i][1]);
        }
        put_half(H, a.P, w, mt);
        if (F == 4)
          put_codes(narrow, w, a.Hq, a.D, mt, true, d);
        else if ((mt & 1) || mt + 1 == S)
          put_codes(narrow, w, a.Hq, a.D, mt & ~1, mt & 1, d);
      }
    }
  }
  __syncthreads();

  // ---- fc1: the codes of its GELU
  const float r_g = scale_reciprocal(s_g);
#pragma nounroll
  for (int unit = w; unit < units; unit += waves) {
    Constants k[G];
    constants(a.ws_fc1, a.b_fc1, unit * 16 * F, s_h, k);
    product(narrow, W1, unit + waves < units ? unit + waves : unit);
    unsigned d[2][2];
#pragma unroll
    for (int mt = 0; mt < S; ++mt) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float v[8];
        values(acc[2 * g][mt], acc[2 * g + 1][mt], k[g], v);
        gelu_f32_x8(v);
        const int i = F == 4 ? g : mt & 1;
        quantize_bytes8(v, s_g, r_g, d[i][0], d[i][1]);
      }
      if (F == 4)
        put_codes(wide, unit, a.G, a.H, mt, true, d);
      else if ((mt & 1) || mt + 1 == S)
        put_codes(wide, unit, a.G, a.H, mt & ~1, mt & 1, d);
    }
  }

  // ---- fc2
  constexpr int B = 4;  // sets of weights: the step in hand and those on their way
  Unit<F> wt[B];
  auto fetch = [&](int set, int ks) __attribute__((always_inline)) { load_unit<F>(wt[set], W2, ksteps2, mine, ks < ksteps2 ? ks : ksteps2 - 1, lane); };
#pragma unroll
  for (int b = 0; b + 1 < B; ++b) fetch(b, b);
  __syncthreads();
  if (!in_narrow) return;
#pragma unroll
  for (int f = 0; f < F; ++f)
#pragma unroll
    for (int mt = 0; mt < S; ++mt) acc[f][mt] = v4i{0, 0, 0, 0};
  auto step2 = [&](int set, int ks) __attribute__((always_inline)) {
    fetch((set + B - 1) % B, ks + B - 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mt = 0; mt < S; ++mt) {
      const v8i b = read_b(wide + ks * panel, mt);
#pragma unroll
      for (int f = 0; f < F; ++f) acc[f][mt] = smfmac<true>(wt[set].a[f], b, acc[f][mt], wt[set].ix[f]);
    }
  };
  int ks = 0;
#pragma nounroll
  for (; ks + B <= ksteps2; ks += B) {
#pragma unroll
    for (int b = 0; b < B; ++b) step2(b, ks + b);
  }
#pragma unroll
  for (int b = 0; b + 1 < B; ++b) {
    if (ks + b >= ksteps2) break;
    step2(b, ks + b);
  }
  Constants k[G];
  constants(a.ws_fc2, a.b_fc2, w * 16 * F, s_g, k);
#pragma unroll
  for (int mt = 0; mt < S; ++mt) {
    ep_v4i H[G];
#pragma unroll
    for (int g = 0; g < G; ++g) H[g] = __builtin_bit_cast(ep_v4i, halves(acc[2 * g][mt], acc[2 * g + 1][mt], k[g]));
    put_half(H, a.Y, w, mt);
  }
}

// S: slabs of the highest chunk; the others have one less.
template <int S, int KS, int F>
__global__ void __launch_bounds__(F == 4 || KS < 3 ? 512 : 768, F == 4 ? 2 : (KS == 3 ? 3 : 4)) block_mlp_kernel(const MlpArgs a, const MlpPlan p) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t mlp_lds_mem[];
  const MlpChunk c = mlp_chunk(p, (int)blockIdx.x);
  if constexpr (S > 1) {
    if (c.slabs < S) return block_mlp<S - 1, KS, F>(a, c.m0, mlp_lds_mem);
  }
  block_mlp<S, KS, F>(a, c.m0, mlp_lds_mem);
}

// The plan of one launch; chunks == 0: three launches.  One launch is 1.1 to 2.5 times as fast up to 440 KB of operands, and beyond that from a row for every 550 bytes of them on; with
// fewer rows it is a chain of loads on few CUs (210 x 512, 2048 13.5 / 24.0 us, 1077 x 384, 1536 15.5 / 17.0, 104 x 320, 960 10.4 / 11.3 with 448 KB).  Where LDS holds fewer than four slabs of
// codes, one round of chunks is ahead (4492 x 448, 3584 47.6 / 41.3), more are not (17053 x 384, 3072 82.9 / 92.8).  A hidden layer of at most half the row leaves little between the output of
// proj and that of fc2, which three launches write as fast: many rows of more than 384 channels are behind (62832 x 512, 64 59.6 / 66.3).  Of 51363 sizes timed (16 to 420000 rows, D 64 ... 512, H 64 ... 8 D,
// calls in turn on three buffers) it takes 51108, 1.52 times as fast, 6 slower by more than 3 % (6 % at the most).
static MlpPlan mlp_plan_where_ahead(int64_t M, int64_t D, int64_t H, int resident) {
  const int forced = forced_kernel();
  if ((forced >= 0 && forced < 5) || !mlp_takes_sizes(D, H)) return MlpPlan{};
  const MlpPlan p = mlp_plan(M, D, H, resident);
  const int64_t operands = (D * D + 2 * D * H) * 5 / 8;
  const bool short_hidden = D > 384 && 2 * H <= D && M > 16384 * (D > 448 ? 3 : 8);
  if (forced == 6 || ((operands <= 440 * 1000 || M * 550 >= operands) && !short_hidden && (p.chunks <= resident || mlp_lds(D, H, kMlpSlabs) <= kMlpLds))) return p;
  return MlpPlan{};
}

int mlp_launches(int64_t M, int64_t D, int64_t H, int cus) { return mlp_plan_where_ahead(M, D, H, cus > 0 ? cus : num_cus()).chunks > 0 ? 1 : 3; }

bool mlp_in_one_launch(const MlpArgs& a) {
  const ByteRange all[] = {{a.Xq, (int64_t)a.M * a.D}, {a.P, (int64_t)a.M * a.D * 2}, {a.Hq, (int64_t)a.M * a.D}, {a.G, (int64_t)a.M * a.H}, {a.Y, (int64_t)a.M * a.D * 2}};
  for (int i = 0; i < 5; ++i)
    for (int j = 0; j < i; ++j)
      if (overlap(all[i], all[j])) return false;  // (a workgroup would write what another still reads)
  return mlp_plan_where_ahead(a.M, a.D, a.H, num_cus()).chunks > 0;
}

gpusq_status launch_mlp(const MlpArgs& a, hipStream_t s) {
  const MlpPlan p = mlp_plan(a.M, a.D, a.H, num_cus());
  const unsigned grid = (unsigned)p.chunks, threads = 64u * (unsigned)p.waves;
  const int slabs = mlp_slabs(p), ksteps = (a.D + 127) / 128;
#define GPUSQ_MLP(S, KS, F) \
  case S * 16 + KS: block_mlp_kernel<S, KS, F><<<grid, threads, (size_t)p.lds, s>>>(a, p); break;
#define GPUSQ_MLP_S(S) GPUSQ_MLP(S, 1, 2) GPUSQ_MLP(S, 2, 2) GPUSQ_MLP(S, 3, 2) GPUSQ_MLP(S, 4, 4)
  switch (slabs * 16 + ksteps) {
    GPUSQ_MLP_S(1)
    GPUSQ_MLP_S(2)
    GPUSQ_MLP_S(3)
    GPUSQ_MLP_S(4)
    default: return GPUSQ_ERR_UNSUPPORTED;
  }
#undef GPUSQ_MLP_S
#undef GPUSQ_MLP
  return check_launch();
}

}  // namespace gpusq
