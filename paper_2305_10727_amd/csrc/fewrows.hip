// Sparse GEMM for few activation rows (one image, a classifier head: M up to a few hundred): the latency kernel.
//
// What bounds such a problem is a chain: launch, first operands from memory, K steps one behind the other, epilogue.  The
// tiles of 64 x 64 outputs of spgemm_small_kernel give it few workgroups (197 x 3072 -> 768: 48 on 256 CUs) that each walk
// all K steps in lockstep, a barrier and an LDS round trip per step (0.26 us per step).  Here
//   - a workgroup is 4 wavefronts on 64 channels x 16 or 32 rows, and the K steps are dealt out over the wavefronts: each
//     multiplies every fourth step of the same tile into accumulators of its own, which are added up in LDS at the end;
//   - a wavefront needs nothing of the others until then, so the K loop has no barrier: kept values and index words go from
//     memory straight into the registers of the wavefront that multiplies them (the packed buffer is in lane order), the
//     rows of X through a wavefront's own piece of LDS, which turns whole 128-byte lines (what the memory pipeline takes at
//     its full rate: 64 bytes per clock and CU, against 16 for the 16 rows x 64 bytes of the operand's own layout) into the
//     operand's layout.  LDS operations of a wavefront execute in order: no wait between its writes and its reads.
//   - a wavefront requests its steps in batches of three before it multiplies the first of them: up to 12 K steps that is
//     one batch per wavefront, and the run time is close to one trip to memory plus the launch.
// Measured against the 64 x 64 tiles (int8 / fp16, us, graph replays): 197 x 768 -> 768 4.8 -> 3.2 / 6.2 -> 3.4, 64 x 768 ->
// 2304 4.8 -> 3.3 / 6.2 -> 3.4, 197 x 3072 -> 768 9.8 -> 4.5 / 16.6 -> 6.0.  With 8 wavefronts instead of 4 the longest K
// gain 2 % and every problem of more than one round of workgroups loses 20-40 %; where the kernel quantises see fewrows_wide.
//
// INT8 with fp16 or fp32 activations: the rows are quantised on their way through the registers, with a given scale, with the partial
// maxima that a range pass left behind, or (small X) with the range of all of X, which every workgroup reads for itself: one
// launch for the whole layer.  The workgroups of the first column of tiles write the codes out if asked.
#include "tile_common.h"

namespace gpusq {

constexpr int kFrBatch = 3, kFrWaves = 4;
constexpr int kFrRow = kStepBytes + 16;  // LDS pitch of a row: 16 rows x 16-byte reads hit 16 distinct bank groups

// The per-tensor scale of fp16 activations from their largest magnitude.
__device__ __forceinline__ float scale_of_range(float amax) { return amax == 0.0f ? 1.0f : __fdiv_rn(amax, 127.0f); }

typedef __attribute__((address_space(1))) v4i global_v4;
typedef __attribute__((address_space(1))) ep_v2u global_v2u;
typedef __attribute__((address_space(1))) unsigned global_u32;

// XQ: 0 = X is the operand; 1 = fp16 or fp32 to be quantised with a given scale; 2 = with the scale of X's range (see GemmArgs)
// PATCH: the rows of X are 16 x 16 patches gathered from an image batch (see patch_chunk_offset).
// XW: bytes of X in memory per byte of the operand (quantised: 2 = fp16, 4 = fp32).
template <bool IS_I8, int TM, int XQ, bool PATCH = false, int NW = kFrWaves, int XW = XQ != 0 ? 2 : 1>
__global__ void __launch_bounds__(64 * NW, 2) spgemm_fewrows_kernel(const GemmArgs a, const int tiles_n, const int tiles_m, const int n_fast) {
  constexpr bool QUANT = XQ != 0, FP32 = XW == 4;
  static_assert(IS_I8 || !QUANT, "the fp16 path takes fp16 X as it is");
  static_assert(QUANT ? XW == 2 || XW == 4 : XW == 1, "an operand as it is, fp16 or fp32");
  typedef typename AccT<IS_I8>::type acc_t;
  constexpr int ES = IS_I8 ? 1 : 2;
  constexpr int ROWS = 16 * TM;
  constexpr int XL = 2 * TM * XW;    // 16-byte loads per lane for the X rows of a step
  constexpr int D = kFrBatch;

  // a wavefront's rows of the K step it multiplies; behind the K loop its accumulators
  constexpr int kPiece = ROWS * kFrRow > 4 * TM * 1024 ? ROWS * kFrRow : 4 * TM * 1024;
  __shared__ __attribute__((aligned(16))) uint8_t lds[NW][kPiece];
  __shared__ float part[NW];
  __shared__ unsigned votes[4];

  // tiles that share the larger operand run side by side on one XCD
  const int tiles_total = tiles_n * tiles_m, per_xcd = (tiles_total + 7) / 8;
  const int local = (int)(blockIdx.x >> 3), tile = (int)(blockIdx.x & 7) * per_xcd + local;
  if (local >= per_xcd || tile >= tiles_total) return;  // the whole workgroup leaves before any barrier
  const int n_blk = n_fast ? tile % tiles_n : tile / tiles_m, m_blk = n_fast ? tile / tiles_n : tile % tiles_m;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t k_bytes = (int64_t)a.K * ES;
  const int ksteps = (int)((k_bytes + kStepBytes - 1) / kStepBytes);
  const int mine = (ksteps - wave + NW - 1) / NW;  // K steps wave, wave + NW, ... (none if there are fewer steps than wavefronts)
  const int tail_bytes = (int)(k_bytes % kStepBytes);

  // X: a load instruction covers 8 (fp16 to be quantised: 4, fp32: 2) rows x 128 (256, 512) bytes, every line whole
  constexpr int LPR = 8 * XW;  // lanes per row
  const int64_t m0 = (int64_t)m_blk * ROWS;
  const int64_t last_row = (int64_t)a.M - 1 - m0;  // >= 0: a tile starts inside X; rows past the end re-read the last one
  const global_u8* Xtile = uniform_ptr((const uint8_t*)a.X + (PATCH ? 0 : m0 * k_bytes * XW));
  // Row (of the 8, 4 or 2) and 16-byte chunk of a step that this lane fetches: consecutive lanes along a row of X, or, for
  // patches, along a row of the image, where neighbouring patches' 16 bytes (fp16: 32) are contiguous.
  int lrow = lane / LPR, lchunk = lane % LPR;
  if constexpr (PATCH) {
    lrow = IS_I8 ? (lane & 7) : ((lane >> 1) & 7);
    lchunk = IS_I8 ? (lane >> 3) : ((lane >> 4) * 2 + (lane & 1));
  }
  uint32_t xoff[XL];
#pragma unroll
  for (int j = 0; j < XL; ++j) {
    const int r = (64 / LPR) * j + lrow;
    const int64_t rr = r < last_row ? r : last_row;
    if constexpr (PATCH)
      xoff[j] = patch_chunk_offset<IS_I8>(a, (uint32_t)(m0 + rr), lchunk);
    else
      xoff[j] = (uint32_t)((int)rr * (int)k_bytes * XW + lchunk * 16);  // (the host keeps 32 rows of X below 2 GiB)
  }
  const int f0 = (n_blk & 3) * 4;
  const global_u8* Wrow = uniform_ptr((const uint8_t*)a.W + (int64_t)(n_blk >> 2) * ksteps * tile_bytes(IS_I8));
  const uint32_t a_lane = (uint32_t)(f0 * kFragValueBytes + lane * 16), i_lane = (uint32_t)index_offset(IS_I8, f0, lane);

  v4i xr[D][XL], ar[D][4];
  v4i ir[D];
  auto load = [&](int i, int slot) {
    const int ks = wave + NW * i;
    // a chunk past the end of a ragged row re-reads the row's first (and is zeroed before it is used)
    const bool ragged = tail_bytes != 0 && ks + 1 == ksteps;
    const global_u8* xb = Xtile + (PATCH ? patch_step_offset<IS_I8>(a, ks) : (int64_t)ks * (kStepBytes * XW));
    const uint32_t back = ragged && (lane % LPR) * 16 >= tail_bytes * XW ? (uint32_t)(lane % LPR) * 16u : 0u;
#pragma unroll
    for (int j = 0; j < XL; ++j) xr[slot][j] = *(const global_v4*)(xb + (xoff[j] - back));
    const global_u8* t = Wrow + (int64_t)ks * tile_bytes(IS_I8);
#pragma unroll
    for (int f = 0; f < 4; ++f) ar[slot][f] = *(const global_v4*)(t + a_lane + f * kFragValueBytes);
    if constexpr (IS_I8) {
      ir[slot] = *(const global_v4*)(t + i_lane);
    } else {
      const ep_v2u w = *(const global_v2u*)(t + i_lane);
      ir[slot] = v4i{(int)w[0], (int)w[1], 0, 0};
    }
  };
  auto load_batch = [&](int base) {
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (base + d < mine) load(base + d, d);  // wavefront-uniform
  };
  load_batch(0);

  // per-channel constants of the 8 channels this lane finishes (wavefront w: fragments 2g, 2g + 1 of slab mt)
  const int unit_g = wave & 1, unit_mt = (wave >> 1) & (TM - 1);
  const int n_lane = n_blk * kRowBlock + unit_g * 32 + (lane >> 4) * 8;
  const bool raw_out = IS_I8 && a.out_dt == GPUSQ_I32;
  float c8[8], b8[8];
#pragma unroll
  for (int j = 0; j < 8; j += 4) {
    float4 cc = float4{1.0f, 1.0f, 1.0f, 1.0f}, bb = float4{0.0f, 0.0f, 0.0f, 0.0f};
    if (n_lane + j < a.N && !raw_out) {  // N % 4 == 0
      if constexpr (IS_I8) cc = *(const float4*)(a.w_scale + n_lane + j);
      if (a.epilogue & GPUSQ_EPI_BIAS) bb = *(const float4*)(a.bias + n_lane + j);
    }
    c8[j] = cc.x; c8[j + 1] = cc.y; c8[j + 2] = cc.z; c8[j + 3] = cc.w;
    b8[j] = bb.x; b8[j + 1] = bb.y; b8[j + 2] = bb.z; b8[j + 3] = bb.w;
  }

  float s_a = 1.0f;
  const OutScale os = out_scale_of<IS_I8>(a);
  Fp16Quantiser qz;
  if constexpr (QUANT) {
    if constexpr (XQ == 2) {
      float amax = 0.0f;
      if (a.range_mode == kRangePartials) {
        for (int i = tid; i < a.npartial; i += 4 * 64 * NW) {  // (none is below 0; a range pass leaves at most 1024)
          float p[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) p[j] = a.partial[i + j * 64 * NW < a.npartial ? i + j * 64 * NW : i];
          amax = fmaxf(fmaxf(amax, fmaxf(p[0], p[1])), fmaxf(p[2], p[3]));
        }
      } else {
        amax = FP32 ? range_of_fp32((const float*)a.X, (int64_t)a.M * a.K, tid, 64 * NW) : range_of_fp16((const uint8_t*)a.X, (int64_t)a.M * a.K, tid, 64 * NW);
      }
      amax = wave_max_magnitude(amax);
      if (lane == 0) part[wave] = amax;
      __syncthreads();
      amax = part[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) amax = fmaxf(amax, part[w]);
      s_a = scale_of_range(amax);
      if (tile == 0 && tid == 0) a.scale_out[0] = s_a;
    } else {
      s_a = a.act_scale[0];
    }
    if constexpr (!FP32) {
      const unsigned wave_votes = qz.prepare(s_a, tid);
      if (lane == 0 && wave < 4) votes[wave] = wave_votes;
      __syncthreads();
      qz.decide((unsigned)__builtin_amdgcn_readfirstlane((int)(votes[0] | votes[1] | votes[2] | votes[3])));  // (threads 0..255)
    }
  } else if (IS_I8 && !raw_out) {
    s_a = a.act_scale[0];
  }
  const float r_a = FP32 ? scale_reciprocal(s_a) : 1.0f;
  const bool write_codes = QUANT && a.xq_out != nullptr && n_blk == 0;
  global_u8* xq_tile = uniform_ptr(a.xq_out + m0 * a.K);  // (rows past the end are the last one again, and so are their codes)

  acc_t acc[4][TM];
#pragma unroll
  for (int f = 0; f < 4; ++f)
#pragma unroll
    for (int mt = 0; mt < TM; ++mt) acc[f][mt] = acc_t{0, 0, 0, 0};

  uint8_t* xs = lds[wave];
  const uint8_t* xread = xs + (lane & 15) * kFrRow + (lane >> 4) * 16;
  auto compute = [&](int i, int slot) {
    const int ks = wave + NW * i;
    if (tail_bytes != 0 && ks + 1 == ksteps && (lane % LPR) * 16 >= tail_bytes * XW) {
#pragma unroll
      for (int j = 0; j < XL; ++j) xr[slot][j] = v4i{0, 0, 0, 0};
    }
    if constexpr (FP32) {
#pragma unroll
      for (int j = 0; j < XL; j += 2) {  // 4 fp32 values of row 2j + lane / 32 and 4 of two rows further -> 8 codes
        const ep_v4f lo = __builtin_bit_cast(ep_v4f, xr[slot][j]), hi = __builtin_bit_cast(ep_v4f, xr[slot][j + 1]);
        const float x[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        unsigned q[2];
        quantize_bytes8(x, s_a, r_a, q[0], q[1]);
        const int col = (lane & 31) * 4;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int r = 2 * (j + h) + (lane >> 5);
          *(unsigned*)(xs + r * kFrRow + col) = q[h];
          if (write_codes && ks * kStepBytes + col < a.K) *(global_u32*)(xq_tile + ks * kStepBytes + xoff[j + h] / XW) = q[h];
        }
      }
    } else if constexpr (QUANT) {
      unsigned c[XL][2];
      qz.codes_of<XQ == 1>(xr[slot], c);
      const int col = (lane & 15) * 8;
#pragma unroll
      for (int j = 0; j < XL; ++j) *(ep_v2u*)(xs + (4 * j + (lane >> 4)) * kFrRow + col) = ep_v2u{c[j][0], c[j][1]};  // 8 fp16 values -> 8 codes
      if (write_codes && ks * kStepBytes + col < a.K) {
#pragma unroll
        for (int j = 0; j < XL; ++j) *(global_v2u*)(xq_tile + ks * kStepBytes + xoff[j] / XW) = ep_v2u{c[j][0], c[j][1]};
      }
    } else {
#pragma unroll
      for (int j = 0; j < XL; ++j) *(v4i*)(xs + (8 * j + lrow) * kFrRow + lchunk * 16) = xr[slot][j];
    }
#pragma unroll
    for (int mt = 0; mt < TM; ++mt) {
      const uint8_t* p = xread + mt * 16 * kFrRow;
      const v4i lo = *(const v4i*)p, hi = *(const v4i*)(p + 64);
      const v8i b = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      if constexpr (IS_I8) {
#pragma unroll
        for (int f = 0; f < 4; ++f) acc[f][mt] = smfmac<true>(ar[slot][f], b, acc[f][mt], ir[slot][f]);
      } else {
        acc[0][mt] = smfmac<false, 0>(ar[slot][0], b, acc[0][mt], ir[slot][0]);
        acc[1][mt] = smfmac<false, 1>(ar[slot][1], b, acc[1][mt], ir[slot][0]);
        acc[2][mt] = smfmac<false, 0>(ar[slot][2], b, acc[2][mt], ir[slot][1]);
        acc[3][mt] = smfmac<false, 1>(ar[slot][3], b, acc[3][mt], ir[slot][1]);
      }
    }
  };
  for (int base = 0; base < mine;) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (base + d < mine) compute(base + d, d);  // wavefront-uniform
      __builtin_amdgcn_sched_barrier(0);          // one step at a time: interleaved, they need more registers than there are
    }
    base += D;
    if (base < mine) load_batch(base);
  }

  // ---- add the wavefronts' accumulators up: wavefront w finishes fragments 2g, 2g + 1 of slab mt
#pragma unroll
  for (int f = 0; f < 4; ++f)
#pragma unroll
    for (int mt = 0; mt < TM; ++mt) *(acc_t*)(xs + (mt * 4 + f) * 1024 + lane * 16) = acc[f][mt];
  __syncthreads();
  if (wave >= 2 * TM) return;
  acc_t sum[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int piece = (unit_mt * 4 + 2 * unit_g + t) * 1024 + lane * 16;
    sum[t] = *(const acc_t*)(&lds[0][piece]);
#pragma unroll
    for (int w = 1; w < NW; ++w) sum[t] += *(const acc_t*)(&lds[w][piece]);
  }
  const bool use_gelu = (a.epilogue & GPUSQ_EPI_GELU) != 0;
  float v[8];
  int raw[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if constexpr (IS_I8) {
      raw[j] = sum[j >> 2][j & 3];
      v[j] = epilogue_value<true>(raw[j], 0.0f, s_a * c8[j], b8[j]);
    } else {
      raw[j] = 0;
      v[j] = epilogue_value<false>(0, sum[j >> 2][j & 3], 1.0f, b8[j]);
    }
  }
  if (use_gelu) gelu_f32_x8(v);
  const int64_t m = m0 + unit_mt * 16 + (lane & 15);
  if (m < a.M) store_8<IS_I8>(a, m, n_lane, v, raw, os);
}

// Rows per tile: a round of 32-row tiles takes about half as long again as one of 16-row tiles, whichever needs less.
static int fewrows_tm(int64_t M, int64_t N, int resident) {
  const int64_t blocks = ceil_div(N, kRowBlock);
  return 2 * ceil_div(ceil_div(M, 16) * blocks, resident) > 3 * ceil_div(ceil_div(M, 32) * blocks, resident) ? 2 : 1;
}

// Quantising on the way in pays while one workgroup per CU carries the whole problem (eight wavefronts then, see below), or two do and
// one batch of K steps per wavefront is all.  Given scale, quantiser and GEMM / both in one, us (graph replays; a launch less is
// worth another microsecond where the host is what launches wait for): one workgroup per CU 320 x 1536 -> 768 6.9 / 5.4, 16 x 3072
// -> 1024 7.5 / 6.7, 96 x 4096 -> 2304 8.8 / 8.0; two, up to 12 steps 224 x 1024 -> 2304 6.7 / 6.2, 160 x 1536 -> 2304 7.2 / 7.2, beyond 160 x
// 3072 -> 2304 9.3 / 9.8, 160 x 4096 -> 2304 10.6 / 11.6; three 272 x 1024 -> 2304 7.3 / 8.8, and so at any K (64 to 1024, 256 to 4352
// channels, both types, either scale; quantiser and GEMM over both in one, graph replays: 2.4 to 3 workgroups 0.74 to 1.03, 6 0.58 to 0.82).
// The tiles are of 16 rows then: with 32 the 2304 channels take longer.
// fp32 rows are twice the bytes and come in vectors of 4: 320 x 384 -> 768 5.2 / 4.1, 320 x 1536 -> 768 6.6 / 6.0, but 320 x 3072 -> 768 8.6 / 10.2; two
// workgroups 672 x 384 -> 768 5.5 / 4.9, 672 x 768 -> 768 6.0 / 6.4.
bool fewrows_folds_quantiser(int64_t M, int64_t N, int64_t K, int resident, bool fp32) {
  const int64_t tiles = ceil_div(M, 16) * ceil_div(N, kRowBlock), ksteps = ceil_div(K, kStepBytes);
  if (fp32) return tiles <= resident ? ksteps <= 12 : (tiles <= 2 * (int64_t)resident && ksteps <= 4);
  return tiles <= resident ? ksteps <= 40 : (tiles <= 2 * (int64_t)resident && ksteps <= kFrWaves * kFrBatch);
}

// 8 wavefronts to a workgroup that quantises, while there is at most one to a CU: a wavefront alone on its SIMD issues an instruction
// every 2.1 ns, and quantising takes some 40 of them per 16 bytes of X and lane.  Up to four K steps, or a range of X found here
// over no more than 96 KB, are too little work for it (graph replays, 4 / 8 wavefronts, us: given scale 333 x 1040 -> 520 5.9 / 5.0, 16 x 3072
// -> 768 8.9 / 6.7, 64 x 1024 -> 1024 5.1 / 4.6, but 197 x 192 -> 768 3.9 / 4.1, 100 x 384 -> 384 3.9 / 4.1; range found here
// 331 x 192 -> 384, 127 KB, 6.2 / 5.9, 197 x 192 -> 768, 75 KB, 5.5 / 5.8).
static bool fewrows_wide(const GemmArgs& a, int tiles_n, int tiles_m, int resident) {
  const bool long_range = a.range_mode == kRangeHere && (int64_t)a.M * a.K * (a.x_f16 == 2 ? 4 : 2) > 96 * 1024;
  return (int64_t)tiles_n * tiles_m <= resident && (ceil_div(a.K, kStepBytes) > 4 || long_range);
}

bool fewrows_supports(const GemmArgs& a) {
  return (int64_t)a.K * 2 * 32 < ((int64_t)1 << 31);  // 32-bit lane offsets inside a tile's rows of X
}

gpusq_status launch_fewrows(bool is_i8, const GemmArgs& a, int resident, hipStream_t s) {
  const int tm = a.x_f16 ? 1 : fewrows_tm(a.M, a.N, resident);
  const int tiles_n = (int)ceil_div(a.N, kRowBlock), tiles_m = (int)ceil_div(a.M, 16 * tm);
  const int n_fast = (int64_t)a.M * 8 > (int64_t)a.N * 5;  // X larger than the packed weights: its rows stay on one XCD
  const unsigned grid = (unsigned)ceil_div((int64_t)tiles_n * tiles_m, 8) * 8;
  const bool quantise = is_i8 && a.x_f16, given = a.range_mode == kRangeGiven;
#define GPUSQ_FEWROWS(...) spgemm_fewrows_kernel<__VA_ARGS__><<<grid, 64 * kFrWaves, 0, s>>>(a, tiles_n, tiles_m, n_fast)
#define GPUSQ_FEWROWS_WIDE(...) spgemm_fewrows_kernel<__VA_ARGS__, false, 8><<<grid, 512, 0, s>>>(a, tiles_n, tiles_m, n_fast)
#define GPUSQ_FEWROWS_FP32(XQ, NW) spgemm_fewrows_kernel<true, 1, XQ, false, NW, 4><<<grid, 64 * NW, 0, s>>>(a, tiles_n, tiles_m, n_fast)
  if (quantise && a.x_f16 == 2) {
    const bool wide = fewrows_wide(a, tiles_n, tiles_m, resident);
    if (wide && given) GPUSQ_FEWROWS_FP32(1, 8);
    else if (wide) GPUSQ_FEWROWS_FP32(2, 8);
    else if (given) GPUSQ_FEWROWS_FP32(1, 4);
    else GPUSQ_FEWROWS_FP32(2, 4);
  }
  else if (quantise && fewrows_wide(a, tiles_n, tiles_m, resident) && given) GPUSQ_FEWROWS_WIDE(true, 1, 1);
  else if (quantise && fewrows_wide(a, tiles_n, tiles_m, resident)) GPUSQ_FEWROWS_WIDE(true, 1, 2);
  else if (quantise && given) GPUSQ_FEWROWS(true, 1, 1);
  else if (quantise) GPUSQ_FEWROWS(true, 1, 2);
  else if (a.patch_P != 0 && is_i8 && tm == 2) GPUSQ_FEWROWS(true, 2, 0, true);
  else if (a.patch_P != 0 && is_i8) GPUSQ_FEWROWS(true, 1, 0, true);
  else if (a.patch_P != 0 && tm == 2) GPUSQ_FEWROWS(false, 2, 0, true);
  else if (a.patch_P != 0) GPUSQ_FEWROWS(false, 1, 0, true);
  else if (is_i8 && tm == 2) GPUSQ_FEWROWS(true, 2, 0);
  else if (is_i8) GPUSQ_FEWROWS(true, 1, 0);
  else if (tm == 2) GPUSQ_FEWROWS(false, 2, 0);
  else GPUSQ_FEWROWS(false, 1, 0);
#undef GPUSQ_FEWROWS
#undef GPUSQ_FEWROWS_WIDE
#undef GPUSQ_FEWROWS_FP32
  return check_launch();
}

}  // namespace gpusq
