// Sparse INT8 GEMM on activations that it quantises itself, for many rows and few output channels: whole rows of Y.
//
// The tile kernels read codes that a quantiser pass has written, each column tile all of them again.  Here a workgroup has all
// channels of its rows (up to 12 blocks of 64; more are split into equal column blocks), so the fp16 or fp32 activations come from
// memory once, are turned into codes on the way and multiplied, and the pass that did nothing else is gone.
//   - 4 wavefronts (producers) request the rows of X several K steps ahead into LDS, quantise a step and put its codes into
//     one of two LDS buffers, and into Xq; one wavefront per 64 channels (consumers) reads the other buffer and multiplies.  One barrier per
//     K step.  The roles are wavefronts of their own because loads return in order per wavefront: a consumer's weights, an L2 hit away,
//     would wait behind rows of X from HBM.
//   - a consumer's kept values and index words go from the packed buffer (in lane order) straight into its registers, one step ahead:
//     no two of them need the same.
//   - persistent: a workgroup keeps its column block and walks row chunks; the producers' requests run on across chunks.
// A K step of 64 rows and 768 channels brings 61 KB of weights and 16 KB of X into the CU (1200 clocks at 64 bytes a clock), its matrix
// instructions take 790 clocks: bound by memory (X in, codes and Y out) as long as a chunk has enough K steps.  In the kernel (12608 rows of 768,
// clocks): 6000 until the first codes (range, constants, HBM), six steps of 1900 to 2000, 2900 for the epilogue.
// The layer in us, the quantiser and the GEMM one after the other against this (fp16 X and Y, normal values, calls in turn on three buffers; cards
// differ by 3 %), own range and given scale:
//   14070 x 576 -> 256  16.3 / 14.2, 12.8 / 10.0     12608 x 768 -> 768  20.6 / 20.0, 17.1 / 15.1     7029 x 1152 -> 256  17.0 / 15.0, 13.5 / 10.9
//   50432 x 192 -> 192  18.9 / 17.4, 15.5 / 13.2     25216 x 3072 -> 768  106.7 / 107.5, 86.5 / 83.9 (GELU's output, own range: 102.5 / 100.3)
#include <type_traits>

#include "tile_common.h"
#include "wide_plan.h"

namespace gpusq {

// s_waitcnt vmcnt(n) (gfx9 encoding: vmcnt [3:0] and [15:14], expcnt [6:4], lgkmcnt [11:8])
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "6-bit counter");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

constexpr int kProducers = 4, kProducerThreads = 64 * kProducers;

typedef __attribute__((address_space(1))) v4i global_v4;
typedef __attribute__((address_space(1))) ep_v2u global_v2u;
typedef __attribute__((address_space(1))) unsigned global_u32;

// S: slabs of 16 rows of the highest chunk.
// GELU, OUT: the epilogue (fp16 or int8 output).  16-byte pieces of a row; 4 channels of a lane's own at a time where a row is no whole 16 channels (3000 x 768 -> 388 from
// fp32, the quantiser and a GEMM with such stores 13.2 us, here 11.4).
// PATCH: X is an image batch, a row a 16 x 16 patch (see patch_chunk_offset), and the codes are those of the images, where their pixels are.
template <int S, bool FP32, int GELU, int OUT, bool PATCH = false>
__global__ void __launch_bounds__(64 * kWideWaves) spgemm_wide_kernel(const GemmArgs a, const WidePlan p) {
  constexpr int XW = FP32 ? 4 : 2;           // bytes of X in memory per code
  constexpr int XL = S * XW / 2;             // 16-byte copies per producer lane and K step
  constexpr int D = kWideDepth;              // K steps of X in flight
  constexpr int kStage = 16 * S * kStepBytes;
  __shared__ __attribute__((aligned(1024))) uint8_t raw[D * XL * 1024 * kProducers];  // X as it is in memory: every lane reads back what it asked for
  __shared__ __attribute__((aligned(16))) uint8_t ring[2][kStage];
  __shared__ __attribute__((aligned(16))) float cs[kWideBlocks * kRowBlock], bs[kWideBlocks * kRowBlock];
  __shared__ float part[kWideWaves];
  __shared__ unsigned votes[4];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = (int)(blockDim.x >> 6);
  const WidePlace at = wide_place(p, (int)blockIdx.x);
  if (at.items == 0) return;  // the whole workgroup leaves before any barrier
  const int ksteps = (a.K + kStepBytes - 1) / kStepBytes, tail = a.K % kStepBytes;
  const int steps = at.items * ksteps;

  // The scale: the consumers read it, or fold the range (the producers' loads would be waited for behind their rows of X).
  const bool given = a.range_mode == kRangeGiven;
  auto ask_scale = [&]() __attribute__((always_inline)) {
    if (given) {
      part[wave] = a.act_scale[0];
      return;
    }
    const int first = tid - kProducerThreads, threads = (int)blockDim.x - kProducerThreads;
    float amax = 0.0f;
    for (int i = first; i < a.npartial; i += 4 * threads) {  // (none is below 0; a range pass leaves at most 1024)
      float v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = a.partial[i + j * threads < a.npartial ? i + j * threads : i];
      amax = fmaxf(fmaxf(amax, fmaxf(v[0], v[1])), fmaxf(v[2], v[3]));
    }
    amax = wave_max_magnitude(amax);
    if (lane == 0) part[wave] = amax;
  };
  auto scale = [&]() __attribute__((always_inline)) {  // behind a barrier
    if (given) return part[kProducers];
    float amax = 0.0f;
    for (int w = kProducers; w < waves; ++w) amax = fmaxf(amax, part[w]);
    return amax == 0.0f ? 1.0f : __fdiv_rn(amax, 127.0f);
  };
  if (wave < kProducers) {
    // ------------------------------------------------------------------------------------------------ producers
    constexpr int LPR = 8 * XW, RPL = kProducerThreads / LPR;  // lanes per row, rows per load
    // row of a lane's first copy, and its first code within the step: consecutive lanes along a row of X, or along a row of the image, where
    // neighbouring patches' pieces of 16 pixels are contiguous
    constexpr int PPR = XW;                                    // 16-byte pieces of 16 pixels
    const int in_wave = PATCH ? (lane / PPR) % (64 / LPR) : lane / LPR;
    const int row = wave * (64 / LPR) + in_wave;
    const int code = PATCH ? lane / (64 / 8) * 16 + lane % PPR * (16 / XW) : lane % LPR * (16 / XW);
    const uint32_t raw_lds = lds_address(raw) + (uint32_t)wave * 1024u;
    // The cursor of the requests, and behind it, D steps, that of the codes: chunk, K step, and where they are in memory.  A row past the
    // chunk's last is the last again, a piece of X past the end of a ragged row the step's first (its weights are zero): their codes are
    // then written once more to where they stand already, and every step has the same copies and stores, without a condition, which the
    // waits count.  So do the requests and the codes past the last step: they are that step again.
    struct Cursor {
      uint32_t unit;      // bytes of a value (X) or a code
      int item, ks;
      int64_t at;         // chunk and step: in values from the first
      uint32_t off[XL];   // this lane's pieces, in bytes from there
    };
    auto clip = [&](Cursor& c) __attribute__((always_inline)) {  // the step is a row's last, and ragged
      if (tail != 0 && c.ks + 1 == ksteps) {
        const uint32_t back = code >= tail ? (uint32_t)code * c.unit : 0u;
#pragma unroll
        for (int j = 0; j < XL; ++j) c.off[j] -= back;
      }
    };
    auto seek = [&](Cursor& c, int item) __attribute__((always_inline)) {
      const WideChunk ch = wide_chunk(p, at, item);
      c.item = item;
      c.ks = 0;
      c.at = PATCH ? 0 : ch.m0 * a.K;
#pragma unroll
      for (int j = 0; j < XL; ++j) {
        const int r = row + RPL * j;
        if constexpr (PATCH)
          c.off[j] = (patch_pixel(a, (uint32_t)ch.m0 + (uint32_t)(r < ch.rows ? r : ch.rows - 1)) + (uint32_t)(code / 16 * a.patch_W + code % 16)) * c.unit;
        else
          c.off[j] = ((uint32_t)(r < ch.rows ? r : ch.rows - 1) * (uint32_t)a.K + (uint32_t)code) * c.unit;  // (the host keeps 64 rows of X below 2 GiB)
      }
      clip(c);
    };
    auto advance = [&](Cursor& c) __attribute__((always_inline)) {
      if (c.ks + 1 < ksteps) {
        ++c.ks;
        c.at = PATCH ? patch_step_offset<true>(a, c.ks) : c.at + kStepBytes;
        clip(c);
      } else if (c.item + 1 < at.items) {
        seek(c, c.item + 1);
      }
    };
    Cursor pf;
    pf.unit = FP32 ? 1 : XW;  // (fp32: to bytes at the request; 1.5 % faster there)
    seek(pf, 0);
    auto request = [&](uint32_t slot) __attribute__((always_inline)) {  // slot: byte offset of the step's stage
      const global_u8* x = uniform_ptr((const uint8_t*)a.X + pf.at * XW);
#pragma unroll
      for (int j = 0; j < XL; ++j) copy16_to_lds((const void*)x, pf.off[j] * (uint32_t)(FP32 ? XW : 1), raw_lds + slot + (uint32_t)j * (1024u * kProducers));
      advance(pf);
    };
    constexpr uint32_t kRawStage = XL * 1024u * kProducers;
    constexpr int early = FP32 ? D : 1;
#pragma nounroll
    for (int d = 0; d < early; ++d) request((uint32_t)d * kRawStage);
    __syncthreads();  // the scale
#pragma nounroll
    for (int d = early; d < D; ++d) request((uint32_t)d * kRawStage);
    const float s_a = scale();
    if (!given && blockIdx.x == 0 && tid == 0) a.scale_out[0] = s_a;
    Fp16Quantiser qz;
    float r_a = 0.0f;
    if constexpr (FP32) {
      r_a = scale_reciprocal(s_a);
    } else {
      const unsigned wave_votes = qz.prepare(s_a, tid);
      if (lane == 0) votes[wave] = wave_votes;
    }
    __syncthreads();
    if constexpr (!FP32) qz.decide((unsigned)__builtin_amdgcn_readfirstlane((int)(votes[0] | votes[1] | votes[2] | votes[3])));

    // where this lane's codes lie in a buffer: row-major, 16-byte chunk c of row r at c ^ ((r >> 1) & 7)
    const uint32_t ring_off = (uint32_t)(row * kStepBytes + (((code >> 4) ^ ((row >> 1) & 7)) << 4) + (code & 15));
    // The codes go past the caches (nothing here reads them again) where a step's are whole 128-byte lines; rows that start inside a line are
    // left to the L2 to put together: 28919 x 2256 -> 128 under a given scale 52.5 us, 75.6 past the caches (the quantiser and the GEMM one after the other: 62.7).
    // Those of images are pieces of 32 or 64 bytes along a row of pixels, whose lines are whole a few instructions later: either way is as fast (123
    // sizes, 0.1 % on average, 3 % at the most).
    auto store_codes = [&](auto v, auto* at) __attribute__((always_inline)) {
      if (tail == 0)
        __builtin_nontemporal_store(v, at);
      else
        *at = v;
    };
    Cursor here;
    here.unit = 1;
    seek(here, 0);
    uint32_t slot = 0;
    // One step: its rows have landed when no more than the copies and stores requested behind them are in flight.
    // MODE (fp16): 0 the scale of X's own range and one fused multiply-add a value (the code of a NaN is 0 as it is: its low byte), 1 a given
    // scale, 2 products that are refined.  Loops of their own, with no question per step, and the first step alone requested in front of the
    // scale's barrier, before -> after on one card: 50432 x 192 -> 192 18.9 -> 17.9 us, under a given scale 14.2 -> 13.4; 12608 x 768 -> 768 -0.3, -0.5 us.
    auto produce = [&](auto write, auto mode, bool first, uint8_t* dst) __attribute__((always_inline)) {
      constexpr bool WRITE = decltype(write)::value;
      constexpr int MODE = decltype(mode)::value;
      if (WRITE && !first)
        wait_vm<(D - 1) * 2 * XL>();
      else
        wait_vm<(D - 1) * XL>();
      asm volatile("" ::: "memory");
      const uint8_t* mine = raw + slot + tid * 16;
      v4i x[XL];
#pragma unroll
      for (int j = 0; j < XL; ++j) x[j] = *(const v4i*)(mine + j * (1024 * kProducers));
      unsigned c[XL][2];
      if constexpr (FP32) {
#pragma unroll
        for (int j = 0; j < XL; j += 2) {
          const ep_v4f lo = __builtin_bit_cast(ep_v4f, x[j]), hi = __builtin_bit_cast(ep_v4f, x[j + 1]);
          const float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
          quantize_bytes8(v, s_a, r_a, c[j][0], c[j + 1][0]);
        }
      } else {
        const bool odd = MODE != 0 && qz.odd(x);
        if (MODE == 2 || __builtin_expect(odd, 0)) {
#pragma unroll
          for (int j = 0; j < XL; ++j) {
            if constexpr (MODE == 1) asm volatile("" : "+v"(x[j]));  // (shares nothing with the other branch)
            qz.codes<true>(x[j], odd, c[j][0], c[j][1]);
          }
        } else {
          const Fp16Quantiser plain{qz.s, qz.r, false};
#pragma unroll
          for (int j = 0; j < XL; ++j) plain.codes<MODE != 0>(x[j], false, c[j][0], c[j][1]);
        }
      }
      global_u8* q = uniform_ptr(a.xq_out + here.at);
#pragma unroll
      for (int j = 0; j < XL; ++j) {
        uint32_t off = here.off[j];
        asm volatile("" : "+v"(off));
        if constexpr (FP32) {
          *(unsigned*)(dst + (ring_off ^ (j & 1 ? 64u : 0u)) + RPL * j * kStepBytes) = c[j][0];  // 8 rows further the swizzle differs in its highest bit
          if constexpr (WRITE) store_codes(c[j][0], (__attribute__((address_space(1))) unsigned*)(q + off));
        } else {
          const ep_v2u both = {c[j][0], c[j][1]};
          *(ep_v2u*)(dst + ring_off + RPL * j * kStepBytes) = both;  // 16 rows further: the same swizzle
          if constexpr (WRITE) store_codes(both, (global_v2u*)(q + off));
        }
      }
      advance(here);
      request(slot);
      slot = slot + kRawStage == D * kRawStage ? 0 : slot + kRawStage;
    };
    auto run = [&](auto write, auto mode) __attribute__((always_inline)) {
      uint32_t buf = 0;
#pragma nounroll
      for (int g = 0; g <= steps; ++g) {  // (behind the last step: that one again, into the buffer that nothing reads any more)
        produce(write, mode, g <= D, ring[0] + buf);
        buf ^= kStage;
        __syncthreads();
      }
    };
    auto run_mode = [&](auto mode) __attribute__((always_inline)) {
      if (at.n_blk == 0)
        run(std::true_type{}, mode);
      else
        run(std::false_type{}, mode);
    };
    if (FP32 || (!given && !qz.refine))
      run_mode(std::integral_constant<int, 0>{});
    else if (!qz.refine)
      run_mode(std::integral_constant<int, 1>{});
    else
      run_mode(std::integral_constant<int, 2>{});
    wait_vm<0>();  // the copies requested past the end land before the LDS is given up
    return;
  }

  // -------------------------------------------------------------------------------------------------- consumers
  const int w = wave - kProducers;
  const int last_blk = (a.N - 1) / kRowBlock;
  const int blk = at.n_blk * p.blocks + w;  // 64-channel block; past the last one (an uneven split): the last again, nothing stored
  const int wblk = blk < last_blk ? blk : last_blk;
  const int f0 = (wblk & 3) * 4;
  const global_u8* Wrow = uniform_ptr((const uint8_t*)a.W + (int64_t)(wblk >> 2) * ksteps * tile_bytes(true));
  const uint32_t a_lane = (uint32_t)(f0 * kFragValueBytes + lane * 16), i_lane = (uint32_t)index_offset(true, f0, lane);
  v4i ar[2][4], ir[2];
  auto load_a = [&](int ks, int set) __attribute__((always_inline)) {
    const global_u8* t = Wrow + (int64_t)ks * tile_bytes(true);
    uint32_t a_now = a_lane, i_now = i_lane;
    asm volatile("" : "+v"(a_now), "+v"(i_now));  // (widened here: scalar-base addressing)
#pragma unroll
    for (int f = 0; f < 4; ++f) ar[set][f] = *(const global_v4*)(t + a_now + f * kFragValueBytes);
    ir[set] = *(const global_v4*)(t + i_now);
  };
  load_a(0, 0);
  // this lane's channel of the wavefront's constants
  const int n_wave = blk * kRowBlock;
  const int n_lane = n_wave + lane < a.N ? n_wave + lane : a.N - 1;
  const float w_lane = a.w_scale[n_lane], b_lane = (a.epilogue & GPUSQ_EPI_BIAS) ? a.bias[n_lane] : 0.0f;
  ask_scale();
  __syncthreads();
  const float s_a = scale();
  const float s_out = OUT == GPUSQ_I8 ? a.out_scale[0] : 1.0f, r_out = scale_reciprocal(s_out);
  cs[w * kRowBlock + lane] = s_a * w_lane;
  bs[w * kRowBlock + lane] = b_lane;
  __syncthreads();
  __syncthreads();  // the first step's codes

  v4i acc[4][S];
  const uint32_t b_lo = (uint32_t)((lane & 15) * kStepBytes + (((lane >> 4) ^ ((lane & 15) >> 1)) << 4)), b_hi = b_lo ^ 64u;
  uint32_t buf = 0;
  // Multiplies a step with one set of weights while the next step's (`next`; the first again behind the last) come into the other.
  auto step = [&](int set, int next) __attribute__((always_inline)) {
    load_a(next, set ^ 1);
    __builtin_amdgcn_sched_barrier(0);
    const uint8_t* src = ring[0] + buf;
#pragma unroll
    for (int mt = 0; mt < S; ++mt) {
      const v4i lo = *(const v4i*)(src + b_lo + mt * 16 * kStepBytes), hi = *(const v4i*)(src + b_hi + mt * 16 * kStepBytes);
      const v8i b = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
#pragma unroll
      for (int f = 0; f < 4; ++f) acc[f][mt] = smfmac<true>(ar[set][f], b, acc[f][mt], ir[set][f]);
    }
    buf ^= kStage;
    __syncthreads();
  };

#pragma nounroll
  for (int item = 0; item < at.items; ++item) {
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
      for (int mt = 0; mt < S; ++mt) acc[f][mt] = v4i{0, 0, 0, 0};
    int ks = 0;
#pragma nounroll
    for (; ks + 2 <= ksteps; ks += 2) {
      step(0, ks + 1);
      step(1, ks + 2 < ksteps ? ks + 2 : 0);
    }
    if (ks < ksteps) {
      step(0, 0);
#pragma unroll
      for (int f = 0; f < 4; ++f) ar[0][f] = ar[1][f];
      ir[0] = ir[1];
    }
    if (blk > last_blk) continue;
    // ---- the epilogue runs beside the producers' first step of the next chunk
    const WideChunk ch = wide_chunk(p, at, item);
    constexpr int OB = dtype_bytes(OUT);
    int lane_now = lane;
    asm volatile("" : "+v"(lane_now));  // (what follows from the lane is computed here, not kept across the K loop)
    const int c16 = lane_now & 15, q = lane_now >> 4, up = c16 >> 3;
    const float *cw = cs + w * kRowBlock + q * 8, *bw = bs + w * kRowBlock + q * 8;
    const int64_t n_bytes = (int64_t)a.N * OB;
    const bool narrow = a.N % 16 != 0;  // rows that start where no 16-byte store may
    global_u8* y = uniform_ptr((uint8_t*)a.Y + ch.m0 * n_bytes + (int64_t)n_wave * OB);
#pragma unroll
    for (int mt = 0; mt < S; ++mt) {
      const int r0 = mt * 16;
      auto values = [&](int g, float (&v)[8]) __attribute__((always_inline)) {
        asm volatile("" ::: "memory");  // the constants are read again for every slab: kept, they and the accumulators are more than 128 registers
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = (float)acc[2 * g + (j >> 2)][mt][j & 3];
        pin8(v);
#pragma unroll
        for (int j = 0; j < 8; j += 4) {
          const float4 cc = *(const float4*)(cw + g * 32 + j), bb = *(const float4*)(bw + g * 32 + j);
          v[j] = __fmaf_rn(v[j], cc.x, bb.x);
          v[j + 1] = __fmaf_rn(v[j + 1], cc.y, bb.y);
          v[j + 2] = __fmaf_rn(v[j + 2], cc.z, bb.z);
          v[j + 3] = __fmaf_rn(v[j + 3], cc.w, bb.w);
        }
        if constexpr (GELU != 0) gelu_f32_x8(v);
        pin8(v);  // (rounded to fp32 before anything else)
      };
      if constexpr (OUT == GPUSQ_F16) {  // two stores of 8 rows x 128 bytes (see store_line_pair)
        ep_v4i H[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          float v[8];
          values(g, v);
          ep_v8h hh;
#pragma unroll
          for (int j = 0; j < 8; ++j) hh[j] = (_Float16)v[j];
          H[g] = __builtin_bit_cast(ep_v4i, hh);
        }
        if (narrow) {  // a lane's own channels, by four
#pragma unroll
          for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              uint32_t off = (uint32_t)(c16 * (int)n_bytes + g * 64 + q * 16 + j * 8);
              asm volatile("" : "+v"(off));
              if (r0 + c16 < ch.rows && n_wave + g * 32 + q * 8 + j * 4 < a.N) *(global_v2u*)(y + r0 * n_bytes + off) = ep_v2u{(unsigned)H[g][2 * j], (unsigned)H[g][2 * j + 1]};
            }
          continue;
        }
        const bool n_ok = n_wave + up * 32 + q * 8 < a.N;
        const int r = r0 + (c16 & 7);
        store_line_pair(H[0], H[1], y + r0 * n_bytes, (uint32_t)((c16 & 7) * (int)n_bytes + up * 64 + q * 16), 8 * n_bytes, n_ok && r < ch.rows, n_ok && r + 8 < ch.rows);
      } else {  // lanes q = 2j, 2j + 1 exchange halves: 16 consecutive codes each, of the first 32 channels and of the second
        unsigned d[2][2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          float v[8];
          values(g, v);
          quantize_bytes8(v, s_out, r_out, d[g][0], d[g][1]);
        }
        if (narrow) {
#pragma unroll
          for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              uint32_t off = (uint32_t)(c16 * (int)n_bytes + g * 32 + q * 8 + j * 4);
              asm volatile("" : "+v"(off));
              if (r0 + c16 < ch.rows && n_wave + g * 32 + q * 8 + j * 4 < a.N) *(global_u32*)(y + r0 * n_bytes + off) = d[g][j];
            }
          continue;
        }
        const ep_v2u lo = __builtin_amdgcn_permlane16_swap(d[0][0], d[1][0], false, false);
        const ep_v2u hi = __builtin_amdgcn_permlane16_swap(d[0][1], d[1][1], false, false);
        const int nl = (q & 1) * 32 + (q >> 1) * 16;
        uint32_t off = (uint32_t)(c16 * (int)n_bytes + nl);
        asm volatile("" : "+v"(off));
        if (r0 + c16 < ch.rows && n_wave + nl < a.N) *(global_v4i*)(y + r0 * n_bytes + off) = ep_v4i{(int)lo[0], (int)hi[0], (int)lo[1], (int)hi[1]};
      }
    }
  }
}

gpusq_status launch_wide(const GemmArgs& a, const WidePlan& p, hipStream_t s) {
  const unsigned grid = 8u * (unsigned)p.per_xcd, threads = 64u * (unsigned)(kProducers + p.blocks);
  const int slabs = wide_slabs(p);
  const bool gelu = (a.epilogue & GPUSQ_EPI_GELU) != 0;
  // (few of the combinations exist with patches: fp16 output without GELU)
#define GPUSQ_WIDE_X(S, FP32)                                                                                              \
  (a.patch_P != 0 ? spgemm_wide_kernel<S, FP32, 0, GPUSQ_F16, true> : a.out_dt == GPUSQ_I8 ? (gelu ? spgemm_wide_kernel<S, FP32, 1, GPUSQ_I8> : spgemm_wide_kernel<S, FP32, 0, GPUSQ_I8>)    \
                        : (gelu ? spgemm_wide_kernel<S, FP32, 1, GPUSQ_F16> : spgemm_wide_kernel<S, FP32, 0, GPUSQ_F16>)) \
      <<<grid, threads, 0, s>>>(a, p)
#define GPUSQ_WIDE(S)         \
  case S:                     \
    if (a.x_f16 == 2)         \
      GPUSQ_WIDE_X(S, true);  \
    else                      \
      GPUSQ_WIDE_X(S, false); \
    break;
  switch (slabs) {
    GPUSQ_WIDE(1)
    GPUSQ_WIDE(2)
    GPUSQ_WIDE(3)
    GPUSQ_WIDE(4)
    default: return GPUSQ_ERR_UNSUPPORTED;
  }
#undef GPUSQ_WIDE
#undef GPUSQ_WIDE_X
  return check_launch();
}

}  // namespace gpusq
