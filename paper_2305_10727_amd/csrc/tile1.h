// Tile kernel of the 2:4 sparse GEMM with one persistent workgroup per CU: tiles of 256 channels x up to 256 rows.  (A header:
// its many instantiations are compiled in four translation units, tile1_{i8,f16}{,_ragged}.hip.)
//
// 8 wavefronts, 2 along n x 4 along m, 128 channels x up to 4 slabs of 16 rows each and 128 accumulator registers.  All of them
// run the K loop of a tile, then all run its epilogue.  With two wavefronts per SIMD in the same phase, a SIMD always has a
// second wavefront to issue from while one waits, and the weight tile is brought into the CU once per 256 rows.
//
// Tile heights.  The rows of X are cut into chunks of whole 32-row units, all of the same height or one unit more (EvenPlan), and
// the number of chunks is chosen so that the tiles fill whole rounds over the CUs: the last round is as full as the others.
// With heights in steps of 64 rows and the rest in short tail tiles, 12608 x 768 -> 3072 took two full tiles and a half one per
// CU, and the half one cost as much time in its K loop as a full one (what a step costs besides its matrix instructions does
// not shrink with it).  A tile's 16-row slabs are dealt out over the four wavefronts along m, the first two take the extra
// ones; the two wavefronts of a SIMD are 2 apart along m, so every SIMD has as many.  (Steps of 16 rows leave two SIMDs with
// a slab less than the others: no faster than the next step of 32.)  With both (and the K step below), before and
// now: 12608 x 768 -> 3072 + GELU fp16 50.2 -> 47.6 us, 3136 x 4096 -> 1024 int8 20.6 -> 17.6, fp16 37.7 -> 30.1, 3152 x 768 ->
// 3072 + GELU int8 14.2 -> 12.5; 65792 x 1280 -> 5120 + GELU int8, whose rounds were even before, stays at 370 (128 of them for its
// matrix instructions alone).
//
// LDS: a ring of stages (X slab NX * 8 KB, kept values 16 KB, index words 4/2 KB).  NX = ceil(slabs of the highest tile / 4) is fixed per launch:
// copies per wavefront and K step along X, and slabs per wavefront; a ring of lower tiles has lower, more stages (3, 3, 4, 5 for
// NX = 4, 3, 2, 1).  K steps are numbered g = 0, 1, ... over the workgroup's whole sequence of tiles; step g lives in stage g % R.
// One workgroup barrier per K step, in front of the last two matrix instructions of its first half: by then a wavefront has
// issued, and waits for, the last LDS read of the step's stage, and it waits for its own copies of step g+1 (the vector-memory
// counter retires in order).  Behind the barrier stage g+1 is complete and is read ahead, and stage g is free: the copies of
// step g+R are requested there, R-1 whole steps before they are needed, also across tile boundaries (the next tile's first
// steps land during the epilogue).  Every wavefront executes exactly one barrier per step of every tile of the workgroup, plus
// one at start-up.
//
// Ragged K (no whole number of 128-byte steps): the weights are packed with zeros past the row end, and in a row's last step the
// lanes whose 16-byte chunk lies past it re-read the step's first.  int8 needs no more (whatever is multiplied by the zeros adds
// nothing); fp16 activations may hold infinities or NaN, so there the wavefront that copied those chunks overwrites them with
// zeros once they have landed, in front of the barrier that publishes the stage.  Such problems took the small kernel's
// 128 x 128 tiles before: 65536 x 592 -> 1280 int8 80.0 -> 57.4 us, fp16 122.8 -> 85.7; 25088 x 4400 -> 1100 int8 148 -> 95, fp16
// 300 -> 182; 12544 x 192 -> 768 int8 12.6 -> 7.7; 3152 x 576 -> 1728 int8 10.4 -> 8.1, fp16 13.3 -> 9.6.
#pragma once
#include <type_traits>

#include "tile_common.h"

namespace gpusq {

constexpr int kTileWM = 4;
static_assert(kTileWM * 16 == kTileUnitRows, "one copy block row per wavefront along m");

template <bool IS_I8, int NX>
struct Ring {
  static constexpr int kXSlab = NX * 8192;  // 64 * NX rows x 128 bytes, 16-byte chunks XOR-swizzled per row
  static constexpr int kStage = kXSlab + tile_bytes(IS_I8);
  static constexpr int kStages = NX == 4 ? 3 : (NX == 3 ? 3 : (NX == 2 ? 4 : 5));
  static constexpr int kCopies = NX + 3;  // copy instructions per wavefront and K step: NX X blocks, 2 fragments, 1 KB of index words
  static_assert(kStages * kStage + 4096 <= 160 * 1024, "the ring and the constants fill the CU's LDS");
};

// s_waitcnt lgkmcnt(0) and vmcnt(n) (gfx9 encoding: vmcnt [3:0] and [15:14], expcnt [6:4], lgkmcnt [11:8])
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "6-bit counter");
  __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
}

// Copy I of one wavefront's share (an eighth) of the copies that bring one K step of a tile into an LDS stage: I < NX are 1 KB
// blocks of the X slab (block j = wave + 8I holds rows 8j..8j+7), I = NX, NX + 1 fragments of kept values, I = NX + 2 1 KB of
// index words.  Each copy moves 64 lanes x 16 bytes from a wavefront-uniform 64-bit base in scalar registers plus a 32-bit
// per-lane offset that is fixed for the whole tile, to 1 KB of consecutive LDS at a scalar base plus a constant: per copy the
// K loop spends one scalar instruction and one wait state besides the copy itself.
//   lds_wave = LDS address of the stage + wave * 1024, lds_idx = that of the index block this wavefront copies;
//   Xks = the X rows of the tile at this K step, Wwave = the packed tile of this K step + wave * 1024;
//   loff = lane * 16, loff8k = loff + 8192, ioff = loff + the index block's offset relative to Wwave.
// Always exactly NX + 3 instructions per step, whatever the tile (a lower tile copies rows it does not use; there are only
// 4 KB / 2 KB of index words, so some wavefronts repeat a block), so that the waits can count instructions.
template <bool IS_I8, int NX, int I>
__device__ __forceinline__ void issue_step_copy(uint32_t lds_wave, uint32_t lds_idx, const uint8_t* Xks, const uint8_t* Wwave,
                                                const uint32_t (&xoff)[NX], uint32_t loff, uint32_t loff8k, uint32_t ioff) {
  constexpr int kXSlab = Ring<IS_I8, NX>::kXSlab;
  if constexpr (I < NX)
    copy16_to_lds_at<8192 * I>(Xks, xoff[I < NX ? I : 0], lds_wave);
  else if constexpr (I == NX)
    copy16_to_lds_at<kXSlab>(Wwave, loff, lds_wave);
  else if constexpr (I == NX + 1)
    copy16_to_lds_at<kXSlab + 8192>(Wwave, loff8k, lds_wave);
  else if constexpr (I == NX + 2)
    copy16_to_lds_at<0>(Wwave, ioff, lds_idx);
}

// Per-lane byte offsets, relative to the tile's first row, of the NX X blocks a wavefront copies per K step: lane l fetches row
// 8j + l/8 of block j, chunk (l%8) ^ ((row >> 1) & 7).  The X slab is stored row-major with the 16-byte chunk c of row r at
// chunk position c ^ ((r >> 1) & 7), so that the 16 rows a quarter-wavefront reads at the same K offset fall in 16 different
// 16-byte bank groups; the swizzle is applied by choosing which global chunk each lane fetches.  Rows past the end of X, and
// rows past the end of the tile (`rows` = its height), re-read the last row they may: their results are never stored, and a
// tile then draws no rows from memory that it does not use (the number of copies stays the same, the waits count them).
template <int NX>
__device__ __forceinline__ void tile_x_offsets(uint32_t (&xoff)[NX], int64_t m0, int M, int rows, int64_t k_bytes, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    const int r = 8 * (wave + i * 8) + (lane >> 3);
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    int64_t last = (int64_t)M - 1 - m0;  // >= 0: a tile starts inside X
    last = last < rows - 1 ? last : rows - 1;
    const int64_t rr = r < last ? r : last;
    xoff[i] = (uint32_t)(rr * k_bytes + c * 16);
  }
}

// The 16-byte chunk of a K step that a lane fetches in tile_x_offsets, the same in each of its NX blocks.
__device__ __forceinline__ int tile_x_chunk(int wave, int lane) { return (lane & 7) ^ ((4 * wave + (lane >> 4)) & 7); }

// The same for the patch-embedding mode with P = 16 (see patch_chunk_offset).
template <bool IS_I8, int NX>
__device__ __forceinline__ void patch_x_offsets(uint32_t (&xoff)[NX], int64_t m0, const GemmArgs& a, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    const int r = 8 * (wave + i * 8) + (lane >> 3);
    const int ch = (lane & 7) ^ ((r >> 1) & 7);  // logical chunk of the step this lane fetches (see tile_x_offsets)
    const uint32_t m = (uint32_t)m0 + (uint32_t)r;
    xoff[i] = patch_chunk_offset<IS_I8>(a, m < (uint32_t)a.M ? m : (uint32_t)a.M - 1u, ch);  // rows past the end re-read the last row
  }
}

// Per-lane byte offsets of the B operand inside an X slab: lane l reads row row0 + 16*mt + l%16 (row0: the wavefront's first), the
// 16-byte chunks l/16 and 4 + l/16 of it (at their swizzled positions).
struct BOffsets {
  uint32_t lo, hi;
};
__device__ __forceinline__ BOffsets b_offsets(int row0, int lane) {
  const int sw = (lane & 15) >> 1, q = lane >> 4;
  const uint32_t row = (uint32_t)(row0 + (lane & 15)) * kStepBytes;
  return BOffsets{row + (uint32_t)((q ^ sw) * 16), row + (uint32_t)(((4 + q) ^ sw) * 16)};
}

// Index words of fragments 4*half .. 4*half+3 of this lane, as they lie in LDS: int8 one word per fragment, fp16 two fragments
// per word (smfmac_of picks the half: no unpacking, which would wait for the read right behind it).
template <bool IS_I8>
struct IndexWords {
  static constexpr int kPerHalf = IS_I8 ? 4 : 2;
  int w[2 * kPerHalf];
  __device__ __forceinline__ void load(int half, const uint8_t* ibase) {
    if constexpr (IS_I8) {
      const v4i x = *(const v4i*)(ibase + half * 16);
#pragma unroll
      for (int j = 0; j < 4; ++j) w[4 * half + j] = x[j];
    } else {
      typedef int v2i __attribute__((ext_vector_type(2)));
      const v2i x = *(const v2i*)(ibase + half * 8);
      w[2 * half] = x[0];
      w[2 * half + 1] = x[1];
    }
  }
};
template <bool IS_I8>
__device__ __forceinline__ typename AccT<IS_I8>::type smfmac_of(int f, v4i a, v8i b, typename AccT<IS_I8>::type c, const IndexWords<IS_I8>& ix) {
  if constexpr (IS_I8)
    return smfmac<true>(a, b, c, ix.w[f]);
  else
    return (f & 1) ? smfmac<false, 1>(a, b, c, ix.w[f >> 1]) : smfmac<false, 0>(a, b, c, ix.w[f >> 1]);
}

__device__ __forceinline__ void read_b_half(v8i& b, int half, const uint8_t* p) {
  const v4i piece = *(const v4i*)p;
#pragma unroll
  for (int j = 0; j < 4; ++j) b[4 * half + j] = piece[j];
}

// What a wavefront holds in registers when a K step begins: its A fragments 0..3 with their index words and all B slabs but
// the last (which the step reads first); read from the stage whose X slab is at `xslab` and whose weight tile is at `wtile`.
template <bool IS_I8, int NX, int TMA>
__device__ __forceinline__ void load_step_head(v8i (&b)[NX], v4i (&av)[kTileTN], IndexWords<IS_I8>& ix, const uint8_t* xslab,
                                               const uint8_t* wtile, const BOffsets& bo, uint32_t a_off, uint32_t i_off) {
#pragma unroll
  for (int f = 0; f < 4; ++f) av[f] = *(const v4i*)(wtile + a_off + f * kFragValueBytes);
  ix.load(0, wtile + i_off);
#pragma unroll
  for (int mt = 0; mt + 1 < TMA; ++mt) {
    read_b_half(b[mt], 0, xslab + bo.lo + mt * 16 * kStepBytes);
    read_b_half(b[mt], 1, xslab + bo.hi + mt * 16 * kStepBytes);
  }
}

// One K step of a wavefront (128 n x 16 TMA m), software-pipelined by hand across steps.
// The matrix instructions go in two halves, A fragments 0..3 against the B slabs in turn, then fragments 4..7 against them.
// In that order an operand is needed at an even pace (one B slab or one A fragment every fourth instruction) and its
// registers fall free early enough to be refilled in place at least 12 instructions before their next use:
//   first half : reads the last B slab, A fragments 4..7 and their index words, the rest of this step's stage;
//   barrier    : in front of the last two instructions of the first half.  By then the reads of the stage have come back and
//                the wavefront's own copies of the next step have landed;
//   second half: reads the next step's A fragments 0..3, index words and, each as soon as its last instruction here is issued,
//                its B slabs; requests the copies of the step that follows in this stage, which has just fallen free.
// The LDS reads are so spread over the whole step (19 in 32 instructions), and beside spread reads and copies the matrix pipe
// runs on (1100 clocks for the 64 instructions of a SIMD's two wavefronts in a probe).  Reading the head of the next step in one
// burst behind a barrier late in the step left the LDS idle before it and the matrix pipe idle behind it.
// Measured: a full step of 256 x 256 x 128 bytes takes 1570 clocks, 250 of them by the copies and 120 by the barrier, at 1.55
// GHz (the board's power limit; 2.2 GHz on all-zero operands).
// The step has no conditional parts but the wait: the last step of a tile reads ahead like any other (the next tile reloads
// those registers) and the steps at the end of a workgroup's sequence request copies like any other (the cursor then stays on
// the last step: they land in a free stage and are never read).
// behind_stores: the awaited copies are older than the previous tile's output stores, of which STORES may stay in flight too.
// drain: nothing may stay in flight.
// landed(): called once, when the wavefront's own copies of the next step have landed, in front of the barrier;
// behind_barrier(): called once, right behind the barrier and before the step's copy requests.
template <bool IS_I8, int NX, int TMA, int STORES, class Landed, class Hook>
__device__ __forceinline__ void tile_step(bool behind_stores, bool drain, const uint8_t* stage, const uint8_t* next, const BOffsets& bo,
                                          typename AccT<IS_I8>::type (&acc)[kTileTN][NX], v8i (&b)[NX], v4i (&av)[kTileTN],
                                          IndexWords<IS_I8>& ix, uint32_t a_off, uint32_t i_off, uint32_t req_lds_wave,
                                          uint32_t req_lds_idx, const uint8_t* req_x, const uint8_t* req_w, const uint32_t (&xoff)[NX],
                                          uint32_t loff, uint32_t loff8k, uint32_t ioff, Landed&& landed, Hook&& behind_barrier) {
  typedef Ring<IS_I8, NX> R;
  const uint8_t* abase = stage + R::kXSlab + a_off;
  const uint8_t* ibase = stage + R::kXSlab + i_off;
  const uint8_t* abase_n = next + R::kXSlab + a_off;
  const uint8_t* ibase_n = next + R::kXSlab + i_off;
  constexpr int H = 4 * TMA;  // matrix instructions per half
  constexpr int kBarrierSlot = TMA > 2 ? H - 2 : H;
  constexpr int kBehind = (R::kStages - 2) * R::kCopies;  // copies of later steps than the awaited one
  auto read_b = [&](const uint8_t* st, int mt, int half) { read_b_half(b[mt], half, st + (half ? bo.hi : bo.lo) + mt * 16 * kStepBytes); };
#pragma unroll
  for (int slot = 0; slot < 2 * H; ++slot) {
    const int mt = (slot % H) >> 2, f = (slot & 3) + (slot < H ? 0 : 4);
    if (slot == kBarrierSlot) {
      __builtin_amdgcn_sched_barrier(0);  // the compiler must not move the wait above the matrix instructions before it
      if (behind_stores)
        wait_vm<kBehind + STORES>();
      else if (R::kStages > 3 && drain)
        wait_vm<0>();
      else
        wait_vm<kBehind>();
      landed();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");  // no LDS read moves above the barrier
      behind_barrier();
    }
    if (slot < H) {
      // the rest of this stage, in the first 7 slots (a 4- or 8-instruction half: as early as it goes)
      auto at = [&](int i) { return slot == (H >= 12 ? i : i * (H / 4) / 4); };
      if (at(0)) read_b(stage, TMA - 1, 0);
      if (at(1)) read_b(stage, TMA - 1, 1);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (at(2 + j)) av[4 + j] = *(const v4i*)(abase + (4 + j) * kFragValueBytes);
      if (at(6)) ix.load(1, ibase);
    } else {
      const int s = slot - H;
      if (s < 4) av[s] = *(const v4i*)(abase_n + s * kFragValueBytes);
      if (s == (H > 6 ? 6 : 3)) ix.load(0, ibase_n);
      // slab mt is free once its four instructions of this half are issued
      if (s >= 4 && (s & 3) < 2 && (s >> 2) - 1 < TMA - 1) read_b(next, (s >> 2) - 1, s & 1);
      auto request = [&](auto c) {  // copy c goes out in slot c * H / kCopies of this half
        constexpr int C = decltype(c)::value;
        if constexpr (C < R::kCopies) {
          if (s == C * H / R::kCopies) issue_step_copy<IS_I8, NX, C>(req_lds_wave, req_lds_idx, req_x, req_w, xoff, loff, loff8k, ioff);
        }
      };
      request(std::integral_constant<int, 0>{});
      request(std::integral_constant<int, 1>{});
      request(std::integral_constant<int, 2>{});
      request(std::integral_constant<int, 3>{});
      request(std::integral_constant<int, 4>{});
      request(std::integral_constant<int, 5>{});
      request(std::integral_constant<int, 6>{});
    }
    __builtin_amdgcn_sched_barrier(0);
    acc[f][mt] = smfmac_of<IS_I8>(f, av[f], b[mt], acc[f][mt], ix);
  }
  __builtin_amdgcn_sched_barrier(0);
}

// NX: see above.  PATCH: the X operand is gathered from an image batch (patch embedding with P = 16, see patch_chunk_offset).
// RAGGED: K is no whole number of steps (a variant of its own: the tail's length in a scalar register more, the kernel spills 4-20
// scalar values more across the K loop).
template <bool IS_I8, int GELU, int OUT, int NX, bool PATCH = false, bool RAGGED = false>
__global__ void __launch_bounds__(512, 1) spgemm_tile_kernel(const GemmArgs a, const EvenPlan plan) {
  typedef typename AccT<IS_I8>::type acc_t;
  typedef Ring<IS_I8, NX> R;
  constexpr int ES = IS_I8 ? 1 : 2;
  constexpr bool RAW = IS_I8 && OUT == GPUSQ_I32;
  // Store instructions per slab of a wavefront whose 128 channels lie inside Y, and how many of the previous tile's a wait may
  // leave in flight: the fewest a wavefront issues for a tile inside Y (a count too high would let copies go unwaited).
  constexpr int kStoresPerSlab = is_f16_out(OUT) ? 4 : (OUT == GPUSQ_I8 ? 2 : 8);
  constexpr int kStores = kStoresPerSlab * (NX > 1 ? NX - 1 : 1);
  __shared__ __attribute__((aligned(1024))) uint8_t ring[R::kStages * R::kStage];
  // per tile parity and 128-channel half: 128 weight scales, 128 biases
  __shared__ __attribute__((aligned(1024))) float prm[2][2][256];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wn = wave & 1, wm = wave >> 1;
  const int64_t k_bytes = (int64_t)a.K * ES;
  const int ksteps = (int)((k_bytes + kStepBytes - 1) / kStepBytes);
  const int tail_bytes = RAGGED ? (int)(k_bytes % kStepBytes) : 0;  // of a row in its last step
  const uint8_t* Xg = (const uint8_t*)a.X;
  const uint8_t* Wg = (const uint8_t*)a.W;
  const int64_t w_col_bytes = (int64_t)ksteps * tile_bytes(IS_I8);
  // All the arguments the kernel needs, asked of memory at once: left to the compiler they come in five groups, each waited for
  // before the next, and each a miss.
  asm volatile("" ::"s"(a.X), "s"(a.W), "s"(a.w_scale), "s"(a.act_scale), "s"(a.bias), "s"(a.Y), "s"(a.M), "s"(a.N), "s"(a.K), "s"(a.epilogue),
               "s"(plan.tiles_n), "s"(plan.chunks), "s"(plan.units), "s"(plan.higher), "s"(plan.tail_units), "s"(plan.inv), "s"(plan.shift),
               "s"(plan.rounds), "s"(plan.last_round), "s"(plan.grid8));
  const int place = (int)(blockIdx.x & 7) * plan.grid8 + (int)(blockIdx.x >> 3);  // in every round
  const int my_items = plan.rounds + (place < plan.last_round ? 1 : 0);
  if (my_items == 0) return;  // the whole workgroup leaves before any barrier
  auto tile_of = [&](int i) { return even_tile(plan, i * 8 * plan.grid8 + place); };
  const bool has_bias = !RAW && (a.epilogue & GPUSQ_EPI_BIAS) != 0;
  const float s_a = (IS_I8 && !RAW) ? a.act_scale[0] : 1.0f;
  const float s_out = OUT == GPUSQ_I8 || OUT == kOutF16Codes ? a.out_scale[0] : 1.0f, r_out = scale_reciprocal(s_out);  // read once: a load in the epilogue would wait for the copies in flight
  if (!has_bias && wm == 0) {  // the bias halves stay zero for the whole launch (visible after the first barrier)
#pragma unroll
    for (int par = 0; par < 2; ++par) {
      prm[par][wn][128 + lane] = 0.0f;
      prm[par][wn][192 + lane] = 0.0f;
    }
  }
  const uint32_t ring_lds = lds_address(ring), prm_lds = lds_address(prm[0][wn]);
  // The 128 channels [n0, n0 + 128) of epilogue constants of this wavefront's half of a tile, into the constants array
  // of the given parity; requested by the first wavefront of the half.  n0 < 0: nothing (there is no such tile).
  auto request_constants = [&](int n0, int parity) {
    if constexpr (!RAW) {
      if (wm == 0 && n0 >= 0) {
        const uint32_t dst = prm_lds + (uint32_t)parity * (uint32_t)sizeof(prm[0]);
        int lane_now = lane;
        asm volatile("" : "+v"(lane_now));  // computed here, per tile: nothing lane-dependent is carried (or spilled) across the K loop
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          int n = n0 + i * 64 + lane_now;
          n = n < a.N ? n : a.N - 1;  // channels past the end are never stored
          if constexpr (IS_I8) copy4_to_lds(a.w_scale, (uint32_t)n * 4u, dst + (uint32_t)i * 256u);
          if (has_bias) copy4_to_lds(a.bias, (uint32_t)n * 4u, dst + 512u + (uint32_t)i * 256u);
        }
      }
    }
  };
  const uint32_t loff = (uint32_t)lane * 16u;
  const uint32_t a_off = (uint32_t)(wn * kTileTN * kFragValueBytes + lane * 16);
  const uint32_t i_off = (uint32_t)index_offset(IS_I8, wn * kTileTN, lane);

  // lane offsets of the copies of kept values and index words, relative to the packed tile of a K step + wave * 1024
  const uint32_t loff8k = loff + 8192u;
  const int idx_block = IS_I8 ? (wave & 3) : (wave & 1);  // the 1 KB of index words this wavefront copies
  const uint32_t ioff = loff + (uint32_t)(kTileValueBytes + idx_block * 1024 - wave * 1024);
  const uint32_t wave_lds = (uint32_t)wave * 1024u, idx_lds = (uint32_t)(R::kXSlab + kTileValueBytes + idx_block * 1024);

  // Cursor of the copy requests: the next K step to request, as (tile, step), with its source addresses (pf_w includes
  // wave * 1024).  At the end of the workgroup's sequence it stays on the last step: the requests go on (the waits
  // count a fixed number of copies per step) and re-fetch that step into a stage that nothing reads any more.
  int pf_item = 0, pf_ks = 0;
  const uint8_t *pf_x = Xg, *pf_w = Wg;
  uint32_t pf_xoff[NX];
  // The cursor has come to a tile's last step: a chunk past the end of a ragged row re-reads the step's first.
  auto clip_tail = [&]() {
    if (RAGGED && pf_ks + 1 == ksteps) {  // uniform
      int lane_now = lane;
      asm volatile("" : "+v"(lane_now));
      const int at = tile_x_chunk(wave, lane_now) * 16;
      const uint32_t back = at >= tail_bytes ? (uint32_t)at : 0u;
#pragma unroll
      for (int i = 0; i < NX; ++i) pf_xoff[i] -= back;
    }
  };
  // fp16: those chunks of the stage at byte offset `stage_off` become zeros, before the barrier that publishes the stage.
  auto zero_tail = [&](int stage_off) {
    int lane_now = lane;
    asm volatile("" : "+v"(lane_now));
    if (tile_x_chunk(wave, lane_now) * 16 >= tail_bytes) {
#pragma unroll
      for (int i = 0; i < NX; ++i) *(v4i*)(ring + stage_off + wave * 1024 + i * 8192 + lane_now * 16) = v4i{0, 0, 0, 0};
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): written
  };
  auto seek = [&](int item) {
    pf_item = item;
    pf_ks = 0;
    const EvenTile t = tile_of(item);
    int lane_now = lane;
    asm volatile("" : "+v"(lane_now));  // (computed here, per tile)
    if constexpr (PATCH) {
      patch_x_offsets<IS_I8>(pf_xoff, t.m0, a, wave, lane_now);
      pf_x = Xg;
    } else {
      tile_x_offsets(pf_xoff, t.m0, a.M, 16 * t.slabs, k_bytes, wave, lane_now);
      pf_x = Xg + t.m0 * k_bytes;
      clip_tail();
    }
    pf_w = Wg + t.n_blk * w_col_bytes + wave_lds;
  };
  auto advance = [&]() {
    if (pf_ks + 1 < ksteps) {
      ++pf_ks;
      if constexpr (PATCH)
        pf_x = Xg + patch_step_offset<IS_I8>(a, pf_ks);
      else
        pf_x += kStepBytes;
      clip_tail();
      pf_w += tile_bytes(IS_I8);
    } else if (pf_item + 1 < my_items) {
      seek(pf_item + 1);
    }
  };
  auto request_step = [&](uint32_t stage_lds) {
    auto request = [&](auto c) {
      if constexpr (decltype(c)::value < R::kCopies)
        issue_step_copy<IS_I8, NX, decltype(c)::value>(stage_lds + wave_lds, stage_lds + idx_lds, pf_x, pf_w, pf_xoff, loff, loff8k, ioff);
    };
    request(std::integral_constant<int, 0>{});
    request(std::integral_constant<int, 1>{});
    request(std::integral_constant<int, 2>{});
    request(std::integral_constant<int, 3>{});
    request(std::integral_constant<int, 4>{});
    request(std::integral_constant<int, 5>{});
    request(std::integral_constant<int, 6>{});
  };

  acc_t acc[kTileTN][NX];
  v8i b[NX];             // B slabs
  v4i av[kTileTN];       // A fragments
  IndexWords<IS_I8> ix;  // and their index words

  // the constants of the first tile, then the first K steps of the sequence
  request_constants(tile_of(0).n_blk * kTileBN + wn * (kTileTN * 16), 0);
  seek(0);
#pragma nounroll
  for (int g = 0; g < R::kStages; ++g) {
    request_step(ring_lds + (uint32_t)g * R::kStage);
    advance();
  }
  wait_vm<(R::kStages - 1) * R::kCopies>();  // the constants and step 0 have landed
  if constexpr (RAGGED && !IS_I8) {
    if (ksteps == 1) zero_tail(0);
  }
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  int slot_off = 0;            // byte offset of the current K step's ring stage
  bool stores_behind = false;  // kStores output stores of the previous tile, or more, lie behind the copies a tile's first steps wait for
#pragma nounroll
  for (int item = 0; item < my_items; ++item) {
    const EvenTile t = tile_of(item);
    // this wavefront's slabs: a quarter of the tile's, the first t.slabs % 4 (0 or 2) wavefronts along m one more
    const int q = t.slabs >> 2, extra = t.slabs & 3;
    const int mine = q + (wm < extra ? 1 : 0), row0 = 16 * (wm * q + (wm < extra ? wm : extra));
    int lane_now = lane;
    asm volatile("" : "+v"(lane_now));  // the offsets are computed here, per tile, not once per kernel and kept (or spilled)
    const BOffsets bo = b_offsets(row0, lane_now);
    const int next_n0 = item + 1 < my_items ? tile_of(item + 1).n_blk * kTileBN + wn * (kTileTN * 16) : -1;
#pragma unroll
    for (int i = 0; i < kTileTN; ++i)
#pragma unroll
      for (int j = 0; j < NX; ++j) acc[i][j] = acc_t{0, 0, 0, 0};
    // A wavefront runs a K loop with the matrix instructions of its own slabs, NX or one less; the copies and the barriers are
    // the same.
    auto k_loop = [&](auto tma) {
      constexpr int TMA = decltype(tma)::value;
      // the stage of the tile's first step has landed: start-up barrier, or the barrier in the previous tile's last step
      load_step_head<IS_I8, NX, TMA>(b, av, ix, ring + slot_off, ring + slot_off + R::kXSlab, bo, a_off, i_off);
#pragma nounroll
      for (int ks = 0; ks < ksteps; ++ks) {
        const int next_off = slot_off + R::kStage == R::kStages * R::kStage ? 0 : slot_off + R::kStage;
        // Outstanding at the barrier of step g, oldest first: the copies of step g+1, then those of the kStages - 2 steps
        // behind it, which may stay in flight.  In the first kStages - 1 steps of a tile the output stores of the previous
        // tile's epilogue sit in the queue behind the copies waited for, so they may stay in flight too: the stores drain to
        // memory while the K loop goes on.  (Only where all of a wavefront's outputs lay inside Y; otherwise the wait covers
        // the stores as well, which is only stricter.)  With fewer steps to a tile than stages the constants requested in the
        // previous tile's last step would not be covered by any of the tile's waits if more than 3 stages' worth of copies may
        // stay in flight: those launches wait for everything.
        tile_step<IS_I8, NX, TMA, kStores>(stores_behind && ks < R::kStages - 1, ksteps < R::kStages, ring + slot_off, ring + next_off, bo, acc, b, av, ix,
                                           a_off, i_off, ring_lds + (uint32_t)slot_off + wave_lds, ring_lds + (uint32_t)slot_off + idx_lds,
                                           pf_x, pf_w, pf_xoff, loff, loff8k, ioff, [&]() {
                           // (the next step is a tile's last)
                           if constexpr (RAGGED && !IS_I8) {
                             if (ks + 2 == ksteps || ksteps == 1) zero_tail(next_off);
                           }
                         }, [&]() {
                           // The next tile's constants go into the other constants array, which was last read in the
                           // previous tile's epilogue (every wavefront has left it: it passed this tile's barriers).
                           // They are older than this step's copy requests, which the next tile's barriers wait for
                           // before its epilogue.
                           if (ks + 1 == ksteps) request_constants(next_n0, (item + 1) & 1);
                         });
        advance();
        slot_off = next_off;
      }
    };
    if constexpr (NX > 1) {
      if (mine == NX)
        k_loop(std::integral_constant<int, NX>{});
      else
        k_loop(std::integral_constant<int, NX - 1>{});
    } else {
      k_loop(std::integral_constant<int, 1>{});
    }
    const int n_wave = t.n_blk * kTileBN + wn * (kTileTN * 16);
    const int64_t m_wave = t.m0 + row0;
    const int64_t rows = (int64_t)a.M - m_wave;
    const int chans = a.N - n_wave;
    const bool lines = OUT == GPUSQ_F16 ? (a.N & 7) == 0 : (OUT == GPUSQ_I8 || OUT == kOutF16Codes ? (a.N & 15) == 0 : true);
    const bool inside = lines && rows >= mine * 16 && chans >= kTileTN * 16;
    const float* p = prm[item & 1][wn];
    // int8 output: one copy of the code for both heights (it is 40 KB with its exact quotients, and the wavefronts of a CU that run
    // NX and NX - 1 slabs would evict each other's from the instruction cache: 12608 x 768 -> 3072 34.5 us against 32.6)
    if (inside && (OUT == GPUSQ_I8 || mine == NX))
      line_epilogue<IS_I8, GELU, OUT, false, NX, NX>(a, acc, p, s_a, s_out, r_out, n_wave, m_wave, lane, OUT == GPUSQ_I8 ? mine : NX);
    else if (OUT != GPUSQ_I8 && inside && NX > 1)
      line_epilogue<IS_I8, GELU, OUT, false, NX, (NX > 1 && OUT != GPUSQ_I8 ? NX - 1 : 1)>(a, acc, p, s_a, s_out, r_out, n_wave, m_wave, lane, NX - 1);
    else if (lines)
      line_epilogue<IS_I8, GELU, OUT, true, NX, NX>(a, acc, p, s_a, s_out, r_out, n_wave, m_wave, lane, mine);
    else
      batch_epilogue<IS_I8, GELU, OUT, NX>(a, acc, p, s_a, OutScale{s_out, r_out}, n_wave, m_wave, lane, mine);
    stores_behind = inside && mine > 0 && ksteps >= R::kStages;
  }
  wait_vm<0>();  // the copies requested past the end of the sequence land before the LDS is given up
}

template <bool IS_I8, bool RAGGED, int NX>
static gpusq_status launch_tile1_nx(const GemmArgs& a, const EvenPlan& plan, unsigned grid, hipStream_t s) {
  const bool gelu = (a.epilogue & GPUSQ_EPI_GELU) != 0;
  if (a.patch_P != 0) {  // (a row is whole steps)
    if constexpr (!RAGGED) spgemm_tile_kernel<IS_I8, 0, GPUSQ_F16, NX, true><<<grid, 512, 0, s>>>(a, plan);
  } else if constexpr (IS_I8) {
    if (a.codes_out != nullptr)
      spgemm_tile_kernel<true, 0, kOutF16Codes, NX, false, RAGGED><<<grid, 512, 0, s>>>(a, plan);
    else if (a.out_dt == GPUSQ_I32)
      spgemm_tile_kernel<true, 0, GPUSQ_I32, NX, false, RAGGED><<<grid, 512, 0, s>>>(a, plan);
    else if (a.out_dt == GPUSQ_I8 && gelu)
      spgemm_tile_kernel<true, 1, GPUSQ_I8, NX, false, RAGGED><<<grid, 512, 0, s>>>(a, plan);
    else if (a.out_dt == GPUSQ_I8)
      spgemm_tile_kernel<true, 0, GPUSQ_I8, NX, false, RAGGED><<<grid, 512, 0, s>>>(a, plan);
    else if (gelu)
      spgemm_tile_kernel<true, 1, GPUSQ_F16, NX, false, RAGGED><<<grid, 512, 0, s>>>(a, plan);
    else
      spgemm_tile_kernel<true, 0, GPUSQ_F16, NX, false, RAGGED><<<grid, 512, 0, s>>>(a, plan);
  } else {
    if (gelu)
      spgemm_tile_kernel<false, 1, GPUSQ_F16, NX, false, RAGGED><<<grid, 512, 0, s>>>(a, plan);
    else
      spgemm_tile_kernel<false, 0, GPUSQ_F16, NX, false, RAGGED><<<grid, 512, 0, s>>>(a, plan);
  }
  return check_launch();
}

template <bool IS_I8, bool RAGGED>
static gpusq_status launch_tile1_typed(const GemmArgs& a, const EvenPlan& plan, unsigned grid, hipStream_t s) {
  switch ((even_units(plan) + 1) / 2) {
    case 1: return launch_tile1_nx<IS_I8, RAGGED, 1>(a, plan, grid, s);
    case 2: return launch_tile1_nx<IS_I8, RAGGED, 2>(a, plan, grid, s);
    case 3: return launch_tile1_nx<IS_I8, RAGGED, 3>(a, plan, grid, s);
    default: return launch_tile1_nx<IS_I8, RAGGED, 4>(a, plan, grid, s);
  }
}

}  // namespace gpusq
