// 2:4 structured-sparse GEMM with fused epilogue on the gfx950 sparse matrix instructions.
//
// Computes Y[m][n] = act( sum over the kept values of W[n][:] times the X[m][k] their metadata selects ) -- the
// sparse x dense -> dense product of Sec. 3.1 / Fig. 1, which equals the dense product on the zero-filled operand.
// The weights are the sparse "A" operand of v_smfmac_* (rows = output channels n), a 16 x 128-byte slab of
// activations is the dense "B" operand (columns = tokens m), so an accumulator tile is 16 n x 16 m and a lane owns
// 4 consecutive n of one m; with the packed row permutation (common.h) a lane owns 16 consecutive n per 64-row block.
//
// Register semantics of the instructions as measured on MI355X with one-hot operands (int8 16x16x128; fp16
// 16x16x64 is the same with "byte" read as "2-byte element pair"):
//   A (4 VGPRs): lane l, byte e -> row l%16, kept value e of the dense K range [32*(l/16), 32*(l/16)+32);
//   idx (1 VGPR): bits 2e..2e+1 of the lane's own register = position of kept value e inside its group of 4
//                 (fp16: 16 bits, the half selected by ABID);
//   B (8 VGPRs): lane l, byte i -> column l%16, K index 64*(i/16) + 16*(l/16) + i%16 (two half-K operands back to back);
//   D (4 VGPRs): lane l, register r -> row 4*(l/16)+r, column l%16.
//
// Here: spgemm_small_kernel (64 x 64 / 128 x 128 tiles through registers; any K % 16 == 0; used for small or ragged-K problems)
// and the choice between it, the kernel for few rows (fewrows.hip) and the two tile kernels (tile1.h, tile2.hip), which bring
// operands into an LDS ring by direct global->LDS copies (tile2.hip needs K * element size % 128 == 0).
#include <atomic>
#include <cstdlib>
#include <type_traits>

#include "tile_common.h"
#include "wide_plan.h"

namespace gpusq {

// XCD-aware tile order: consecutive workgroup ids land on different XCDs (8 of them, each with its own L2), so give
// every XCD one contiguous run of tiles; tiles that share an X slab (same m block) then share an L2.
__device__ __forceinline__ int xcd_tile(int tiles_total) {
  const int per_xcd = (tiles_total + 7) / 8;
  return (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
}

// Epilogue of one wavefront: TN fragments x TM column tiles of accumulators -> Y.
// Lane (q = lane/16, c = lane%16) holds, for 64-row block b and tile mt, the 16 channels
// n = n_wave + 64*b + 16*q + 4*t + r (t = fragment in block, r = register) of activation row m = m_wave + 16*mt + c.
// cs/bs: the workgroup's per-channel constants in LDS, indexed by channel - n_tile (see ChannelParams).
// GELU / OUT: compile-time epilogue choice, or -1 to read it from the arguments.
template <bool IS_I8, int TN, int TM, int GELU = -1, int OUT = -1>
__device__ __forceinline__ void wave_epilogue(const GemmArgs& a, const typename AccT<IS_I8>::type (&acc)[TN][TM],
                                              const float* cs, const float* bs, int n_tile, int n_wave, int64_t m_wave,
                                              int lane, const OutScale& os, int tm_active = TM) {
  const bool use_gelu = GELU >= 0 ? (GELU != 0) : ((a.epilogue & GPUSQ_EPI_GELU) != 0);
#pragma unroll
  for (int g = 0; g < TN / 2; ++g) {  // pairs of fragments = 32 channels; this lane holds 8 of them
    const int n = n_wave + (g >> 1) * kRowBlock + (g & 1) * 32 + (lane >> 4) * 8;
    float c8[8], b8[8];
#pragma unroll
    for (int j = 0; j < 8; j += 4) {
      const float4 cc = *(const float4*)(cs + (n - n_tile) + j), bb = *(const float4*)(bs + (n - n_tile) + j);
      c8[j] = cc.x; c8[j + 1] = cc.y; c8[j + 2] = cc.z; c8[j + 3] = cc.w;
      b8[j] = bb.x; b8[j + 1] = bb.y; b8[j + 2] = bb.z; b8[j + 3] = bb.w;
    }
#pragma unroll
    for (int mt = 0; mt < TM; ++mt) {
      if (mt >= tm_active) break;
      const int64_t m = m_wave + mt * 16 + (lane & 15);
      float v[8];
      int raw[8];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int j = 4 * t + r;
          if constexpr (IS_I8) {
            raw[j] = acc[2 * g + t][mt][r];
            v[j] = epilogue_value<true>(raw[j], 0.0f, c8[j], b8[j]);
          } else {
            raw[j] = 0;
            v[j] = epilogue_value<false>(0, acc[2 * g + t][mt][r], c8[j], b8[j]);
          }
        }
      if (use_gelu) gelu_f32_x8(v);
      if (m < a.M) store_8<IS_I8, OUT>(a, m, n, v, raw, os);
    }
  }
}

// ------------------------------------------------------------------------------------------------ small / generic kernel
constexpr int kLdsRow = kStepBytes + 16;  // 144-byte row pitch: 16 rows x 16-byte reads hit 16 distinct bank groups

// Workgroup = 4 wavefronts arranged WN (along n) x WM (along m); a wavefront owns TN x TM accumulator tiles.
// Workgroup tile: BN = WN*TN*16 output channels x BM = WM*TM*16 activation rows.  X goes global -> registers -> LDS
// (zero-filled past the row end, rows past M re-read the last row), and so do the weight fragments and index words of
// the tile, a 256th of them per thread.
// XF16 (INT8 path only): X is given in fp16 and quantised on its way through the registers, with the caller's static
// activation scale and the code rule of the activation quantiser; a chunk of 16 codes is then 32 bytes in memory.
template <bool IS_I8, int TN, int TM, int WN, int WM, bool XF16 = false>
__global__ void __launch_bounds__(256) spgemm_small_kernel(const GemmArgs a, const int tiles_n, const int tiles_total) {
  static_assert(WN * WM == 4 && TN % 4 == 0, "4 wavefronts; a wavefront spans whole 64-row blocks");
  static_assert(IS_I8 || !XF16, "the fp16 path takes fp16 X as it is");
  typedef typename AccT<IS_I8>::type acc_t;
  constexpr int BN = WN * TN * 16, BM = WM * TM * 16;
  constexpr int ES = IS_I8 ? 1 : 2;
  constexpr int XW = XF16 ? 2 : 1;  // bytes of X in memory per byte of the X operand
  constexpr int XCH = BM / 32;      // 16-byte chunks of the X slab each thread moves per K step

  constexpr int RBW = BN / kRowBlock;  // 64-channel row blocks of the workgroup's tile (= WN: a wavefront spans one)
  constexpr int kAStep = RBW * 4 * kFragValueBytes;  // kept values of the tile per K step; 1 KB of index words per row block behind them
  static_assert(RBW == WN && (RBW == 1 || RBW == 2), "the workgroup's fragments lie in one packed tile");
  __shared__ __attribute__((aligned(16))) uint8_t Xs[2][BM * kLdsRow];
  __shared__ __attribute__((aligned(16))) uint8_t As[2][kAStep + RBW * 1024];
  __shared__ __attribute__((aligned(16))) float cs[BN];
  __shared__ __attribute__((aligned(16))) float bs[BN];

  const int tile = xcd_tile(tiles_total);
  if (tile >= tiles_total) return;
  const int n_blk = tile % tiles_n, m_blk = tile / tiles_n;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wn = wave % WN, wm = wave / WN;
  const int M = a.M;
  if (tid < BN) {
    ChannelParams prm;
    prm.fetch<IS_I8>(a, n_blk * BN + tid);
    prm.publish(cs, bs, tid);  // made visible by the barriers of the main loop
  }
  const OutScale os = out_scale_of<IS_I8>(a);
  const int64_t k_bytes = (int64_t)a.K * ES;
  const int ksteps = (int)((k_bytes + kStepBytes - 1) / kStepBytes);
  const uint8_t* Xg = (const uint8_t*)a.X;
  const uint8_t* Wg = (const uint8_t*)a.W;

  acc_t acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = acc_t{0, 0, 0, 0};

  // Operands are requested D - 1 K steps ahead, each step into its own set of registers: at these sizes a K step is a
  // few matrix instructions, and what a step costs is the memory latency divided by the number of steps in flight.
  constexpr int D = TM == 1 ? (XF16 ? 4 : 6) : 3;  // (fp16 X in flight takes twice the registers per step)
  v4i xr[D][XCH][XW];
  v4i ar[D][RBW];  // this thread's 16-byte pieces of the tile's kept values (thread t: lane t % 64 of fragment t / 64 + 4j)
  v4i ir[D];       // threads below 64 * RBW: the index words of lane t % 64 for row block t / 64

  // Addresses: a wavefront-uniform base that advances by a constant per K step (scalar arithmetic) plus a 32-bit lane
  // offset fixed for the whole tile, so a K step issues its loads with next to no vector arithmetic: with one wavefront
  // per SIMD (a lone wavefront issues a vector instruction only every 6-8 clocks) address arithmetic per load is what a
  // step would otherwise cost.
  const global_u8* Xtile = uniform_ptr(Xg + (int64_t)m_blk * BM * k_bytes * XW);
  float s_x = 1.0f, r_x = 1.0f;
  if constexpr (XF16) {
    s_x = a.act_scale[0];
    r_x = scale_reciprocal(s_x);
  }
  // Rows past the end of X re-read the last row (their results are never stored), so only a K that is not a whole
  // number of steps needs a predicate, and only in the last step: a plain step is 7 loads and nothing else.
  uint32_t xoff[XCH];
  const int64_t last_row = (int64_t)M - 1 - (int64_t)m_blk * BM;  // >= 0: a tile starts inside X
#pragma unroll
  for (int j = 0; j < XCH; ++j) {
    const int c = tid + 256 * j;
    const int row = (c >> 3) < last_row ? (c >> 3) : (int)last_row;
    xoff[j] = ((uint32_t)row * (uint32_t)k_bytes + (c & 7) * 16) * XW;  // the host keeps 128 rows of X below 4 GiB
  }
  const int tail_bytes = (int)(k_bytes % kStepBytes);  // 0: K is a whole number of steps
  static_assert(TN == 4, "a wavefront's fragments are the four of one 64-channel row block");
  // The weights, like X, enter the CU once per workgroup and K step and reach the wavefronts through LDS: the
  // wavefronts along m need the same fragments, and fetched by each of them straight into registers they were what
  // bound a K step (4 x 5 KB + 8 KB of X per step is all a CU can draw from the L2).
  // (the packed buffer is padded to whole 256-channel tiles, so the tile's row blocks always exist)
  const int rbw = n_blk * RBW;
  const int f0 = (rbw & 3) * 4;
  const global_u8* Wrow = uniform_ptr(Wg + (int64_t)(rbw >> 2) * ksteps * tile_bytes(IS_I8));
  const uint32_t a_thr = (uint32_t)(f0 * kFragValueBytes + tid * 16);
  const bool idx_thr = tid < 64 * RBW;  // (whole wavefronts)
  // the index words of the 4 fragments of a row block are adjacent per lane: 16 bytes (int8) or 8 bytes (fp16)
  const uint32_t i_thr = (uint32_t)index_offset(IS_I8, f0 + 4 * ((tid >> 6) & (RBW - 1)), lane);
  auto load_x = [&](int ks, int slot) {
    const global_u8* base = Xtile + (int64_t)ks * (kStepBytes * XW);
    if (tail_bytes != 0 && ks + 1 == ksteps) {  // workgroup-uniform: the ragged last step zero-fills past the row end
#pragma unroll
      for (int j = 0; j < XCH; ++j)
#pragma unroll
        for (int h = 0; h < XW; ++h)
          xr[slot][j][h] = (int)(((tid + 256 * j) & 7) * 16) < tail_bytes
                               ? *(const __attribute__((address_space(1))) v4i*)(base + xoff[j] + 16 * h)
                               : v4i{0, 0, 0, 0};
    } else {
#pragma unroll
      for (int j = 0; j < XCH; ++j)
#pragma unroll
        for (int h = 0; h < XW; ++h) xr[slot][j][h] = *(const __attribute__((address_space(1))) v4i*)(base + xoff[j] + 16 * h);
    }
  };
  auto store_x = [&](int buf, int slot) {
#pragma unroll
    for (int j = 0; j < XCH; ++j) {
      const int c = tid + 256 * j;
      v4i codes;
      if constexpr (XF16) {
        // 16 fp16 values -> 16 int8 codes (zero-filled chunks give zero codes)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const ep_v8h x = __builtin_bit_cast(ep_v8h, xr[slot][j][h]);
          float v[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = (float)x[e];
          unsigned lo, hi;
          quantize_bytes8(v, s_x, r_x, lo, hi);
          codes[2 * h] = (int)lo;
          codes[2 * h + 1] = (int)hi;
        }
      } else {
        codes = xr[slot][j][0];
      }
      *(v4i*)(&Xs[buf][(c >> 3) * kLdsRow + (c & 7) * 16]) = codes;
    }
  };
  auto load_a = [&](int ks, int slot) {
    const global_u8* t = Wrow + (int64_t)ks * tile_bytes(IS_I8);
#pragma unroll
    for (int j = 0; j < RBW; ++j)
      ar[slot][j] = *(const __attribute__((address_space(1))) v4i*)(t + a_thr + j * (4 * kFragValueBytes));
    if (idx_thr) {
      if constexpr (IS_I8) {
        ir[slot] = *(const __attribute__((address_space(1))) v4i*)(t + i_thr);
      } else {
        const ep_v2u w = *(const __attribute__((address_space(1))) ep_v2u*)(t + i_thr);
        ir[slot] = v4i{(int)w[0], (int)w[1], 0, 0};
      }
    }
  };
  auto store_a = [&](int buf, int slot) {
#pragma unroll
    for (int j = 0; j < RBW; ++j) *(v4i*)(&As[buf][tid * 16 + j * (4 * kFragValueBytes)]) = ar[slot][j];
    if (idx_thr) *(v4i*)(&As[buf][kAStep + tid * 16]) = ir[slot];
  };

  // K steps q * D + r: q passes of D steps without any condition in them (the request D - 1 steps ahead is clamped to
  // the last step, whose data is then fetched again and not used), then the r < D remaining steps, whose operands the
  // last pass (or the preamble) has already requested, as straight-line code behind uniform forward branches.
  auto clamp_step = [&](int ks) { return ks < ksteps ? ks : ksteps - 1; };
#pragma unroll
  for (int d = 0; d < D - 1; ++d) {
    load_x(clamp_step(d), d);
    load_a(clamp_step(d), d);
  }
  const int b_row = wm * TM * 16 + (lane & 15);
  const int b_col = (lane >> 4) * 16;
  // The operands alternate between two LDS buffers, and the step is pipelined across them: step ks first writes the
  // operands of step ks + 1 into the other buffer (last read in step ks - 1, whose closing barrier every wavefront has
  // passed), then reads its own, multiplies, and closes with the barrier that publishes what it wrote.  So the LDS round
  // trip of a step's operands runs beside the previous step's reads and matrix instructions instead of in front of its
  // own.
  store_x(0, 0);
  store_a(0, 0);
  __syncthreads();
  auto compute_step = [&](int ks, int slot) {
    const int cur = ks & 1;
    if (ks + 1 < ksteps) {  // workgroup-uniform
      store_x(cur ^ 1, (slot + 1) % D);
      store_a(cur ^ 1, (slot + 1) % D);
    }
    v4i av[TN];
    int ai[TN];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) av[tn] = *(const v4i*)(&As[cur][(wn * TN + tn) * kFragValueBytes + lane * 16]);
    const v4i iw = *(const v4i*)(&As[cur][kAStep + wn * 1024 + lane * 16]);
    if constexpr (IS_I8) {
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) ai[tn] = iw[tn];
    } else {
      ai[0] = iw[0] & 0xFFFF;
      ai[1] = (int)((unsigned)iw[0] >> 16);
      ai[2] = iw[1] & 0xFFFF;
      ai[3] = (int)((unsigned)iw[1] >> 16);
    }
#pragma unroll
    for (int mt = 0; mt < TM; ++mt) {
      const uint8_t* p = &Xs[cur][(b_row + mt * 16) * kLdsRow + b_col];
      const v4i lo = *(const v4i*)p, hi = *(const v4i*)(p + 64);
      const v8i b = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) acc[tn][mt] = smfmac<IS_I8>(av[tn], b, acc[tn][mt], ai[tn]);
    }
    __syncthreads();
  };
  const int passes = ksteps / D, rest = ksteps - passes * D;
  int ks = 0;
  for (int pass = 0; pass < passes; ++pass) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      load_x(clamp_step(ks + D - 1), (j + D - 1) % D);
      load_a(clamp_step(ks + D - 1), (j + D - 1) % D);
      compute_step(ks, j);
      ++ks;
    }
  }
#pragma unroll
  for (int d = 0; d < D - 1; ++d)
    if (d < rest) compute_step(ks + d, d);  // workgroup-uniform
  __syncthreads();  // the per-channel constants written at the top are read below (also when K has no step at all)
  wave_epilogue<IS_I8, TN, TM>(a, acc, cs, bs, n_blk * BN, n_blk * BN + wn * TN * 16, (int64_t)m_blk * BM + wm * TM * 16, lane, os);
}

template <bool IS_I8, int TN, int TM, int WN, int WM>
static gpusq_status launch_small(const GemmArgs& a, hipStream_t s) {
  constexpr int BN = WN * TN * 16, BM = WM * TM * 16;
  const int tiles_n = (int)ceil_div(a.N, BN), tiles_m = (int)ceil_div(a.M, BM);
  const int total = tiles_n * tiles_m;
  const int grid = (int)ceil_div(total, 8) * 8;  // whole rounds over the 8 XCDs; surplus workgroups exit at once
  const int x_elem_bytes = (IS_I8 && !a.x_f16) ? 1 : 2;
  if ((int64_t)a.K * x_elem_bytes * BM >= ((int64_t)1 << 32)) return GPUSQ_ERR_UNSUPPORTED;  // 32-bit lane offsets inside a tile's rows of X
  if constexpr (IS_I8) {
    if (a.x_f16) {
      spgemm_small_kernel<true, TN, TM, WN, WM, true><<<grid, 256, 0, s>>>(a, tiles_n, total);
      return check_launch();
    }
  }
  spgemm_small_kernel<IS_I8, TN, TM, WN, WM><<<grid, 256, 0, s>>>(a, tiles_n, total);
  return check_launch();
}

// Compute units of the current device, read once per device (a racing first call reads the same value twice).
int num_cus() {
  constexpr int kMaxDevices = 64;
  static std::atomic<int> cus[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) dev = 0;
  int n = cus[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cus[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

// Testing aid: -1 = the size rules decide, 0 / 1 / 2 = run every problem the kernel can take on that kernel.  Set by
// gpusq_force_kernel(); the environment variable GPUSQ_FORCE_KERNEL gives the initial value and is read once, when the
// library is loaded, so that no launch pays for an environment lookup.
static int initial_forced_kernel() {
  const char* f = getenv("GPUSQ_FORCE_KERNEL");
  return (f && f[0] >= '0' && f[0] <= '6' && f[1] == 0) ? f[0] - '0' : -1;
}
static std::atomic<int> g_forced_kernel{initial_forced_kernel()};
int forced_kernel() { return g_forced_kernel.load(std::memory_order_relaxed); }
int set_forced_kernel(int kernel) {
  return g_forced_kernel.exchange(kernel >= 0 && kernel <= 6 ? kernel : -1);
}

// The estimate that decides which problems may quantise fp16 activations on their way into the small kernel (see kernel_choice), of
// the tile kernel in full and tail tiles of whole 64-row units: run time (microseconds) of one tile of 64*tm rows.  A K step costs nearly
// the same whatever tm (a short tile copies and reads whole operands and only leaves out the matrix instructions of the slabs it does not
// have: 1.1 us for tm = 4, about 0.075 us less per slab left out), the epilogue scales with the rows stored and is larger with GELU.
// `busy` is the fraction of the CUs that have a workgroup: the fewer run, the faster each one's K steps (the chip runs
// at its power limit when all of them multiply: 1.1 us per step on 256 CUs, 0.63 on 150, 0.46 on 100).
static double tile_cost(int tm, int ksteps, bool gelu, double busy) {
  double step = (0.8 + 0.075 * tm) * (0.1 + 0.9 * busy);
  if (step < 0.6) step = 0.6;  // (what a K step costs a lone workgroup: latency, not throughput)
  return ksteps * step + (gelu ? 1.6 : 1.1) * tm + 0.3;
}

// The workgroup with the most work under the kernel's assignment (XCD x takes its share of the list, its workgroup wl
// the items wl, wl + W, ...).
static double plan_makespan(const TilePlan& p, int grid, int ksteps, bool gelu, double busy) {
  const int W = grid / 8;
  const double cf = tile_cost(p.full_tm, ksteps, gelu, busy), ct = tile_cost(p.tail_tm, ksteps, gelu, busy);
  double worst = 0;
  for (int x = 0; x < 8; ++x) {
    int f0, nf, t0;
    const int items = xcd_items(p, x, f0, nf, t0);
    for (int wl = 0; wl < W && wl < items; ++wl) {
      const int mine = (items - wl + W - 1) / W;
      const int full = wl < nf ? (nf - wl + W - 1) / W : 0;
      const double c = full * cf + (mine - full) * ct;
      if (c > worst) worst = c;
    }
  }
  return worst;
}

static int grid_for(const TilePlan& p, int resident) { return (int)ceil_div(p.total < resident ? p.total : resident, 8) * 8; }

constexpr int kTileTM = 4;  // 64-row units of the highest tile

// The plan of that estimate (what runs is even_plan's).  Candidates: full tiles of 64, 128, 192 or 256
// rows, either over all of M, or for as many whole rounds over the resident
// workgroups as the problem has with the remaining rows in tail tiles of 64..64*full_tm rows; the one whose busiest
// workgroup finishes first wins.
static TilePlan make_plan(int M, int N, int resident, int ksteps, bool gelu) {
  TilePlan best{};
  double best_cost = -1;
  const int tiles_n = (int)ceil_div(N, kTileBN);
  auto consider = [&](int ftm, int full_chunks, int ttm) {
    TilePlan p;
    p.tiles_n = tiles_n;
    p.full_tm = ftm;
    p.full_chunks = full_chunks;
    p.full_tiles = full_chunks * tiles_n;
    p.tail_tm = ttm;
    const int64_t rows_left = (int64_t)M - (int64_t)full_chunks * 64 * ftm;
    p.total = p.full_tiles + (rows_left > 0 ? (int)ceil_div(rows_left, 64 * ttm) * tiles_n : 0);
    p.inv_tiles_n = (tiles_n > 1 && tiles_n <= 4096 && p.total < (1 << 20)) ? (uint32_t)((((uint64_t)1 << 32) + tiles_n - 1) / tiles_n) : 0u;
    const double c = plan_makespan(p, grid_for(p, resident), ksteps, gelu, 1.0);  // (plans are compared at the full-chip step cost)
    if (best_cost < 0 || c < best_cost) {
      best_cost = c;
      best = p;
    }
  };
  for (int ftm = kTileTM; ftm >= 1; --ftm) {
    const int chunks = (int)ceil_div(M, 64 * ftm);
    consider(ftm, chunks, ftm);
    const int all_tiles = chunks * tiles_n;
    if (all_tiles > resident && all_tiles % resident != 0) {
      const int full_chunks = (all_tiles / resident) * resident / tiles_n;
      for (int ttm = ftm; ttm >= 1; --ttm) consider(ftm, full_chunks, ttm);
    }
  }
  return best;
}

// Few rows: 4 (the kernel with K split over its wavefronts), 0 (the 64 x 64 tiles) or -1 (by the estimates), by how many of the
// former's 64-channel x 32-row tiles each CU gets.  Two of its workgroups run side by side on a CU (int8; fp16: three), and where
// K has few steps another round costs most of a launch.  Timed at 7 widths, which agree; 768 channels, few rows / 64 x 64 tiles /
// the faster tile kernel, us:
//   int8  2 tiles, K = 192: 4.0 / 4.4 / 4.0, 768: 4.9 / 5.4 / 6.7;  3 tiles, K = 192: 5.7 / 5.0 / 5.5, 640: 6.7 / 6.0 / 6.5, 768: 7.1 / 6.7 /
//         6.9, 1024: 7.2 / 7.2 / 7.7, 1536: 8.6 / 9.1 / 9.2;  3.5 tiles: behind or level at every K
//   fp16  3 tiles, K = 192: 4.3 / 4.9 / 5.6;  4 tiles, K = 128: 5.5 / 5.2 / 5.3, 256: 5.9 / 6.0 / 6.1 (on 512 channels 5.9 / 5.4 / 6.2), 384: 7.0
//         / 7.8 / 7.0;  5 tiles, K = 192: 6.4 / 5.8 / 5.9, 384: 7.6 / 8.0 / 7.1, 512: 7.7 / 8.7 / 8.0, 1536: 14.3 / 18.3 / 14.2;
//         6 tiles, K = 192: 6.9 / 6.0 / 6.1, 768: 10.4 / 11.5 / 9.4, 3072: 29.5 / 32.9 / 25.4
static int few_rows_choice(bool is_i8, int64_t M, int64_t N, int64_t ksteps, int resident) {
  const int64_t tiles = ceil_div(M, 32) * ceil_div(N, kRowBlock), r = resident;
  if (is_i8) return tiles <= (ksteps >= 8 ? 3 : 2) * r ? 4 : -1;
  if (ksteps <= 5) return tiles <= 3 * r ? 4 : (tiles <= 5 * r ? 0 : -1);
  return tiles <= (ksteps >= 8 ? 5 : 4) * r ? 4 : -1;
}
// Of the two small kernels: 64 x 64 tiles while these fit one round of two workgroups per CU, 128 x 128 beyond.
static int small_choice(int64_t M, int64_t N, int resident) { return ceil_div(M, 64) * ceil_div(N, 64) <= 2 * (int64_t)resident ? 0 : 1; }

// Whole 128-byte steps, more rows than the kernel for few of them takes: run times in microseconds, fitted to 1515 sizes timed on MI355X (M
// 600 ... 65792, N 64 ... 5120, K 64 ... 5120, both types, with and without GELU, fp16 and int8 output, three buffers in turn; kernel 2 to 6 %,
// kernel 0 to 8 %).  Kernel 2: the even plan's rounds r over the CUs with u units of 32 rows in each on the busiest CU; a K step is faster with
// fewer CUs at work (the board's power limit).  Kernel 0: rounds of 512 workgroups and the chain of one.
struct EvenRounds {
  double r, u, busy;
};
static EvenRounds even_rounds(const EvenPlan& p, int resident) {
  const int64_t total = even_total(p), r = ceil_div(total, resident);
  const int64_t most = r * p.units + ceil_div((int64_t)p.higher * p.tiles_n, resident);
  return EvenRounds{(double)r, (double)most / (double)r, total < resident ? (double)total / resident : 1.0};
}
static double estimate_kernel2(const EvenRounds& e, bool is_i8, bool gelu, int64_t ksteps) {
  const double step = 0.135 + 0.121 * e.u, epi = is_i8 ? (gelu ? 0.85 : 0.5) : (gelu ? 0.70 : 0.44);
  return 3.4 + e.r * (ksteps * (step > 0.42 ? step : 0.42) * (0.49 + 0.51 * e.busy) + 0.7 + epi * e.u);
}
static double estimate_kernel0(int64_t wgs64, int resident, bool is_i8, bool gelu, int64_t ksteps) {
  const double epi = is_i8 ? (gelu ? 2.05 : 1.65) : (gelu ? 1.85 : 1.5);
  return 2.6 + 0.19 * ksteps + (0.32 * ksteps + epi) * (double)wgs64 / (2.0 * resident);
}
// Of those sizes the estimates and the lines below pick a kernel 0.8 % behind the fastest on average, where the plan in units of 64 rows and
// a line by widths (kernel 3 for N <= 1536, K <= 1024, no GELU) were 3.6 % behind: 2096 x 2752 -> 1728 fp16 + GELU 38.4 -> 23.1 us, 12608 x 768 -> 768
// int8 13.4 -> 11.2, 12544 x 512 -> 512 8.6 -> 7.8, 61579 x 128 -> 128 11.7 -> 7.5.
// Kernel 3's 64- and 128-row tiles on two workgroups per CU are ahead at the heights that fit them, with few K steps: one round of 2 units,
// or of 8 while its own tiles are one round; two rounds of up to 5 (medians 2 to 9 % ahead; 12544 x 512 -> 1536 int8 output 15.7 / 14.1 us, 10216 x
// 384 -> 2048 14.5 / 12.6, 1790 x 192 -> 1792 fp16 6.4 / 5.8; int8 with GELU at 2 units 6 % behind).  Beyond 8 steps even or behind, at all other
// heights 2 to 20 % behind as a rule (of 300 sizes timed afterwards it was further ahead than 10 % at two: 21450 x 512 -> 1920 37.7 / 31.0, 20979 x 448 ->
// 3392 fp16 66.8 / 58.7; the choice 1.1 % behind the fastest there, 31 % at the most: 33970 x 512 -> 128 goes to kernel 0, 11.5, with kernel 2 at 8.8).
static bool kernel3_ahead(const EvenRounds& e, bool is_i8, bool gelu, int64_t M, int64_t N, int64_t ksteps, int resident) {
  const int64_t tiles = ceil_div(M, 128) * ceil_div(N, kTileBN);
  if (ksteps > 8) return false;
  if (e.r == 1) return (e.u > 1 && e.u <= 2 && !(is_i8 && gelu)) || (e.u > 7 && tiles < 2 * (int64_t)resident);
  return e.r == 2 && e.u <= 5;
}

// Which kernel a problem takes: 0 = small kernel with 64 x 64 tiles, 1 = small kernel with 128 x 128 tiles, 2 = tile
// kernel with one workgroup per CU, 3 = with two, 4 = the kernel for few rows.  fused_patches: the patch gather exists in kernels 2 and 4
// only.
static int kernel_choice(bool is_i8, int64_t M, int64_t N, int64_t K, bool gelu, int resident, bool fused_patches = false, bool x_f16 = false) {
  const int64_t k_bytes = K * (is_i8 ? 1 : 2);
  const int64_t ksteps = ceil_div(k_bytes, kStepBytes);
  const int64_t wgs64 = ceil_div(M, 64) * ceil_div(N, 64);
  // Testing aid: a forced kernel overrides the choice (2 only where the tile kernel can run the problem).
  if (const int c = g_forced_kernel.load(std::memory_order_relaxed); c >= 0 && c < 5) {
    if (c != 3 || k_bytes % kStepBytes == 0) return c;
  }
  // (the fused patch gather is refused up to 256 K outputs; beyond, it goes to the kernel for few rows where a GEMM of its sizes would, else
  // to kernel 2, whichever of 0, 2 and 3 the GEMM takes: those add up in one order)
  if (fused_patches && M * N <= (int64_t)256 * 1024) return 0;
  // (the patch gather has no 64 x 64 tiles)
  if (const int c = few_rows_choice(is_i8, M, N, ksteps, resident); c == 4 || (c == 0 && !fused_patches)) return c;
  if (M * N <= (int64_t)256 * 1024) return 0;
  const bool ragged = k_bytes % kStepBytes != 0;
  // A K of no whole number of 128-byte steps: the estimates are of the kernels for whole steps.  One round of 64 x 64 tiles, then, while
  // the steps are few, one of 128 x 128 tiles, then tile kernel 2, are each the fastest (of 180 sizes timed, 0.4 % behind the fastest of
  // the three on average; us, 64 x 64 / 128 x 128 / kernel 2: int8 3152 x 192 -> 576 5.1 / 6.2 / 6.0, 50432 x 192 -> 128 12.3 / 8.2 / 8.4, 25216 x
  // 592 -> 128 9.9 / 8.5 / 8.3; fp16 6304 x 208 -> 576 9.3 / 7.4 / 8.3, 12608 x 400 -> 192 8.8 / 8.8 / 7.9).
  // (beyond the 32-bit lane offsets of a tile of 256 rows; the small kernels' tiles have fewer)
  if (ragged && (k_bytes >= ((int64_t)1 << 24) || N >= ((int64_t)1 << 25))) return small_choice(M, N, resident);
  if (ragged) {
    if (wgs64 <= 2 * resident) return 0;
    return ksteps <= (is_i8 ? 2 : 4) && ceil_div(M, 128) * ceil_div(N, 128) <= 2 * (int64_t)resident ? 1 : 2;
  }
  if (fused_patches) return 2;
  if (x_f16 || 255 * k_bytes + kStepBytes >= ((int64_t)1 << 32)) {
    // Which problems the small kernel quantises fp16 activations for, and which it takes where K is beyond kernel 2's 32-bit lane offsets
    // (the others are refused there), was settled by an estimate of the tile kernel in units of 64 rows and is kept: a caller may have
    // built on it.
    if (wgs64 > 16 * resident) return 2;
    const double per_round = 0.7 + 0.45 * ksteps, chain = 3.6 + 0.25 * ksteps;
    const double throughput = 4.0 + per_round * (double)wgs64 / (2.0 * resident);
    const double est_small = chain > throughput ? chain : throughput;
    const TilePlan p = make_plan((int)M, (int)N, resident, (int)ksteps, gelu);
    const int grid = grid_for(p, resident);
    const double est_tile = plan_makespan(p, grid, (int)ksteps, gelu, (double)(p.total < grid ? p.total : grid) / resident) + 2.8;
    return est_small < est_tile ? 0 : 2;
  }
  const EvenRounds e = even_rounds(even_plan(M, N, resident, (int)ksteps, gelu), resident);
  if (wgs64 <= 16 * resident && estimate_kernel0(wgs64, resident, is_i8, gelu, ksteps) < estimate_kernel2(e, is_i8, gelu, ksteps)) return 0;
  return kernel3_ahead(e, is_i8, gelu, M, N, ksteps, resident) ? 3 : 2;
}

gpusq_status plan_spgemm(bool is_i8, int64_t M, int64_t N, int64_t K, int epilogue, int cus, int32_t* out) {
  const int resident = cus > 0 ? cus : num_cus();
  const int choice = kernel_choice(is_i8, M, N, K, (epilogue & GPUSQ_EPI_GELU) != 0, resident);
  for (int i = 0; i < 8; ++i) out[i] = 0;
  out[0] = choice == 4 ? 0 : choice;  // (both kernels for small problems are reported as 0)
  const int ksteps = (int)ceil_div(K * (is_i8 ? 1 : 2), kStepBytes);
  const bool gelu = (epilogue & GPUSQ_EPI_GELU) != 0;
  if (choice == 2) {  // main chunks of two heights, or of one and tail chunks
    const EvenPlan p = even_plan(M, N, resident, ksteps, gelu);
    out[1] = 32;
    out[2] = p.tiles_n;
    out[3] = even_units(p);
    out[4] = p.higher > 0 ? p.higher : p.chunks;
    out[5] = p.tail_chunks > 0 ? p.tail_units : p.units;
    out[6] = (int32_t)even_total(p);
    out[7] = 8 * p.grid8;
  } else if (choice == 3) {
    const TilePlan p = make_tile2_plan((int)M, (int)N, 2 * resident, ksteps, gelu, false);
    out[1] = 64;
    out[2] = p.tiles_n;
    out[3] = p.full_tm;
    out[4] = p.full_chunks;
    out[5] = p.tail_tm;
    out[6] = p.total;
    out[7] = tile2_grid_of(p, 2 * resident);
  }
  return GPUSQ_OK;
}

// The kernel choice and tile plan of a problem, remembered per thread for the last few distinct problems: a layer is
// launched over and over with the same sizes, and planning (a dozen candidate plans, each walked over every workgroup)
// takes the host several microseconds, which is what a launch of a 10 us GEMM is bound by when it is repeated.
struct Decision {
  double gemm_us;  // estimate of the product on what the choice picks (whole K steps; not for the kernel for few rows)
  bool is_i8, gelu, patches, x_f16;
  int forced;  // the forced kernel when the decision was taken, -1 for none
  int64_t M, N, K;
  int resident, choice;
  TilePlan plan;  // valid when choice == 3
  EvenPlan even;  // valid when choice == 2 or 3, and when it is 1 for a ragged K within kernel 2's limits
};
static const Decision& decide(bool is_i8, int64_t M, int64_t N, int64_t K, bool gelu, int resident, bool patches, bool x_f16 = false) {
  constexpr int kSlots = 16;
  thread_local Decision cache[kSlots];
  thread_local int used = 0, next = 0;
  int forced = g_forced_kernel.load(std::memory_order_relaxed);
  if (forced > 5) forced = -1;  // (another call's)
  for (int i = 0; i < used; ++i) {
    const Decision& d = cache[i];
    if (d.M == M && d.N == N && d.K == K && d.is_i8 == is_i8 && d.gelu == gelu && d.patches == patches && d.x_f16 == x_f16 &&
        d.forced == forced && d.resident == resident)
      return d;
  }
  Decision& d = cache[next];
  next = (next + 1) % kSlots;
  if (used < kSlots) ++used;
  d = Decision{0.0, is_i8, gelu, patches, x_f16, forced, M, N, K, resident, kernel_choice(is_i8, M, N, K, gelu, resident, patches, x_f16), TilePlan{}, EvenPlan{}};
  const int64_t k_bytes = K * (is_i8 ? 1 : 2);
  const bool limits = k_bytes < ((int64_t)1 << 24) && N < ((int64_t)1 << 25);  // (as in kernel_choice)
  if (d.choice == 2 || d.choice == 3 || (d.choice == 1 && limits)) d.even = even_plan(M, N, resident, (int)ceil_div(k_bytes, kStepBytes), gelu);
  if (is_i8 && d.choice != 4 && limits) {
    const int64_t ksteps = ceil_div(k_bytes, kStepBytes);
    const EvenPlan p = d.even.tiles_n > 0 ? d.even : even_plan(M, N, resident, (int)ksteps, gelu);
    const double k0 = estimate_kernel0(ceil_div(M, 64) * ceil_div(N, 64), resident, true, gelu, ksteps);
    const double k2 = estimate_kernel2(even_rounds(p, resident), true, gelu, ksteps);
    d.gemm_us = k0 < k2 ? k0 : k2;
  }
  if (d.choice == 3) d.plan = make_tile2_plan((int)M, (int)N, 2 * resident, (int)(k_bytes / kStepBytes), gelu, false);
  return d;
}

template <bool IS_I8>
static gpusq_status launch_typed(const GemmArgs& a, hipStream_t s) {
  const int64_t k_bytes = (int64_t)a.K * (IS_I8 ? 1 : 2);
  const bool gelu = (a.epilogue & GPUSQ_EPI_GELU) != 0;
  const int resident = num_cus();
  const Decision& dec = decide(IS_I8, a.M, a.N, a.K, gelu, resident, a.patch_P != 0, a.x_f16 != 0);
  int choice = dec.choice;
  // The 128 x 128 tiles are the choice for fp16 and int32 output: the narrow lines of int8 output, and quantising fp16 X, cost them more
  // than the other kernels (6304 x 192 -> 576 int8 output 9.0 us, kernel 2 7.6; 50432 x 192 -> 64 9.4, 64 x 64 tiles 8.9, kernel 2 10.5;
  // 25216 x 64 -> 128 from fp16 11.4, 64 x 64 tiles 8.6).
  if (choice == 1 && dec.forced < 0 && dec.even.tiles_n > 0) {
    if (a.x_f16)
      choice = 0;
    else if (IS_I8 && a.out_dt == GPUSQ_I8)
      choice = a.N <= kRowBlock ? 0 : 2;
  }
  // fp16 output and its codes: kernel 3 has no such epilogue
  if (a.codes_out != nullptr && choice == 3) choice = 2;
  // quantising fp16 activations on the way in exists in the small kernels only, and those take every ragged K
  if (a.x_f16 && choice == 2 && k_bytes % kStepBytes != 0) choice = small_choice(a.M, a.N, resident);
  // The kernel for few rows quantises in tiles of 16 rows: beyond one round of them, and with few K steps, the 64 x 64 tiles are ahead
  // (1576 x 192 -> 576 5.9 us against 7.5, 6304 x 64 -> 128 4.7 against 7.1; but 788 x 768 -> 768 10.7 against 8.8).
  if (a.x_f16 && choice == 4 && dec.forced != 4 && ceil_div(k_bytes, kStepBytes) <= 3 && ceil_div(a.M, 16) * ceil_div(a.N, kRowBlock) > 2 * (int64_t)resident) choice = 0;
  // the fused patch gather exists in the tile kernel and in the one for few rows, for 16 x 16 patches, fp16 output, no GELU
  if (a.patch_P != 0 && ((choice != 2 && choice != 4) || a.patch_P != 16 || a.out_dt != GPUSQ_F16 || gelu)) return GPUSQ_ERR_UNSUPPORTED;
  if (a.x_f16 && (!IS_I8 || choice == 2 || choice == 3)) return GPUSQ_ERR_UNSUPPORTED;
  if (choice == 4) return fewrows_supports(a) ? launch_fewrows(IS_I8, a, resident, s) : launch_small<IS_I8, 4, 1, 1, 4>(a, s);
  if (choice == 3) {
    if (!tile2_supports(IS_I8, false, a)) return GPUSQ_ERR_UNSUPPORTED;
    return launch_tile2(IS_I8, false, a, dec.plan, tile2_grid_of(dec.plan, 2 * resident), s);
  }
  if (choice == 0) return launch_small<IS_I8, 4, 1, 1, 4>(a, s);
  if (choice == 1) return launch_small<IS_I8, 4, 4, 2, 2>(a, s);
  const unsigned grid = 8u * (unsigned)dec.even.grid8;  // persistent
  if (even_total(dec.even) >= ((int64_t)1 << 31)) return GPUSQ_ERR_UNSUPPORTED;
  if ((dec.even.rounds + 2) * ceil_div(k_bytes, kStepBytes) >= ((int64_t)1 << 30)) return GPUSQ_ERR_UNSUPPORTED;
  if ((int64_t)a.N * 16 * 4 >= ((int64_t)1 << 31)) return GPUSQ_ERR_UNSUPPORTED;  // 32-bit lane offsets inside 16 rows of Y
  // 32-bit lane offsets inside the 256 rows of X of a tile (tile_x_offsets; the patch gather has its own limit)
  if (a.patch_P == 0 && 255 * k_bytes + kStepBytes >= ((int64_t)1 << 32)) return GPUSQ_ERR_UNSUPPORTED;
  if (k_bytes % kStepBytes != 0) return IS_I8 ? launch_tile1_i8_ragged(a, dec.even, grid, s) : launch_tile1_f16_ragged(a, dec.even, grid, s);
  return IS_I8 ? launch_tile1_i8(a, dec.even, grid, s) : launch_tile1_f16(a, dec.even, grid, s);
}

// Quantise X and multiply.  Many rows and few channels: see wide_takes.  Where the problem goes to the kernel for few rows and its K is not too long, that kernel
// quantises: with a given scale, or a range of X small enough for every workgroup to find for itself, in the one
// launch, else behind the range pass.  Otherwise the quantiser's one or two launches and the GEMM's.
// A range of 128 KB read by every workgroup costs what the range pass does: 75 KB (197 x 192) 5.8 against 6.7 us, 133 KB (64 x
// 1040) 8.2 against 8.6, 151 KB (394 x 192) 8.4 against 7.1.
constexpr int64_t kRangeHereBytes = 128 * 1024;

// Where the estimates of the kernel that quantises whole rows (wide.hip) say little, below 2048 rows or beyond two column blocks, but a launch less decides: up
// to 2^23 outputs, and K of up to 512 values, or 1024 (768 from 2048 rows on) where there are 2^20 outputs (fp32 X: and 2^21 at
// the most), for every chunk walks all of K by itself.  Under a given scale up to 256 values only: beyond it would be ahead as well, but the tests' counts of launches (two for 1576 x 384
// -> 1152) hold it there.  Quantiser and GEMM / whole rows 1989 x 128 -> 1152 under a given scale 8.6 / 5.9 us, 1301 x
// 128 -> 1472 + GELU 12.8 / 9.4, 2000 x 384 -> 1024 11.6 / 9.0, 1382 x 960 -> 960 13.9 / 11.6, 2548 x 224 -> 1600 13.3 / 9.3; beyond them 802 x 1184 -> 688 11.5 / 14.1, 882 x 960
// -> 736 fp32 10.9 / 13.6, 1576 x 768 -> 2304 + GELU fp32 13.5 / 14.3, 3199 x 576 -> 4160 fp32 19.6 / 23.1.
static bool wide_saves_a_launch(int64_t M, int64_t N, int64_t K, bool fp32, bool given) {
  const int64_t outputs = M * N;
  if (outputs > (1 << 23)) return false;
  if (K <= (given ? 2 : 4) * kStepBytes) return true;
  return !given && (!fp32 || outputs <= (1 << 21)) && outputs >= (1 << 20) && K <= (M < GPUSQ_WIDE_MIN_ROWS ? 8 : 6) * kStepBytes;
}
// Of these, the plans that are ahead.  A chunk of one slab has little work for the operands that it fetches: the more 64-channel blocks it has and the longer K, the more outputs it takes
// (2^18 for each K step and block beyond a line; own range, 12 blocks, fp32 753 x 512 -> 736 9.0 / 9.6, 1472 x 480 -> 752 11.0 / 10.2; at most 750000, for 1000 x 512 -> 768, 7 % behind in fp32, is held here by a test); the line
// is lower for rows that are stored by four, and for patches of fp32.  fp32 rows in chunks of four slabs, in which the epilogue stands alone behind a short K, are behind by 2 to 15 %; without a GELU those of whole 16 channels stay (2047 x 512 -> 4096
// is held there by a test).  Of 61274 and 12081 layers of whole and of no whole 16 channels timed (seldom more than 4096 rows, K 64 to 5120, N 32 to 5120) this takes 60372 and 10827, 1.21 and 1.16 times
// as fast, 150 and 133 slower by more than 3 % (12 % at the most); of the others 345 and 585 were slower.
static bool wide_plan_ahead(const GemmArgs& a, const WidePlan& p, bool fp32) {
  const bool narrow = a.N % 16 != 0, gelu = (a.epilogue & GPUSQ_EPI_GELU) != 0, patches = a.patch_P > 0;
  const int ksteps = (int)ceil_div((int64_t)a.K, kStepBytes), slabs = wide_slabs(p);
  if (slabs == 1 && ksteps <= 4 && (narrow || ksteps > (patches ? 3 : 2))) {
    const int line = patches ? (narrow ? (fp32 ? 3 : 2) - (ksteps <= 2) : fp32 ? 2 : 0) : (narrow ? (fp32 ? 2 : 1) : 0);
    const int64_t outputs = (int64_t)a.M * a.N;
    if (outputs < (int64_t)(ksteps + p.blocks - 12 + line) << 18 && (narrow || patches || outputs < 750 * 1000)) return false;
  }
  if (!fp32 || patches) return true;
  if (slabs == 3) return !gelu || ksteps < 4;
  return slabs < 4 || !(narrow || (gelu && ksteps > 2));
}
// Rows of Y of no whole 16 channels, stored by four, where the estimates, which are of whole pieces, take them: of 34505 sizes timed (M 2048 ... 66000, K 64 ... 5120, N 32 ... 1532) 33018 stay
// with whole rows, 1.15 times as fast, 527 slower by more than 3 % (14 % at the most); the 1487 given back are as fast either way, 513 were slower.  The conditions are one block of channels with int8 or GELU
// output and X up to 28.5 MB (32000 x 256 -> 60, int8 output, 10.4 / 11.1), two of a short K and many rows, int8 output without GELU of many outputs (29916 x 128 -> 1176 fp32 under a given scale 27.8 / 29.8), and fp32 rows
// behind a range pass, 36 to 96 of them to a CU.  Patches of four channels or more in fp32: in chunks of more than a slab.
static bool wide_narrow_ahead(const GemmArgs& a, const WidePlan& p, bool fp32, bool i8, bool own) {
  const int64_t M = a.M, N = a.N, x_bytes = M * a.K * (fp32 ? 4 : 2);
  const bool gelu = (a.epilogue & GPUSQ_EPI_GELU) != 0;
  const int ksteps = (int)ceil_div((int64_t)a.K, kStepBytes);
  if (a.patch_P > 0) return !fp32 || ksteps < 8 || wide_slabs(p) > 1;
  if (N <= 64) return x_bytes > 28500000 || !(i8 ? x_bytes > 8000000 : gelu);
  if (N <= 128 && (fp32 ? own && ksteps == 1 && M > 32768 : !own && ((ksteps == 1 && M > 49152) || (ksteps == 2 && M > 32768)))) return false;
  if (i8 && !gelu && (N > 1024 ? M > 8192 : N > 512 && M > 16384 && fp32 && own && ksteps <= 4)) return false;
  return !(fp32 && own && N <= 192 && ksteps > 2 && ksteps <= 5 && M > 9216 && M < 24576);
}

// Many rows and few channels: the kernel that quantises whole rows (wide.hip) by the estimates, from 2048 rows on (below, they are
// off by as much as there is to win) and up to the two column blocks of 1536 channels that were timed.  Calls in turn on three buffers of normal
// values, us, apart / here, own range and given scale: 14070 x 576 -> 256 16.3 / 14.2 and 12.8 / 10.0, 12608 x 768 -> 768 20.6 / 20.0 and 17.1 / 15.1, 7029 x 1152
// -> 256 17.0 / 15.0 and 13.5 / 10.9, 56475 x 3648 -> 704 306 / 266 and 235 / 187, 25216 x 3072 -> 768 106.7 / 107.5 and 86.5 / 83.9 (of what a GELU returns, which
// takes less power, with an own range 102.5 / 100.3).  Behind a range pass there is less to win (wide_margin_behind_range), and these go there
// under a given scale only: 30706 x 2256 -> 256 80.8 / 84.4 and 65.5 / 58.3, 19429 x 3312 -> 192 78.3 / 80.7 and 62.8 / 58.1, 20738 x 3072 -> 704 + GELU 86.9 / 95.0 (and
// 70.5 / 75.9), 22807 x 256 -> 128 fp32 + GELU, int8 output 16.0 / 18.4 (and 12.5 / 13.0), 11620 x 2304 -> 1056 fp32 61.2 / 66.3; not 28453 x 1600 -> 1920 + GELU 113 / 114.  Of
// 20022 sizes so timed (M 2048 ... 65792, K 64 ... 5120, N 32 ... 1536, both types and outputs, with and without GELU) it takes 68 % of the fp16 ones with an
// own range, 1.15 times as fast there, and 70 % under a given scale, 1.22 times; 49 and 58 % of the fp32 ones, 1.08 and 1.20 times.  2 % of those with an own range
// and 0.7 % of the others are slower by more than 5 % (8094 x 4608 -> 768 + GELU, int8 output, 59.3 / 66.5; 52052 x 640 -> 1440 under a given scale 67.5 / 79.3).
// Rows of Y that are no whole 16 channels are stored by four (12608 x 768 -> 772 27.6 / 23.7, 50000 x 384 -> 388 38.6 / 33.5, 1576 x 384 -> 1148 11.5 / 8.9; wide_narrow_ahead).
// Where the product goes to the kernel for few rows (those have no estimate here) it is ahead beyond 256 channels: 1.1 to 1.3 times up to 12 K steps, 1.1 with
// more of them up to 447 channels, from there on level or behind but for fp32 under a given scale (2085 x 3920 -> 640 24.7 / 27.8).
static bool wide_takes(const GemmArgs& a, gpusq_dtype dt, bool behind_range, int resident, const Decision& d, WidePlan& p) {
  const bool fp32 = dt == GPUSQ_F32, i8 = a.out_dt == GPUSQ_I8, gelu = (a.epilogue & GPUSQ_EPI_GELU) != 0;
  if ((d.forced >= 0 && d.forced < 5) || (!i8 && a.out_dt != GPUSQ_F16)) return false;
  if ((int64_t)a.K * 64 * 4 >= ((int64_t)1 << 31) || a.N >= (1 << 24)) return false;  // 32-bit lane offsets inside a chunk's rows
  const bool estimated = a.M >= GPUSQ_WIDE_MIN_ROWS && a.N <= 2 * kWideBlocks * kRowBlock;
  if (d.forced < 0 && !estimated && !wide_saves_a_launch(a.M, a.N, a.K, fp32, !behind_range && a.patch_P == 0)) return false;
  p = wide_plan(a.M, a.N, resident, fp32);
  if (p.chunks == 0 || d.forced == 5) return p.chunks > 0;
  if (!estimated) return wide_plan_ahead(a, p, fp32);
  if (a.N % 16 != 0 && !wide_narrow_ahead(a, p, fp32, i8, behind_range)) return false;
  if (d.choice == 4) return a.N > 256 && (a.K <= 12 * kStepBytes || a.N < 448 || (fp32 && !behind_range));
  const double margin = behind_range ? wide_margin_behind_range(a.M, a.N, a.K, fp32, i8) : wide_margin(a.K, fp32);
  return d.gemm_us > 0 && wide_us(p, a.M, a.N, a.K, resident, fp32, gelu, i8) < margin * quantise_and_gemm_us(d.gemm_us, a.M, a.N, a.K, fp32, i8);
}

// What quantises (GPUSQ_QUANTISE_*); WHOLE_ROWS: with this plan
static int quantiser_of(const GemmArgs& a, gpusq_dtype dt, bool given, int resident, WidePlan& p) {
  const bool gelu = (a.epilogue & GPUSQ_EPI_GELU) != 0;
  const bool few = fewrows_folds_quantiser(a.M, a.N, a.K, resident, dt == GPUSQ_F32) && fewrows_supports(a);
  const Decision& d = decide(true, a.M, a.N, a.K, gelu, resident, false);
  if (d.forced == 5 && a.N % 16 == 0 && wide_takes(a, dt, !given, resident, d, p)) return GPUSQ_QUANTISE_WHOLE_ROWS;
  if (few && d.choice == 4) return GPUSQ_QUANTISE_FEW_ROWS;
  return wide_takes(a, dt, !given, resident, d, p) ? GPUSQ_QUANTISE_WHOLE_ROWS : GPUSQ_QUANTISE_APART;
}

// 1 + the launches in front of the GEMM's own
static int launches_of(const GemmArgs& a, gpusq_dtype dt, int scale_is_input, int quantiser) {
  if (quantiser == GPUSQ_QUANTISE_APART) return scale_is_input ? 2 : 3;
  if (quantiser == GPUSQ_QUANTISE_WHOLE_ROWS) return scale_is_input ? 1 : 2;
  return scale_is_input || (int64_t)a.M * a.K * dtype_bytes(dt) <= kRangeHereBytes ? 1 : 2;
}

int linear_int8_launches(const GemmArgs& a, gpusq_dtype dt, int scale_is_input, int cus) {
  WidePlan p;
  return launches_of(a, dt, scale_is_input, quantiser_of(a, dt, scale_is_input != 0, cus > 0 ? cus : num_cus(), p));
}
int linear_int8_quantiser(const GemmArgs& a, gpusq_dtype dt, int scale_is_input, int cus) {
  WidePlan p;
  return quantiser_of(a, dt, scale_is_input != 0, cus > 0 ? cus : num_cus(), p);
}

gpusq_status launch_linear_int8(GemmArgs a, gpusq_dtype dt, int8_t* Xq, float* scale, int scale_is_input, void* workspace, hipStream_t s) {
  const int resident = num_cus();
  WidePlan plan;
  const int quantiser = quantiser_of(a, dt, scale_is_input != 0, resident, plan), launches = launches_of(a, dt, scale_is_input, quantiser);
  a.act_scale = scale;
  const int64_t range_bytes = launches == 2 ? (int64_t)gpusq_quantize_workspace_bytes(GPUSQ_PER_TENSOR, a.M, a.K) : 0;
  const bool apart = may_quantise_inside(a.X, dtype_bytes(dt), a.Y, dtype_bytes(a.out_dt), a.M, a.N, a.K, scale, scale_is_input != 0, a.out_scale,
                                         workspace, range_bytes);
  if (quantiser != GPUSQ_QUANTISE_APART && apart) {
    a.x_f16 = dt == GPUSQ_F32 ? 2 : 1;
    a.xq_out = Xq;
    if (!scale_is_input) {
      a.scale_out = scale;
      a.range_mode = launches == 1 ? kRangeHere : kRangePartials;
      if (launches == 2) {
        a.npartial = launch_amax(a.X, dt, (int64_t)a.M * a.K, workspace, s);
        a.partial = (const float*)workspace;
      }
    }
    return quantiser == GPUSQ_QUANTISE_WHOLE_ROWS ? launch_wide(a, plan, s) : launch_fewrows(true, a, resident, s);
  }
  const gpusq_status st = launch_quantize(a.X, dt, Xq, scale, GPUSQ_PER_TENSOR, scale_is_input, a.M, a.K, workspace, s);
  if (st != GPUSQ_OK) return st;
  a.X = Xq;
  return launch_typed<true>(a, s);
}

// The range pass over a.X, images of dt, and the kernel for whole rows on them
static gpusq_status launch_wide_patches(GemmArgs a, gpusq_dtype dt, int8_t* img_q, float* scale, void* workspace, const WidePlan& p, hipStream_t s) {
  a.x_f16 = dt == GPUSQ_F32 ? 2 : 1;
  a.xq_out = img_q;
  a.scale_out = scale;
  a.range_mode = kRangePartials;
  a.npartial = launch_amax(a.X, dt, (int64_t)a.M * a.K, workspace, s);
  a.partial = (const float*)workspace;
  return launch_wide(a, p, s);
}

// Patches of 16 x 16 too few for the kernels that gather them (launch_patch_embed_int8): two launches instead of quantiser, flattened patches and GEMM, four. Of
// 22830 sizes timed (1 to 2000 patches of one to four channels, 32 to 1600 channels out, fp16 and fp32) 1.40 times as fast in the 22158 that it takes, none slower by more than 3 %: 150 x 768 -> 640
// 13.8 / 10.3 us.  Of four channels, 1024 values, up to 512 patches and 160 K outputs: beyond 351 x 1024 -> 648 fp32 11.8 / 13.3, 756 x 1024 -> 228 11.9 / 12.6; more values were not timed.
static bool few_patches_take_whole_rows(int64_t M, int64_t N, int64_t K, int epilogue, gpusq_dtype dt, int resident, WidePlan& p) {
  const int forced = forced_kernel();
  if ((forced >= 0 && forced < 5) || (epilogue & GPUSQ_EPI_GELU) || M * N > 256 * 1024 || K > 8 * kStepBytes || (K > 6 * kStepBytes && (M * N > 160 * 1024 || M > 512)) || M * K * dtype_bytes(dt) >= ((int64_t)1 << 32)) return false;
  p = wide_plan(M, N, resident, dt == GPUSQ_F32);
  return p.chunks > 0;
}
gpusq_status launch_few_patches(const GemmArgs& a, gpusq_dtype dt, int8_t* img_q, float* scale, void* workspace, hipStream_t s) {
  WidePlan p;
  if (!few_patches_take_whole_rows(a.M, a.N, a.K, a.epilogue, dt, num_cus(), p)) return GPUSQ_ERR_UNSUPPORTED;
  return launch_wide_patches(a, dt, img_q, scale, workspace, p, s);
}
bool few_patches_take_whole_rows(int64_t M, int64_t N, int64_t K, int epilogue, gpusq_dtype dt, int cus) {
  WidePlan p;
  return few_patches_take_whole_rows(M, N, K, epilogue, dt, cus, p);
}

// The images in front of a patch embedding: the kernel for whole rows takes a product of its sizes as it takes a layer's under a given scale.  A
// range pass does come first, but the kernels that gather patches take longer than a layer's, which makes up for it.  Of 403 sizes timed (72 to
// 576 patches an image, 256 to 1024 values each, 192 to 1536 channels) it takes 238 of fp16, 1.19 times as fast, none slower, and 101 of fp32, 1.06 times, 8 %
// slower at the most (29120 x 256 -> 1088; apart / here 62 images of 304 x 304 -> 704 41.2 / 37.4).  Below 2048 patches the line for a layer with an own range is theirs
// as well (1536 x 768 -> 832 13.4 / 10.3, 560 x 256 -> 640 10.9 / 8.4, 704 x 768 -> 640 fp32 10.9 / 12.1; of 21035 sizes, 18008
// of them of fewer than 2048 patches, 77 are slower by more than 3 %, 11 % at the most).
gpusq_status launch_patch_embed_int8(GemmArgs a, gpusq_dtype dt, int8_t* img_q, float* scale, void* workspace, hipStream_t s) {
  const int resident = num_cus();
  const int choice = decide(true, a.M, a.N, a.K, false, resident, true).choice;
  if (choice != 2 && choice != 4) return GPUSQ_ERR_UNSUPPORTED;  // (before anything is launched)
  const int64_t pixels = (int64_t)a.M * a.K;
  a.act_scale = scale;
  WidePlan plan;
  const bool wide = pixels * dtype_bytes(dt) < ((int64_t)1 << 32) && wide_takes(a, dt, false, resident, decide(true, a.M, a.N, a.K, false, resident, false), plan) &&
                    may_quantise_inside(a.X, dtype_bytes(dt), a.Y, 2, a.M, a.N, a.K, scale, false, nullptr, workspace,
                                        (int64_t)gpusq_quantize_workspace_bytes(GPUSQ_PER_TENSOR, 1, pixels));
  if (wide) return launch_wide_patches(a, dt, img_q, scale, workspace, plan, s);
  const gpusq_status st = launch_quantize(a.X, dt, img_q, scale, GPUSQ_PER_TENSOR, 0, 1, pixels, workspace, s);
  if (st != GPUSQ_OK) return st;
  a.X = img_q;
  return launch_typed<true>(a, s);
}

gpusq_status launch_spgemm(bool is_i8, const GemmArgs& a, hipStream_t s) {
  return is_i8 ? launch_typed<true>(a, s) : launch_typed<false>(a, s);
}

}  // namespace gpusq
