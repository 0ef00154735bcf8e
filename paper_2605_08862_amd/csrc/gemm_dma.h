// Main loop of the GEMMs on the f16 MFMA with both operands copied to LDS by the memory pipeline (global -> LDS loads).
//
//   C^T[N, M] = W[N, K] * X[M, K]^T      W = packed weights (gemm_mfma.h), X = activations in chunk order (act_index).
//
// Why this shape.
//   * Both operands lie in memory in MFMA operand order, so a piece (1 KiB: 32 rows x 16 of K) is one load instruction
//     whose bytes land in LDS as they are: no registers hold what is in flight, no LDS stores are issued.  A fragment of a 16 x 16 x 32 product is 16 rows of
//     two consecutive pieces, four runs of 256 bytes, and its LDS read is free of conflicts (frag_lane).  Loops with the weights in a register ring (three tiles of them plus the
//     activations' staging registers) had 8 .. 24 KiB per wave in flight; here it is up to 130 KiB per CU, whatever the accumulators take.
//   * A stage is 32 of K (two pieces) of every row tile; NST stages are in LDS, NST - 2 of them in flight.  It is computed in two steps, 16 rows of each tile of
//     one operand in each.  One barrier per stage, between its two steps: the second step already reads the next stage's first fragments, so a stage starts with its
//     operands in registers, and the slot of the previous stage is free for stage i + NST - 1.
//   * The tile (MW x NW accumulator tiles of 32 x 32 per wave, WM x WN waves) is a template parameter: few rows take all rows and few
//     columns per workgroup, so that a weight is read once and as many CUs stream as columns allow.
// What bounds it (MI355X, 7B shape, gate/up in whole steps): 64 rows 55 -> 48.7 us, 5.6 TB/s of weights: memory.  1152 rows 272 -> 254 us: power.  Whatever
// the tile, busy share of the matrix units x clock ends at 1.24 GHz (1.28 PFLOP/s); 128 x 256 tiles whose operands come from the first-level cache
// only reach 1.39, without loads of weights 1.57, without reads of activations from LDS 1.33.
#pragma once
#include "gemm_mfma.h"

// Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2: a launch's (K split, N block, M block) space, M block
// fastest, is cut into 8 contiguous ranges, one per XCD, so that the M blocks that share weights run back to back on one XCD.
// Returns the position of this workgroup in that space, or -1.
__device__ __forceinline__ int xcd_flat(int total) {
  const int per_xcd = (total + 7) / 8, flat = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  return (int)(blockIdx.x / 8) < per_xcd && flat < total ? flat : -1;
}

template <int MW_, int NW_, int WM_, int WN_, int NST_>
struct DmaGemm {
  static constexpr int MW = MW_, NW = NW_, WM = WM_, WN = WN_, NST = NST_;
  static constexpr int RT = MW * WM, CT = NW * WN, BM = 32 * RT, WAVES = WM * WN, THREADS = 64 * WAVES;
  static constexpr int PIECES = 2 * (RT + CT);                    // 1 KiB pieces of a stage: activation tiles, then weight tiles
  static constexpr int PPW = (PIECES + WAVES - 1) / WAVES;        // pieces a wave requests (where they do not divide, the last one several times: the same bytes)
  static constexpr int STAGE_BYTES = PIECES * 1024, LDS_BYTES = NST * STAGE_BYTES;
  static_assert(NST >= 3 && LDS_BYTES <= 160 * 1024, "");
  static constexpr int WGS = WAVES <= 4 && 2 * LDS_BYTES <= 160 * 1024 ? 2 : 1;     // workgroups per CU

  struct Operands {
    const char* at[PPW];        // each piece of the next stage to be requested (activations: without the row)
    uint32_t lane[PPW];         // byte offset of this lane
    uint32_t step[PPW];         // bytes from one stage to the next
    int left;                   // stages not yet requested
  };
  __device__ static __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

  // x_row(r): row of X (clamped by the caller) for row r of the workgroup's tile; w_at(t): byte offset of the packed row tile at
  // position t of the workgroup's CT weight tiles (wave wn multiplies positions wn * NW .. wn * NW + NW - 1); w_half: bytes from a
  // tile's first 16 rows to its last 16 (kWHalf, unless a tile is put together from two).  s0: first stage (32 of K).
  template <typename XRow, typename WAt>
  __device__ static __forceinline__ void make_operands(Operands& op, const f16* X, int ld, XRow x_row, const f16* Wp, WAt w_at,
                                                       uint32_t w_half, int s0) {
    const int wave = wave_id(), lane = threadIdx.x & 63, ln = lane & 31, lg = lane >> 5;
    const uint32_t w_lane = (lg * 32 + (ln & 15)) * 16u + (ln >= 16 ? w_half : 0u);
#pragma unroll
    for (int j = 0; j < PPW; ++j) {
      const int p = min(wave * PPW + j, PIECES - 1), t = p >> 1, half = p & 1;
      if (p < 2 * RT) {
        op.at[j] = (const char*)X + ((size_t)s0 * 4 + half * 2) * ld * 16;
        op.lane[j] = (uint32_t)(lg * ld + x_row(t * 32 + ln)) * 16u;
        op.step[j] = 64u * ld;
      } else {
        op.at[j] = (const char*)Wp + w_at(t - RT) + (size_t)s0 * 2048 + half * 1024;
        op.lane[j] = w_lane;
        op.step[j] = 2048u;
      }
    }
  }
  // Requests piece j of the next stage into a slot.  Past the last stage that one is requested again, into slots
  // nobody reads: unconditional, so that the wait counts hold.
  __device__ static __forceinline__ void request(Operands& op, char* slot, int j) {
    char* dst = slot + (PIECES % WAVES == 0 ? wave_id() * PPW + j : min(wave_id() * PPW + j, PIECES - 1)) * 1024;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(wt_buffer(op.at[j]), (__attribute__((address_space(3))) void*)dst, 16, op.lane[j], 0, 0, 0);
    op.at[j] += op.left > 1 ? op.step[j] : 0u;
  }
  // Waits until at most N of this wave's requests are in flight, then for the other waves.
  template <int N> __device__ static __forceinline__ void wait_stage() {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
#endif
  }

  // Computes the workgroup's tile, ns stages of 32 of K.  operands(op) sets up its requests, finish(acc) stores it: C^T tiles, accumulator rows = weight
  // rows, lane = activation row (acc_row, acc_col).  finish() may use LDS behind a barrier.  All threads must call it.
  template <typename Ops, typename Finish>
  __device__ static __forceinline__ void run(int ns, char* lds, Ops operands, Finish finish) {
    const int wave = wave_id(), lane = frag_lane(), wm = wave / WN, wn = wave % WN;
    Operands op;
    operands(op);
    op.left = ns;
#pragma unroll
    for (int st = 0; st < NST - 1; ++st) {
#pragma unroll
      for (int j = 0; j < PPW; ++j) request(op, lds + st * STAGE_BYTES, j);
      --op.left;
    }
    // The operand with more tiles per wave goes through the registers in two halves (16 of each tile's 32 rows), the fragments of the other
    // one stay for the whole stage and are refilled in place, each after its last product.
    constexpr bool XH = MW >= NW;                         // the activations in halves
    constexpr int NH = XH ? MW : NW, NK = XH ? 2 * NW : 2 * MW, NM = NH * NK;
    const char* hb = lds + (XH ? wm * MW : RT + wn * NW) * 2048 + lane;
    const char* kb = lds + (XH ? RT + wn * NW : wm * MW) * 2048 + lane;
    u32x4 half[2][NH], keep[NK];
    wait_stage<PPW * (NST - 2)>();
#pragma unroll
    for (int i = 0; i < NH; ++i) half[0][i] = *(const u32x4*)(hb + i * 2048);
#pragma unroll
    for (int i = 0; i < NK; ++i) keep[i] = *(const u32x4*)(kb + i * 1024 - (i & 1) * (1024 - kWHalf));
    f32x4 acc[2 * MW][2 * NW];
#pragma unroll
    for (int a = 0; a < 2 * MW; ++a)
#pragma unroll
      for (int b = 0; b < 2 * NW; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    int slot = 0;
    for (int i = 0; i < ns; ++i) {
      const int next = slot + 1 == NST ? 0 : slot + 1, prev = slot == 0 ? NST - 1 : slot - 1;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        if (s == 1) {
          wait_stage<PPW * (NST - 3)>();                  // the next stage is complete, the previous one no longer read
          __builtin_amdgcn_sched_barrier(0);
        }
        const char* hs = s == 0 ? hb + slot * STAGE_BYTES + kWHalf : hb + next * STAGE_BYTES;
        const char* ks = kb + next * STAGE_BYTES;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          const int k = m / NH, h = k & 1 ? NH - 1 - m % NH : m % NH, a = XH ? 2 * h + s : k, b = XH ? k : 2 * h + s;
          if (m < NH) half[1 - s][m] = *(const u32x4*)(hs + m * 2048);
          if (s == 1) {
#pragma unroll
            for (int j = m * PPW / NM; j < (m + 1) * PPW / NM; ++j) request(op, lds + prev * STAGE_BYTES, j);
          }
          acc[a][b] = XH ? mfma_f16(keep[k], half[s][h], acc[a][b]) : mfma_f16(half[s][h], keep[k], acc[a][b]);
          __builtin_amdgcn_sched_barrier(0);
          if (s == 1 && m % NH == NH - 1) {
            keep[k] = *(const u32x4*)(ks + k * 1024 - (k & 1) * (1024 - kWHalf));
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      slot = next;
      --op.left;
    }
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // LDS must not be given away, nor reused, while a request may still write it
#endif
    finish(acc);
  }
};

// The same with the weights in registers: all rows of the tile in every wave (WM = 1), so a weight fragment has one reader and LDS
// would only be a buffer; LDS then carries the activations alone, and short stages leave room for two workgroups per CU.  RW stages
// of weights are in registers or in flight, as many stages of activations in LDS, one tile per workgroup.
template <int MW_, int NW_, int WN_, int RW_, int KS_ = 4>
struct StreamGemm {
  static constexpr int MW = MW_, NW = NW_, WM = 1, WN = WN_, RW = RW_, NSX = RW + 1, KS = KS_;   // KS: pieces (16 of K) of a stage, and its steps
  static constexpr int RT = MW, CT = NW * WN, BM = 32 * RT, WAVES = WN, THREADS = 64 * WAVES;
  static constexpr int PIECES = KS * MW, PX = (PIECES + WAVES - 1) / WAVES;
  static constexpr int STAGE_BYTES = PIECES * 1024, LDS_BYTES = NSX * STAGE_BYTES;
  // workgroups per CU: accumulators, weights and fragments in a SIMD's registers divided by its waves, LDS in half of a CU's
  static constexpr int WGS = WAVES <= 4 && 16 * MW * NW + 4 * RW * NW * KS + 8 * MW <= 232 && 2 * LDS_BYTES <= 160 * 1024 ? 2 : 1;
  static_assert(RW >= 2 && LDS_BYTES <= 160 * 1024, "");

  struct Operands {
    const char *x, *w[NW];      // next stage to be requested
    uint32_t x_lane[PX], x_step, w_half;
    int left_x, left_w;
  };
  __device__ static __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
  template <typename XRow, typename WAt>
  __device__ static __forceinline__ void make_operands(Operands& op, const f16* X, int ld, XRow x_row, const f16* Wp, WAt w_at,
                                                       uint32_t w_half, int s0) {
    const int wave = wave_id(), lane = threadIdx.x & 63, ln = lane & 31, lg = lane >> 5;
    op.x = (const char*)X + (size_t)s0 * 64 * ld;
    op.x_step = 32u * KS * ld;
#pragma unroll
    for (int j = 0; j < PX; ++j) {
      const int p = min(wave * PX + j, PIECES - 1);
      op.x_lane[j] = (uint32_t)((p % KS * 2 + lg) * ld + x_row(p / KS * 32 + ln)) * 16u;
    }
#pragma unroll
    for (int b = 0; b < NW; ++b) op.w[b] = (const char*)Wp + w_at(wave * NW + b) + (size_t)s0 * 2048;
    op.w_half = w_half;
  }
  __device__ static __forceinline__ void request_x(Operands& op, char* slot, int j) {
    char* dst = slot + (PIECES % WAVES == 0 ? wave_id() * PX + j : min(wave_id() * PX + j, PIECES - 1)) * 1024;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(wt_buffer(op.x), (__attribute__((address_space(3))) void*)dst, 16, op.x_lane[j], 0, 0, 0);
    if (j == PX - 1) op.x += op.left_x-- > 1 ? op.x_step : 0u;
  }
  // w[b][s]: rows 16 (s & 1) .. of tile b, 32 of K from 32 (s >> 1) on
  __device__ static __forceinline__ void load_w(Operands& op, u32x4 (&w)[NW][KS], int s) {
#pragma unroll
    for (int b = 0; b < NW; ++b) {
      w[b][s] = __builtin_amdgcn_raw_buffer_load_b128(wt_buffer(op.w[b]), frag_lane() + (s >> 1) * 2048, s & 1 ? (int)op.w_half : 0, 0);
      if (s == KS - 1) op.w[b] += op.left_w > 1 ? 1024 * KS : 0;
    }
    if (s == KS - 1) --op.left_w;
  }
  template <int N> __device__ static __forceinline__ void wait_stage() {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
#endif
  }
  // One stage, its weights in w: KS steps of 32 of K and 16 rows of each weight tile.  The weights of a step are requested for the stage RW
  // further as soon as the step is issued; the activations stay for two steps and are refilled in place, each after its last product.
  __device__ static __forceinline__ void stage(f32x4 (&acc)[2 * MW][2 * NW], u32x4 (&w)[NW][KS], u32x4 (&xf)[2 * MW], Operands& op, int& slot,
                                               char* lds, const char* xb) {
    constexpr int NM = 2 * MW * NW;
    const int next = slot + 1 == NSX ? 0 : slot + 1, prev = slot == 0 ? NSX - 1 : slot - 1;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (s == KS - 1) {
        wait_stage<KS * NW + (NSX - 3) * (PX + KS * NW)>();
        __builtin_amdgcn_sched_barrier(0);
      }
      const char* xs = s < KS - 1 ? xb + slot * STAGE_BYTES + (s + 1) * 1024 : xb + next * STAGE_BYTES;
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        const int a = m / NW, b = a & 1 ? NW - 1 - m % NW : m % NW;
        if (s == KS - 1) {
#pragma unroll
          for (int j = m * PX / NM; j < (m + 1) * PX / NM; ++j) request_x(op, lds + prev * STAGE_BYTES, j);
        }
        acc[a][2 * b + (s & 1)] = mfma_f16(w[b][s], xf[a], acc[a][2 * b + (s & 1)]);
        __builtin_amdgcn_sched_barrier(0);
        if ((s & 1) && m % NW == NW - 1) {
          xf[a] = *(const u32x4*)(xs + (a >> 1) * KS * 1024 + (a & 1) * kWHalf);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      load_w(op, w, s);
      __builtin_amdgcn_sched_barrier(0);
    }
    slot = next;
  }
  // The arguments are those of DmaGemm::run.
  template <typename Ops, typename Finish>
  __device__ static __forceinline__ void run(int n32, char* lds, Ops operands, Finish finish) {
    const int ns = n32 / (KS / 2);                        // n32: 32s of K (KS = 4: an even number)
    Operands op;
    operands(op);
    op.left_x = op.left_w = ns;
    u32x4 w[RW][NW][KS], xf[2 * MW];
    // in the order of the loop: the wait counts hold from the first stage on
#pragma unroll
    for (int st = 0; st < RW; ++st) {
#pragma unroll
      for (int j = 0; j < PX; ++j) request_x(op, lds + st * STAGE_BYTES, j);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < KS; ++s) load_w(op, w[st], s);
      __builtin_amdgcn_sched_barrier(0);
    }
    f32x4 acc[2 * MW][2 * NW];
#pragma unroll
    for (int a = 0; a < 2 * MW; ++a)
#pragma unroll
      for (int b = 0; b < 2 * NW; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const char* xb = lds + frag_lane();
    wait_stage<RW * KS * NW + (RW - 1) * PX>();
#pragma unroll
    for (int a = 0; a < 2 * MW; ++a) xf[a] = *(const u32x4*)(xb + (a >> 1) * KS * 1024 + (a & 1) * kWHalf);
    int slot = 0, i = 0;
    for (; i + RW <= ns; i += RW) {
#pragma unroll
      for (int r = 0; r < RW; ++r) stage(acc, w[r], xf, op, slot, lds, xb);
    }
#pragma unroll
    for (int r = 0; r < RW - 1; ++r)
      if (i + r < ns) stage(acc, w[r], xf, op, slot, lds, xb);
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // LDS must not be given away, nor reused, while a request may still write it
    // The wait counts hold only if every load of weights is issued where it is written.  A use of the whole ring on every path
    // keeps the compiler from dropping those of stages past the last one and from sinking those of the first stages into the loop.
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
      for (int b = 0; b < NW; ++b)
#pragma unroll
        for (int s = 0; s < KS; ++s) asm volatile("" ::"v"(w[r][b][s]));
#endif
    finish(acc);
  }
};
