// Projection GEMMs of the verify pass (Sec. 3.3 "token-wise" linear layers):
//   QKV (float32 out), O (+residual), gate/up (+SwiGLU), down (+residual).
// bf16 models run on the f16 MFMA main loop of gemm_dma.h over packed weights; float32 models (the
// tiny parity configuration, latency bound) run on the float32 MFMA.
#include "gemm_dma.h"
#include <type_traits>

__device__ __forceinline__ float silu_f(float x) { return x / (1.0f + __expf(-x)); }
// same function with the hardware reciprocal (1 ulp): used in the MFMA epilogue, where a full-precision
// division per output element costs more than the matrix products of a small tile
__device__ __forceinline__ float silu_fast(float x) { return x * __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }

// ------------------------------------------------------------------ float32 models
// One workgroup = 32 rows x 32 output columns (EPI_SWIGLU: 32 gate and the 32 up columns of the same features), its eight
// waves split K and meet in LDS at the end.  The products run on the float32 MFMA (32x32x2: float32 operands, float32
// accumulation).  The contraction index is permuted the same way for both operands (lane group g multiplies k = 8 i + 4 g + j), so
// that a lane loads 16 bytes of its row at a time; a wave keeps U loads of each operand in flight, eight, or four where it has no
// more (with eight the others were loaded again).  These models are
// small (the parity configuration), so latency is what bounds a launch: with 64 x 64 tiles on plain FMAs, one to four
// workgroups walked K alone.  20 rows, d_model 256, FFN 1024: O / down projections 62.5 us before (mean of the two), 9.1 us
// here; gate / up 28.9 and 9.4 us; QKV and the 4096-token LM head 26.2 and 6.5 us.  Four loads instead of eight for K = 256: O 5.7 -> 5.1, gate / up 10.0 -> 7.2, QKV
// 6.4 -> 4.9, LM head 6.7 -> 5.2 (sixteen for K = 1024: 12.2 -> 13.6).
constexpr int kF32Waves = 8;
template <int EPI, int U>
__global__ void __launch_bounds__(64 * kF32Waves) gemm_f32_kernel(const int32_t* __restrict__ n_rows_dev, int M_max, int N, int K,
                                                                  const float* __restrict__ A, const float* __restrict__ W,
                                                                  float* __restrict__ out) {
  constexpr int NB = (EPI == EPI_SWIGLU) ? 2 : 1;
  __shared__ f32x4 s_part[kF32Waves][NB][4][64];
  const int M = n_rows_dev ? min(*n_rows_dev, M_max) : M_max;
  const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
  if (m0 >= M) return;
  const int lane = threadIdx.x & 63, ln = lane & 31, lg = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb8 = K / 8, i0 = nb8 * wave / kF32Waves, i1 = nb8 * (wave + 1) / kF32Waves;      // K is a multiple of 64
  const float* ap = A + (size_t)min(m0 + ln, M - 1) * K + 4 * lg;
  const float* wp[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) wp[nb] = W + ((size_t)min(n0 + ln, N - 1) + (size_t)nb * N) * K + 4 * lg;
  f32x16 acc[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[nb][i] = 0.f;
  for (int i = i0; i < i1; i += U) {
    f32x4 a[U], w[NB][U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = min(i + u, i1 - 1) * 8;
      a[u] = *(const f32x4*)(ap + k);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) w[nb][u] = *(const f32x4_u*)(wp[nb] + k);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i + u < i1) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) acc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[nb][u][j], a[u][j], acc[nb], 0, 0, 0);
      }
  }
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4)
      s_part[wave][nb][i4][lane] = f32x4{acc[nb][4 * i4], acc[nb][4 * i4 + 1], acc[nb][4 * i4 + 2], acc[nb][4 * i4 + 3]};
  __syncthreads();
  if (wave >= 4) return;                                 // wave w finishes registers 4 w .. 4 w + 3: columns 8 w + 4 g ..
  const int m = m0 + ln, n = n0 + 8 * wave + 4 * lg;
  f32x4 v[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    v[nb] = s_part[0][nb][wave][lane];
#pragma unroll
    for (int w = 1; w < kF32Waves; ++w) {
      const f32x4 u = s_part[w][nb][wave][lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[nb][e] += u[e];
    }
  }
  if (m >= M) return;
  float* dst = out + (size_t)m * N + n;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (n + e >= N) continue;
    if (EPI == EPI_RESID_ADD) dst[e] += v[0][e];
    else if (EPI == EPI_SWIGLU) dst[e] = silu_f(v[0][e]) * v[NB - 1][e];
    else dst[e] = v[0][e];
  }
}

// ------------------------------------------------------------------ weight packing (once per context)
// bf16 row-major [N, K] -> float16 MFMA operand order (see gemm_mfma.h); rows beyond N are zero.
__global__ void __launch_bounds__(256) pack_weight_kernel(const bf16* __restrict__ w, int N, int K, f16* __restrict__ packed,
                                                          size_t n_chunks, int32_t* __restrict__ status) {
  const size_t c = (size_t)blockIdx.x * 256 + threadIdx.x;     // one 16-byte chunk of the packed array
  if (c >= n_chunks) return;
  const int nk = K / kBK;
  const int lane = c & 63, s = (c >> 6) & 3;
  const size_t blk = c >> 8;
  const int kt = blk % nk, nt = blk / nk;
  const int n = nt * 32 + (lane & 31), k = kt * kBK + (lane >> 5) * 32 + s * 8;
  f16x8 v;
  if (n < N) {
    const bf16x8 src = *(const bf16x8*)(w + (size_t)n * K + k);
    const f16x4 lo = to_f16x4_guarded((float)src[0], (float)src[1], (float)src[2], (float)src[3], status);
    const f16x4 hi = to_f16x4_guarded((float)src[4], (float)src[5], (float)src[6], (float)src[7], status);
#pragma unroll
    for (int j = 0; j < 4; ++j) { v[j] = lo[j]; v[4 + j] = hi[j]; }
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (f16)0.f;
  }
  *(f16x8*)(packed + c * 8) = v;
}

size_t packed_weight_elems(int N, int K) { return (size_t)((N + 31) / 32) * (K / kBK) * kWBlock; }

void launch_pack_weight(const void* w_bf16, int N, int K, void* packed_f16, int32_t* status, hipStream_t st) {
  const size_t n_chunks = packed_weight_elems(N, K) / 8;
  hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)((n_chunks + 255) / 256)), dim3(256), 0, st, (const bf16*)w_bf16,
                     N, K, (f16*)packed_f16, n_chunks, status);
}

// ------------------------------------------------------------------ bf16 models
// ---- gate/up projection + SwiGLU.  F = features; the packed matrix holds the F gate rows, then the F up rows.  Both rows of a
// feature land in the same lane:
//   NW even  the wave's weight tiles alternate: gate tile, up tile of the same 32 features;
//   NW == 1  ("mixed") a tile is 16 gate rows and their 16 up rows, put together by the addresses.  16 features per wave instead of
//            32 fill 256 CUs in finer steps.
struct GluArgs {
  const int32_t* n_rows_dev;
  int M_max, F, K;
  const f16 *A, *Wp;
  f16* out;
  int32_t* status;
};
// Tile id of the launch, M block fastest, BM rows apart.
template <typename G, int BM = G::BM>
__device__ __forceinline__ void glu_tile(const GluArgs& g, int m_blocks, int id, char* lds) {
  constexpr bool MIX = G::NW == 1;
  const int lane = threadIdx.x & 63;
  const int wave = G::wave_id(), wm = wave / G::WN, wn = wave % G::WN;
  const size_t tile_bytes = (size_t)(g.K / kBK) * 4096, half = (size_t)(g.F / 32) * tile_bytes;    // up rows behind the gate rows
  const int t_last = g.F / 32 - 1;
  const int m0 = id % m_blocks * BM, t0 = id / m_blocks * G::CT;
  auto operands = [&](typename G::Operands& op) {
    // position t: features 16 (t0 + t) .. (mixed), or the gate (t even) / up (t odd) rows of features 32 ((t0 + t) / 2) ..
    auto w_at = [&](int t) -> size_t { return min((t0 + t) >> 1, t_last) * tile_bytes + (((t0 + t) & 1) ? (MIX ? 256 : half) : 0); };
    G::make_operands(op, g.A, g.M_max, [&](int r) { return min(m0 + r, g.M_max - 1); }, g.Wp, w_at, MIX ? (uint32_t)half : kWHalf, 0);
  };
  auto finish = [&](f32x4 (&acc)[2 * G::MW][2 * G::NW]) {
    const int M = min(*g.n_rows_dev, g.M_max);
#pragma unroll
    for (int a = 0; a < 2 * G::MW; ++a) {
      const int m = m0 + (wm * 2 * G::MW + a) * 16 + acc_col(lane);
      if (m >= M) continue;
#pragma unroll
      for (int b = 0; b < G::NW; ++b) {                  // 16 features each
        const int f0 = (t0 + wn * G::NW + b) * 16;
        if (f0 >= g.F) continue;                         // F is a multiple of 64: whole tiles only
        const int gate = MIX ? 0 : (b >> 1) * 4 + (b & 1), up = MIX ? 1 : gate + 2;
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = silu_fast(acc[a][gate][e]) * acc[a][up][e];
        *(f16x4*)(g.out + act_index(m, f0 + acc_row(lane), g.M_max)) = to_f16x4_guarded(y[0], y[1], y[2], y[3], g.status);
      }
    }
  };
  G::run(g.K / 32, lds, operands, finish);
}
// Tile fixed by the launch, a CU for every workgroup: it does not wait for the row count before its first loads (rows beyond it are stale rows of the
// same buffer, each affecting only its own output row).
constexpr int kFewRows = 320;
template <typename G>
__global__ void __launch_bounds__(G::THREADS, (G::WGS * G::WAVES + 3) / 4) glu_kernel(GluArgs g, int m_blocks, int n_blocks) {
  extern __shared__ __align__(16) char lds[];
  const int id = xcd_flat(m_blocks * n_blocks);
  if (id >= 0) glu_tile<G>(g, m_blocks, id, lds);
}
// Rows and columns of a workgroup from the step's row count (glu_rule; Plan::n_rows[at]: place in its list).  Row blocks beyond the count are left out, and a
// last one of at most GT::BM live rows is one of GT (1.5B shape, 390 of 702 rows: 43 us with a whole last one, 40.6 here).
template <typename G, typename GT = G>
__device__ __forceinline__ void glu_rows(const GluArgs& g, int M, char* lds) {
  static_assert(GT::CT == G::CT && GT::THREADS == G::THREADS && GT::LDS_BYTES <= G::LDS_BYTES, "");
  const int m_blocks = (M + G::BM - 1) / G::BM, id = xcd_flat(m_blocks * ((g.F / 16 + G::CT - 1) / G::CT));
  if (id < 0) return;
  if (!std::is_same<G, GT>::value && M - id % m_blocks * G::BM <= GT::BM) glu_tile<GT, G::BM>(g, m_blocks, id, lds);
  else glu_tile<G>(g, m_blocks, id, lds);
}
// Four waves, two workgroups per CU: one's fill and epilogue run beside the other's products, and the last round of the CUs is a fine one.  64 features
// per workgroup (weights of 16 in a wave) for few row blocks, 128 for many.
typedef StreamGemm<3, 2, 4, 2> Glu96;
typedef StreamGemm<4, 2, 4, 2> Glu128;
typedef StreamGemm<2, 1, 4, 4> Glu64x64;
typedef StreamGemm<6, 1, 4, 4, 2> Glu192x64;
__global__ void __launch_bounds__(256, 2) glu_w4_kernel(GluArgs g, int at) {
  extern __shared__ __align__(16) char lds[];
  const int M = min(*g.n_rows_dev, g.M_max);
  switch (g.n_rows_dev[at]) {
    case 0: glu_rows<Glu96>(g, M, lds); break;
    case 1: glu_rows<Glu128, StreamGemm<2, 2, 4, 2>>(g, M, lds); break;
    case 2: glu_rows<Glu64x64>(g, M, lds); break;
    default: glu_rows<Glu192x64>(g, M, lds);
  }
}
// Eight waves of one weight tile each, or two (256 features), one workgroup per CU: a weight is read by fewer workgroups, and its round by a whole CU.
typedef StreamGemm<3, 1, 8, 3> Wide96;
typedef StreamGemm<4, 1, 8, 3> Wide128;
typedef StreamGemm<5, 1, 8, 3> Wide160;
typedef StreamGemm<6, 1, 8, 3> Wide192;
typedef StreamGemm<7, 1, 8, 2> Wide224;
typedef DmaGemm<4, 2, 2, 4, 4> Wide256;
typedef StreamGemm<4, 2, 8, 2> Wide128x256;
__global__ void __launch_bounds__(512, 2) glu_w8_kernel(GluArgs g, int at) {
  extern __shared__ __align__(16) char lds[];
  const int M = min(*g.n_rows_dev, g.M_max);
  switch (g.n_rows_dev[at]) {
    case 0: glu_rows<Wide96>(g, M, lds); break;
    case 1: glu_rows<Wide128>(g, M, lds); break;
    case 2: glu_rows<Wide160>(g, M, lds); break;
    case 3: glu_rows<Wide192>(g, M, lds); break;
    case 4: glu_rows<Wide224>(g, M, lds); break;
    case 5: glu_rows<Wide256>(g, M, lds); break;
    default: glu_rows<Wide128x256>(g, M, lds);
  }
}
// ---- float32 results (O and down projections, unfused QKV projection): one partial [M_max, N] slab per K split,
// out[split][m][n]; the consumer (RMSNorm, rotary kernel) sums the slabs.  Float atomics into the residual were measured at
// ~25 us per launch and are not used.
template <typename G>
__device__ __forceinline__ void slab_tile(const int32_t* __restrict__ n_rows_dev, int M_max, int N, int K, const f16* __restrict__ A,
                                          const f16* __restrict__ Wp, float* __restrict__ out, int m0, int nb, int split, int n_split, char* lds) {
  const int lane = threadIdx.x & 63;
  const int wave = G::wave_id(), wm = wave / G::WN, wn = wave % G::WN;
  const size_t tile_bytes = (size_t)(K / kBK) * 4096;
  const int t0 = nb * G::CT, t_last = N / 32 - 1;
  const int nk = K / kBK, s0 = 2 * (nk * split / n_split), s1 = 2 * (nk * (split + 1) / n_split);
  auto operands = [&](typename G::Operands& op) {
    G::make_operands(op, A, M_max, [&](int r) { return min(m0 + r, M_max - 1); }, Wp, [&](int t) { return min(t0 + t, t_last) * tile_bytes; }, kWHalf, s0);
  };
  auto finish = [&](f32x4 (&acc)[2 * G::MW][2 * G::NW]) {
    const int M = min(*n_rows_dev, M_max);
    float* dst = out + (size_t)split * M_max * N;
#pragma unroll
    for (int a = 0; a < 2 * G::MW; ++a) {
      const int m = m0 + (wm * 2 * G::MW + a) * 16 + acc_col(lane);
      if (m >= M) continue;
#pragma unroll
      for (int b = 0; b < 2 * G::NW; ++b) {
        const int n0 = (t0 + wn * G::NW) * 32 + b * 16;
        if (n0 >= N) continue;                           // N is a multiple of 32: whole tiles only
        *(f32x4*)(dst + (size_t)m * N + n0 + acc_row(lane)) = acc[a][b];
      }
    }
  };
  G::run(s1 - s0, lds, operands, finish);
}
// Tile and number of splits fixed by the launch, which does not wait for the row count either.
template <typename G>
__global__ void __launch_bounds__(G::THREADS, (G::WGS * G::WAVES + 3) / 4) slab_kernel(const int32_t* __restrict__ n_rows_dev, int M_max, int N, int K, const f16* __restrict__ A,
                                                          const f16* __restrict__ Wp, float* __restrict__ out, int n_blocks, int n_split) {
  extern __shared__ __align__(16) char lds[];
  const int m_blocks = (M_max + G::BM - 1) / G::BM, tiles = m_blocks * n_blocks;
  const int id = xcd_flat(tiles * n_split);
  if (id < 0) return;
  slab_tile<G>(n_rows_dev, M_max, N, K, A, Wp, out, id % tiles % m_blocks * G::BM, id % tiles / m_blocks, id / tiles, n_split, lds);
}
// Two tiles to choose from: tile and splits both from the step's row count (SlabRule).
template <typename G, typename GA>
__global__ void __launch_bounds__(256, 2) slab_alt_kernel(const int32_t* __restrict__ n_rows_dev, int M_max, int N, int K, const f16* __restrict__ A,
                                                          const f16* __restrict__ Wp, float* __restrict__ out, int nb_g, int nb_ga, int at) {
  extern __shared__ __align__(16) char lds[];
  const int M = min(*n_rows_dev, M_max), choice = n_rows_dev[at], n_split = choice & 15;
  const bool first = choice >> 4 == G::BM;
  const int bm = first ? G::BM : GA::BM, m_blocks = first ? (M + G::BM - 1) / G::BM : (M + GA::BM - 1) / GA::BM, tiles = m_blocks * (first ? nb_g : nb_ga);
  const int id = xcd_flat(tiles * n_split);
  if (id < 0) return;
  const int split = id / tiles, tile = id % tiles, m0 = tile % m_blocks * bm, nb = tile / m_blocks;
  if (first) slab_tile<G>(n_rows_dev, M_max, N, K, A, Wp, out, m0, nb, split, n_split, lds);
  else slab_tile<GA>(n_rows_dev, M_max, N, K, A, Wp, out, m0, nb, split, n_split, lds);
}

// ------------------------------------------------------------------ launchers
template <typename K_>
static void allow_lds(K_ kern, int bytes, bool& done) {  // more than 64 KiB of dynamic LDS needs an opt-in
  if (!done) { (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); done = true; }
}
static int grid8(int n) { return (n + 7) / 8 * 8; }

template <typename G>
static void launch_glu_t(const GluArgs& g, hipStream_t st) {
  const int m_blocks = (g.M_max + G::BM - 1) / G::BM, n_blocks = (g.F / 16 + G::CT - 1) / G::CT;
  static bool done = false;
  allow_lds(glu_kernel<G>, G::LDS_BYTES, done);
  hipLaunchKernelGGL(glu_kernel<G>, dim3(grid8(m_blocks * n_blocks)), dim3(G::THREADS), G::LDS_BYTES, st, g, m_blocks, n_blocks);
}
// Measured in us (gate/up of the 1.5B shape, 8960 features, and of the 7B shape, 18944; the loops with weights in registers and
// activations staged through registers that were here before in brackets; 7B at 64, 288 and 1185 rows and 1.5B from 432 rows in whole steps):
//   64 rows 13.3 (22.3) / 48.7 (55.0)    144 rows 18.6 (28.7) / 59.4 (73.4)    288 rows 22.9 (31.6) / 80.1 (104)
//   432 rows 28.9 (44.7)    576 rows 33.9 (41.4)    1037 rows 58.4 (73.0)    1152 rows - / 254 (324)    3480 rows 157.6 (190.9)
static bool glu_wide(int F) { return F / 16 > 3 * kCUs; }   // more columns than 256 workgroups of three waves with 16 features each take
static bool glu_mix(int F, int K) { return packed_weight_elems(F, K) * 2 < ((size_t)1 << 32); }   // the mixed tiles address the up rows with a 32-bit offset
// One row block for all rows of the limit (a wide matrix: up to 320 rows), columns in steps of 16 features per wave: launch_glu.  Where a tile of at most 192 rows takes one
// round of the CUs, up to 640 rows, it is fixed, too: a launch that reads the step's choice first took 0.4 us more (1.5B shape, 576 rows).  Otherwise the tile follows from the step's
// row count, in one of two launch shapes: four waves and two workgroups per CU, or eight and one.  Measured by themselves with weights that no cache holds, us (rows x features),
// 96 / 128 x 128 and 64 / 192 x 64 in four waves | 96 / 128 / 160 / 192 / 224 / 256 x 128 and 128 x 256 in eight:
//    8960 x 1536,   43 rows  21.2 / 21.2 / 14.1 / 16.2 | 21.1 / 21.3 / 22.3 / 23.3 / 29.6 / 30.6 / 36
//    8960 x 1536,  128 rows  21.9 / 25.8 / 24.3 / 19 | 21.5 / 25.4 / 25.9 / 26.4 / 30.9 / 32.3 / 41.4
//    8960 x 1536,  277 rows  23.5 / 23.3 / 31.7 / 33.2 | 24.1 / 24.8 / 27.7 / 30.1 / 35.3 / 38.8 / 38.9
//    8960 x 1536,  432 rows  38.4 / 38.5 / 40.7 / 34.2 | 39.2 / 40.9 / 29 / 32.3 / 35.6 / 38.8 / 40
//    8960 x 1536, 1037 rows  65.4 / 59.5 / 86 / 63.7 | 67.8 / 67.4 / 58.1 / 64.1 / 71.1 / 77.5 / 72.3
//   18944 x 3584,   43 rows  52.7 / 52.5 / 63.7 / 85.4 | 52.4 / 52.5 / 54.3 / 56.9 / 75.7 / 83.9 / 85.8
//   18944 x 3584,  144 rows  91 / 88.3 / 90.9 / 89.2 | 93.9 / 103 / 64 / 64.8 / 76.2 / 80.9 / 87.3
//   18944 x 3584,  256 rows  91 / 105 / 117 / 102 | 92.5 / 110 / 115 / 120 / 144 / 81.9 / 93.4
//   18944 x 3584,  320 rows  120 / 96 / 137 / 110 | 122 / 104 / 122 / 125 / 145 / 157 / 92.5
//   18944 x 3584,  505 rows  156 / 141 / 217 / 145 | 162 / 155 / 164 / 133 / 159 / 166 / 173
//   18944 x 3584, 1037 rows  272 / 260 / 399 / 255 | 285 / 282 / 279 / 261 / 239 / 276 / 255
//   18944 x 3584, 1500 rows  377 / 319 / 554 / 357 | 403 / 352 / 350 / 342 / 373 / 343 / 343
//   11008 x 4096,  505 rows  123 / 112 / 151 / 112 | 121 / 118 / 123 / 131 / 145 / 93.6 / 105
// The times of the rule lose least against the fastest tile, of each shape and of both, at 16 .. 4352 rows of those and of 5632 x 2048, 9728 x 2560 and 1408 x 512 (features x K).  The
// launch shape can only follow from the row limit: the faster one there.  Above 640 rows eight waves are also taken at up to 6 % more time of a full step, since steps of few live rows lose
// more without them (18944 x 3584, 144 rows: 82 .. 90 us in four waves, 64 in eight), but with fewer than 32 K tiles four waves, where eight gain 3 % of a full step at best and lose up to
// 10 % of others (8960 x 1536, 1200 rows 60.4 / 67.6 us).
// Tiles fixed by the row limit up to 640 rows, and of 128 rows above, were here before: 7B shape, 280 of 504 rows 129 us (102), 134 of 714 rows 99 (75); 1.5B shape, 197 of 639 rows 34 (25).
static TileRule glu_rule(int M_max, int F, int K) {
  TileRule r;
  const bool mix = glu_mix(F, K);
  if (mix && ((M_max + 31) / 32 <= 5 || (M_max <= kFewRows && glu_wide(F)))) return r;
  const int n64 = F / 64, n128 = (F + 127) / 128, nk = K / kBK;
  const TileRule w4{CHOICE_GLU, 0, nk, mix ? 4 : 2, {{96, n128, 78, 350}, {128, n128, 78, 483}, {64, n64, 45, 200}, {192, n64, 66, 612}}};
  const TileRule w8{CHOICE_GLU, 0, nk, 7, {{96, n128, 75, 539}, {128, n128, 86, 709}, {160, n128, 105, 571}, {192, n128, 112, 940}, {224, n128, 134, 819}, {256, n128, 141, 915},
                                          {128, (F + 255) / 256, 145, 722}}};
  if (M_max <= 640) {
    const TileRule one{0, 0, nk, mix ? 4 : 2, {w4.tile[0], w4.tile[1], w8.tile[2], w8.tile[3]}};
    const int c = one.choice(M_max);
    if (one.blocks(c, M_max) <= kCUs) { r.fixed = 1 + c; return r; }
  }
  r = w4;
  if (mix) {
    const int per_cent = M_max <= 640 ? 100 : nk >= 32 ? 106 : 0;
    if (w8.cost(w8.choice(M_max), M_max) * 100 <= w4.cost(w4.choice(M_max), M_max) * per_cent) { r = w8; r.waves = 8; }
  }
  r.size_grid(M_max);
  return r;
}
static void launch_glu(const int32_t* n_rows_dev, int M_max, int F, int K, const void* A, const void* W, void* out, int32_t* status, const TileRule& rule, hipStream_t st) {
  const GluArgs g{n_rows_dev, M_max, F, K, (const f16*)A, (const f16*)W, (f16*)out, status};
  const int rt = (M_max + 31) / 32;
  const bool wide = glu_wide(F);
  if (!rule.at && !rule.fixed && rt <= 5) {
    // one row block, columns in steps of 16 features per wave: one workgroup per CU
    if (wide) {
      if (rt <= 2) launch_glu_t<StreamGemm<2, 1, 5, 3>>(g, st);
      else if (rt == 3) launch_glu_t<StreamGemm<3, 1, 5, 3>>(g, st);
      else if (rt == 4) launch_glu_t<StreamGemm<4, 1, 5, 6, 2>>(g, st);
      else launch_glu_t<StreamGemm<5, 1, 5, 6, 2>>(g, st);
    } else {
      if (rt <= 2) launch_glu_t<StreamGemm<2, 1, 3, 3>>(g, st);
      else if (rt == 3) launch_glu_t<StreamGemm<3, 1, 3, 3>>(g, st);
      else if (rt == 4) launch_glu_t<StreamGemm<4, 1, 3, 3>>(g, st);
      else launch_glu_t<StreamGemm<5, 1, 3, 3>>(g, st);
    }
    return;
  }
  switch (rule.fixed) {
    case 1: launch_glu_t<Glu96>(g, st); return;
    case 2: launch_glu_t<Glu128>(g, st); return;
    case 3: launch_glu_t<Wide160>(g, st); return;
    case 4: launch_glu_t<Wide192>(g, st); return;
    default: break;
  }
  if (!rule.at) {
    // the same, for more than seven row tiles with two or three groups of waves side by side in the rows and both operands copied to LDS (192 / 224 rows by
    // themselves 68 / 74 us, 60.5 / 67 here; 288 rows 87, 95 with 96-row tiles of 128 features)
    if (rt == 6) launch_glu_t<StreamGemm<6, 1, 5, 4, 2>>(g, st);
    else if (rt == 7) launch_glu_t<StreamGemm<7, 1, 5, 4, 2>>(g, st);
    else if (rt == 8) launch_glu_t<DmaGemm<4, 1, 2, 5, 6>>(g, st);
    else if (rt == 9) launch_glu_t<DmaGemm<3, 1, 3, 5, 5>>(g, st);
    else launch_glu_t<DmaGemm<5, 1, 2, 5, 5>>(g, st);
    return;
  }
  static bool w4 = false, w8 = false;
  if (rule.waves == 8) {
    constexpr int lds = Wide256::LDS_BYTES;
    static_assert(Wide96::LDS_BYTES <= lds && Wide128::LDS_BYTES <= lds && Wide160::LDS_BYTES <= lds && Wide192::LDS_BYTES <= lds && Wide224::LDS_BYTES <= lds && Wide128x256::LDS_BYTES <= lds, "");
    allow_lds(glu_w8_kernel, lds, w8);
    hipLaunchKernelGGL(glu_w8_kernel, dim3(grid8(rule.grid)), dim3(512), lds, st, g, rule.at);
    return;
  }
  constexpr int lds = Glu192x64::LDS_BYTES;
  static_assert(Glu96::LDS_BYTES <= lds && Glu128::LDS_BYTES <= lds && Glu64x64::LDS_BYTES <= lds && 2 * lds <= 160 * 1024, "");
  allow_lds(glu_w4_kernel, lds, w4);
  hipLaunchKernelGGL(glu_w4_kernel, dim3(grid8(rule.grid)), dim3(256), lds, st, g, rule.at);
}

template <typename G>
static void launch_slab(const int32_t* n_rows_dev, int M_max, int N, int K, const void* A, const void* W, void* out, int n_split,
                        hipStream_t st) {
  const int m_blocks = (M_max + G::BM - 1) / G::BM, n_blocks = (N + G::CT * 32 - 1) / (G::CT * 32), tiles = m_blocks * n_blocks;
  static bool done = false;
  allow_lds(slab_kernel<G>, G::LDS_BYTES, done);
  hipLaunchKernelGGL(slab_kernel<G>, dim3(grid8(tiles * n_split)), dim3(G::THREADS), G::LDS_BYTES, st, n_rows_dev, M_max, N, K, (const f16*)A, (const f16*)W,
                     (float*)out, n_blocks, n_split);
}
template <typename G, typename GA>
static void launch_slab_alt(const int32_t* n_rows_dev, int M_max, int N, int K, const void* A, const void* W, void* out, const SlabRule& rule, hipStream_t st) {
  const int nb = (N + G::CT * 32 - 1) / (G::CT * 32), nba = (N + GA::CT * 32 - 1) / (GA::CT * 32);
  const int ta = (M_max + G::BM - 1) / G::BM * nb, tb = (M_max + GA::BM - 1) / GA::BM * nba, tiles = ta > tb ? ta : tb;
  constexpr int lds = G::LDS_BYTES > GA::LDS_BYTES ? G::LDS_BYTES : GA::LDS_BYTES;
  static bool done = false;
  allow_lds(slab_alt_kernel<G, GA>, lds, done);
  // tiles(M) * splits(M) never exceeds max(tiles(M_max), cap)
  hipLaunchKernelGGL((slab_alt_kernel<G, GA>), dim3(grid8(tiles > rule.cap ? tiles : rule.cap)), dim3(256), lds, st, n_rows_dev, M_max, N, K, (const f16*)A,
                     (const f16*)W, (float*)out, nb, nba, rule.at);
}
// Tile and split of a float32-result GEMM of at most 640 rows: the cheapest of the tiles below by rounds of the CUs x (K tiles per split x time of
// one + 3.9 us) + slabs.  The times (and what a slab weighs) are those under which the choices lose least against the fastest of all tiles and
// splits, measured with weights that no cache holds at 40 .. 640 rows of 1536 x 1536, 2048 x 1536, 1536 x 8960, 3584 x 3584, 4608 x 3584 and 3584 x
// 18944 (columns x K): 0.8 % on average, 4.7 % with the times of launches by themselves that were here before (7B shape, down projection, 400 rows
// 66.7 us and six slabs, now 60.4 and three; O projection, 64 rows 8.9 and seven, now 8.1 and four).  On 13 more matrices from 512 x 1024 to 6144 x 4096 they lose 1.2 %.
typedef StreamGemm<2, 1, 2, 4> T64x64;
typedef StreamGemm<2, 1, 4, 4> T64x128;
typedef StreamGemm<3, 1, 4, 3> T96x128;
typedef StreamGemm<4, 1, 4, 3> T128x128;
typedef StreamGemm<5, 1, 4, 3> T160x128;
typedef StreamGemm<3, 2, 4, 2> T96x256;
typedef StreamGemm<4, 2, 4, 2> T128x256;
struct SlabPick { int tile, split, cost; };
static SlabPick pick_slab(int M_max, int N, int nk) {
  static const struct { int bm, bn, t; } cfg[] = {{64, 64, 26}, {64, 128, 43}, {96, 128, 47}, {128, 128, 57}, {160, 128, 67}, {96, 256, 74}, {128, 256, 82}};
  SlabPick best{0, 1, 0x7fffffff};
  for (int i = 0; i < 7; ++i) {
    const int tiles = (M_max + cfg[i].bm - 1) / cfg[i].bm * ((N + cfg[i].bn - 1) / cfg[i].bn);
    for (int s = 1; s <= kMaxGemmSplit && (s == 1 || 4 * s <= nk); ++s) {
      const int c = (tiles * s + kCUs - 1) / kCUs * ((nk + s - 1) / s * cfg[i].t + 390) + (s - 1) * gemm_slab_cost(M_max, N) * 13 / 10;
      if (c < best.cost) best = SlabPick{i, s, c};
    }
  }
  return best;
}
int gemm_slab_time(int M_max, int N, int K) { return pick_slab(M_max, N, K / kBK).cost; }
enum SlabTile { T_96x256_128x128 = 7, T_96x256_160x128, T_96x256_128x256, T_96x128_128x128, T_96x128_160x128 };   // up to 6: place in pick_slab's list
static SlabRule slab_rule(int M_max, int N, int nk, int at) {
  if (M_max <= 640) {
    const SlabPick pick = pick_slab(M_max, N, nk);
    SlabRule r{pick.split, 0, 0, 0, 0, 0};
    r.tile = pick.tile;
    return r;
  }
  const int nb128 = (N + 127) / 128, nb256 = (N + 255) / 256;
  // (The times of a K tile here are from launches by themselves on loops of 32 x 32 x 16 products; those of pick_slab have been measured since, these not.)
  // The first tile: 96 rows x 256 columns, 128 where the row limit has too few of those to fill the CUs (two layers of d = 256, 390 of
  // 702 rows: O and down 6.6 us with 256 columns or 128 rows, 5.6 here; 1.5B shape 10.1 and 22.9, 9.7 and 23.3).  96 x 128 takes 43 per K tile where it is
  // the better one.
  const bool few = (M_max + 95) / 96 * nb256 < 128;
  SlabRule r{0, T96x256::BM, few ? nb128 : nb256, nk, 2 * kCUs, 0, 0, few ? 43 : 83, 0, N, at};
  if (few || nk < 96) {                                  // the second tile: the better one at the row limit
    auto cost = [&](int bm, int t) {
      const int tiles = (M_max + bm - 1) / bm * nb128, tsl = gemm_slab_cost(M_max, N);
      return gemm_split_cost(tiles, nk, 2 * kCUs, gemm_adaptive_split(tiles, nk, 2 * kCUs, t, tsl), t, tsl);
    };
    const bool rows128 = nk >= 96 || cost(128, 51) < cost(160, 68);
    r.bm_alt = rows128 ? T128x128::BM : T160x128::BM;
    r.n_blocks_alt = nb128;
    r.t_alt = rows128 ? 51 : 68;
    r.tile = few ? (rows128 ? T_96x128_128x128 : T_96x128_160x128) : rows128 ? T_96x256_128x128 : T_96x256_160x128;
  } else {
    r.bm_alt = T128x256::BM;
    r.n_blocks_alt = nb256;
    r.t_alt = 92;
    r.tile = T_96x256_128x256;
  }
  return r;
}
void gemm_slab_rules(const Shape& s, int M_max, SlabRule (&r)[3]) {
  if (s.dtype != BS_BF16) return;
  r[SLAB_QKV] = slab_rule(M_max, s.Nqkv(), s.d / kBK, CHOICE_SLABS + SLAB_QKV);
  r[SLAB_O] = slab_rule(M_max, s.d, s.Hq * s.D / kBK, CHOICE_SLABS + SLAB_O);
  r[SLAB_DOWN] = slab_rule(M_max, s.d, s.F / kBK, CHOICE_SLABS + SLAB_DOWN);
}
TileRule gate_up_rule(const Shape& s, int M_max) { return s.dtype == BS_BF16 ? glu_rule(M_max, s.F, s.d) : TileRule{}; }
static SlabCount launch_slabs(const int32_t* n_rows_dev, int M_max, int N, int K, const void* A, const void* W, void* out, const SlabRule& r, hipStream_t st) {
#define BS_SLAB(T_) launch_slab<T_>(n_rows_dev, M_max, N, K, A, W, out, r.fixed, st)
#define BS_SLAB_ALT(G_, T_) launch_slab_alt<G_, T_>(n_rows_dev, M_max, N, K, A, W, out, r, st)
  switch (r.tile) {
    case 0: BS_SLAB(T64x64); break;
    case 1: BS_SLAB(T64x128); break;
    case 2: BS_SLAB(T96x128); break;
    case 3: BS_SLAB(T128x128); break;
    case 4: BS_SLAB(T160x128); break;
    case 5: BS_SLAB(T96x256); break;
    case 6: BS_SLAB(T128x256); break;
    case T_96x256_128x128: BS_SLAB_ALT(T96x256, T128x128); break;
    case T_96x256_160x128: BS_SLAB_ALT(T96x256, T160x128); break;
    case T_96x256_128x256: BS_SLAB_ALT(T96x256, T128x256); break;
    case T_96x128_128x128: BS_SLAB_ALT(T96x128, T128x128); break;
    default: BS_SLAB_ALT(T96x128, T160x128);
  }
#undef BS_SLAB
#undef BS_SLAB_ALT
  return SlabCount{r.fixed, r.at};
}

template <int EPI>
static void launch_f32(const int32_t* n_rows_dev, int M_max, int N, int K, const void* A, const void* W, void* out, hipStream_t st) {
  const int loads = (K / 8 + kF32Waves - 1) / kF32Waves;           // of a wave, per operand
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((N + 31) / 32, (M_max + 31) / 32), dim3(64 * kF32Waves), 0, st, n_rows_dev, M_max, N, K,
                       (const float*)A, (const float*)W, (float*)out);
  };
  if (loads <= 4) go(gemm_f32_kernel<EPI, 4>);
  else go(gemm_f32_kernel<EPI, 8>);
}

SlabCount launch_gemm(int dtype, GemmEpilogue epi, const int32_t* n_rows_dev, int M_max, int N, int K, const void* A, const void* W, void* out,
                      int32_t* status, hipStream_t st, const SlabRule& rule, const TileRule& glu) {
  const SlabCount none{0, 0};
  if (dtype == BS_F32) {
    if (epi == EPI_SWIGLU) launch_f32<EPI_SWIGLU>(n_rows_dev, M_max, N, K, A, W, out, st);
    else if (epi == EPI_RESID_ADD) launch_f32<EPI_RESID_ADD>(n_rows_dev, M_max, N, K, A, W, out, st);
    else launch_f32<EPI_STORE_F32>(n_rows_dev, M_max, N, K, A, W, out, st);
    return none;
  }
  if (epi != EPI_SWIGLU) return launch_slabs(n_rows_dev, M_max, N, K, A, W, out, rule, st);
  launch_glu(n_rows_dev, M_max, N, K, A, W, out, status, glu, st);
  return none;
}
