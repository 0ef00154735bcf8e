// QKV projection fused with the rotary embedding and the tentative KV append (bf16 models, head size 128).
//
//   [M, d] x [ (Hq + 2 Hkv) * 128, d ]^T, then per head: q and k rotated at the row's absolute position
//   (pairs (j, j + 64)), q stored as float16 rows (attention operand), k and v rounded to bf16 and written
//   into the slot's KV page in the page layout.
//
// One workgroup = rows x one head.  The partner of column j (< 64) of a head is two weight tiles further:
//   two columns of waves (many rows)  wave column w multiplies tiles w and w + 2, so that both halves of a rotation are in one
//                                     lane and the epilogue needs no exchange;
//   four columns of waves (fewer rows) one tile each; the waves exchange their accumulators through LDS once.
// The float32 projection never goes to memory and q, k, v are rounded exactly once, after the rotation.
#include "gemm_dma.h"
#include <type_traits>

namespace {
constexpr int kD = 128;
constexpr int kLdx = kD + 4;                            // padded row (floats) of the exchange buffer

struct QkvArgs {
  int M_max, K, Hq, Hkv;
  const f16 *A, *Wp;
  const float *cos_t, *sin_t;
  f16 *q_out, *k_pages, *v_pages;
};

template <typename G>
__device__ __forceinline__ void qkv_tile(const Plan& p, const QkvArgs& g, int m0, int head, char* lds) {
  constexpr bool PAIR = G::NW == 2;
  static_assert(G::CT == 4 && (PAIR ? G::WN == 2 : G::WN == 4), "a workgroup's columns are one head");
  const int wave = G::wave_id(), wm = wave / G::WN, wn = wave % G::WN;
  const int lane = threadIdx.x & 63;
  const size_t tile_bytes = (size_t)(g.K / kBK) * 4096;
  // position t = wn * NW + b of the LDS tiles holds tile wn + 2 b of the head (PAIR), or tile t
  auto operands = [&](typename G::Operands& op) {
    G::make_operands(op, g.A, g.M_max, [&](int r) { return min(m0 + r, g.M_max - 1); }, g.Wp,
                     [&](int t) { return (size_t)(head * 4 + (PAIR ? (t >> 1) + 2 * (t & 1) : t)) * tile_bytes; }, kWHalf, 0);
  };
  auto finish = [&](f32x4 (&acc)[2 * G::MW][2 * G::NW]) {
  const int M = min(p.n_rows[0], g.M_max);
  // Accumulator acc[a][b][e]: row m0 + 16 (2 wm MW + a) + acc_col, column 16 b' + acc_row + e of the head, b' = b, or that of the tile.
  const bool is_v = head >= g.Hq + g.Hkv;
  int place[2 * G::MW];                                 // k or v head: the rows' cache places
#pragma unroll
  for (int a = 0; a < 2 * G::MW; ++a) place[a] = head >= g.Hq ? p.row_kv[min(m0 + (wm * 2 * G::MW + a) * 16 + acc_col(lane), g.M_max - 1)] : 0;
  float* s_x = (float*)lds;                             // [BM][kLdx]
  if constexpr (!PAIR) {
    if (!is_v) {
      __syncthreads();                                  // every wave is done reading the loop's LDS stages
#pragma unroll
      for (int a = 0; a < 2 * G::MW; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          *(f32x4*)(s_x + ((wm * 2 * G::MW + a) * 16 + acc_col(lane)) * kLdx + 32 * wn + 16 * b + acc_row(lane)) = acc[a][b];
      __syncthreads();
    }
  }
#pragma unroll
  for (int a = 0; a < 2 * G::MW; ++a) {
    const int m = m0 + (wm * 2 * G::MW + a) * 16 + acc_col(lane);
    if (m >= M) continue;
    const int tok = place[a] & (kPage - 1);
    const size_t pbase = (size_t)(place[a] / kPage) * kv_page_elems(g.Hkv, kD);
    // four consecutive columns d .. d + 3 of the head
    auto store = [&](int d, const float (&y)[4]) {
      if (head < g.Hq) {
        *(f16x4*)(g.q_out + ((size_t)m * g.Hq + head) * kD + d) = to_f16x4_guarded(y[0], y[1], y[2], y[3], p.status);
        return;
      }
      // bf16-rounded values in float16 encoding (page format)
      const f16x4 v = to_f16x4_guarded((float)(bf16)y[0], (float)(bf16)y[1], (float)(bf16)y[2], (float)(bf16)y[3], p.status);
      if (!is_v) {
        *(f16x4*)(g.k_pages + pbase + k_index_bf16(kD, head - g.Hq, tok, d)) = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) g.v_pages[pbase + v_index_bf16(kD, head - g.Hq - g.Hkv, tok, d + e)] = v[e];
      }
    };
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int d = 32 * wn + 16 * b + acc_row(lane);
      f32x4 c = f32x4{1.f, 1.f, 1.f, 1.f}, sn = f32x4{0.f, 0.f, 0.f, 0.f};
      if (!is_v) {
        c = *(const f32x4*)(g.cos_t + (size_t)m * 64 + (d & 63));
        sn = *(const f32x4*)(g.sin_t + (size_t)m * 64 + (d & 63));
      }
      float y[4];
      if constexpr (PAIR) {
        float y2[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x1 = acc[a][b][e], x2 = acc[a][(2 + b) % (2 * G::NW)][e];
          y[e] = is_v ? x1 : x1 * c[e] - x2 * sn[e];
          y2[e] = is_v ? x2 : x2 * c[e] + x1 * sn[e];
        }
        store(d, y);
        store(d + 64, y2);
      } else {
        if (is_v) {
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = acc[a][b][e];
        } else {
          const f32x4 other = *(const f32x4*)(s_x + ((wm * 2 * G::MW + a) * 16 + acc_col(lane)) * kLdx + (d ^ 64));
          const float sign = d < 64 ? -1.0f : 1.0f;     // y1 = x1 c - x2 s (columns < 64), y2 = x2 c + x1 s
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = acc[a][b][e] * c[e] + sign * other[e] * sn[e];
        }
        store(d, y);
      }
    }
  }
  };
  G::run(g.K / 32, lds, operands, finish);
}

// The row count is only needed for the stores (rows beyond it are stale rows, each affecting only its own output).
template <typename G>
__global__ void __launch_bounds__(G::THREADS) qkv_kernel(Plan p, QkvArgs g, int m_blocks) {
  extern __shared__ __align__(16) char lds[];
  const int id = xcd_flat(m_blocks * (g.Hq + 2 * g.Hkv));
  if (id >= 0) qkv_tile<G>(p, g, id % m_blocks * G::BM, id / m_blocks, lds);
}
// Rows of a workgroup's tile, with the time of one K tile in 0.01 us when a launch fills the CUs once.  The first stages, the epilogue
// and the launch's ragged start take as long as about 8 K tiles.  Measured, 16 heads, K 1536 / 36 heads, K 3584:
//   432 rows  32: 11.8 us, 64: 14.6, 128: 18.9     576 rows  32: 15.8, 64: 15.0, 128: 18.0
//   1024 rows 64: 15.5, 128: 18.5, 192: 22         2048 rows 64: 26.3, 128: 20.2, 192: 24     3700 rows 64: 48, 128: 33.5, 192: 46
//   64 rows   32: 24, 64: 28.5     288 rows 32: 35, 64: 26.6     816 rows 64: 50, 128: 36, 192: 41
//   1185 rows 64: 73, 128: 57, 192: 49             2048 rows 64: 119, 128: 86, 192: 90
// 128 and 192 rows are eight and twelve waves of two accumulator tiles and 80 KB, so that two workgroups share a CU and one's epilogue
// runs beside the other's loop.  In four waves of six tiles 192 rows take 54 us at 1185 rows, 57 at 3700; 256 rows in one workgroup
// per CU take 51 and 33, but a kernel that offers them has one workgroup per CU for every tile (128 rows: 62 and 39).
// Up to 640 rows the weights of the small tiles are in registers (StreamGemm).  Beyond, the tile is chosen on the device: a workgroup
// has twelve waves, of which four or eight leave at once where the tile has eight or four.  32 rows are for steps with few live rows.
typedef StreamGemm<1, 1, 4, 6> Few32;
typedef StreamGemm<2, 1, 4, 4> Few64;
typedef DmaGemm<1, 1, 1, 4, 8> Rows32;
typedef DmaGemm<1, 1, 2, 4, 6> Rows64;
typedef DmaGemm<1, 2, 4, 2, 5> Rows128;
typedef DmaGemm<1, 2, 6, 2, 4> Rows192;
__host__ __device__ inline int rows_cost(int M, int bm, int heads, int nk, int t) { return ((M + bm - 1) / bm * heads + kCUs - 1) / kCUs * (nk + 8) * t; }
constexpr int kRows32Tiles = 2 * kCUs;                   // most 32-row tiles that the launch of the device's choice is sized for
__host__ __device__ inline int pick_rows(int M, int heads, int nk, bool few, int& cost) {
  int bm = 128;
  cost = rows_cost(M, 128, heads, nk, 48);
  int c = rows_cost(M, 64, heads, nk, 37);
  if (c < cost) { bm = 64; cost = c; }
  c = rows_cost(M, 32, heads, nk, 31);
  if ((few || (M + 31) / 32 * heads <= kRows32Tiles) && c < cost) { bm = 32; cost = c; }
  c = rows_cost(M, 192, heads, nk, 72);
  if (!few && c < cost) { bm = 192; cost = c; }
  return bm;
}
constexpr int kFewRows = 640;
template <typename G> constexpr int qkv_lds() {
  constexpr int x = G::NW == 2 ? 0 : G::BM * kLdx * 4;  // exchange buffer
  return G::LDS_BYTES > x ? G::LDS_BYTES : x;
}
// Many rows: the rows of a tile from the step's row count.
__global__ void __launch_bounds__(Rows192::THREADS, 6) qkv_rows_kernel(Plan p, QkvArgs g) {
  extern __shared__ __align__(16) char lds[];
  const int M = min(p.n_rows[0], g.M_max), heads = g.Hq + 2 * g.Hkv;
  int cost;
  const int bm = pick_rows(M, heads, g.K / kBK, false, cost), m_blocks = (M + bm - 1) / bm;
  const int id = xcd_flat(m_blocks * heads);
  if (id < 0) return;
  const int m0 = id % m_blocks * bm, head = id / m_blocks;
  if (bm == 192) {
    qkv_tile<Rows192>(p, g, m0, head, lds);
    return;
  }
  if (bm == 32) {
    if (threadIdx.x < Rows32::THREADS) qkv_tile<Rows32>(p, g, m0, head, lds);
    return;
  }
  if (threadIdx.x >= 512) return;
  if (bm == 64) qkv_tile<Rows64>(p, g, m0, head, lds);
  else qkv_tile<Rows128>(p, g, m0, head, lds);
}
template <auto KERN, typename... Args>
void launch_one(int blocks, int threads, int lds, hipStream_t st, const Args&... args) {
  static bool done = false;                              // one per kernel
  if (!done) { (void)hipFuncSetAttribute((const void*)KERN, hipFuncAttributeMaxDynamicSharedMemorySize, lds); done = true; }
  hipLaunchKernelGGL(KERN, dim3((blocks + 7) / 8 * 8), dim3(threads), lds, st, args...);
}
}  // namespace

// Few rows have too few (rows, head) tiles for 256 CUs: the GEMM split over K and the rotary kernel behind it are then faster, although both
// together have more launches and latency (the 300 and the 440, in 0.01 us) and the rotary kernel reads the slabs and scatters K and V.  Steps
// measured with either route, 2048 cached tokens, us per layer, two kernels / fused:
//   7B shape    72 rows 138.9 / 143.8   189 rows 196.7 / 197.5   243 rows 212.5 / 215.9   288 rows 223.8 / 225.0   342 rows 277.2 / 276.8   387 rows 316.2 / 312.5
//   1.5B shape  63 rows 65.0 / 67.5   99 rows 72.5 / 73.1   135 rows 77.4 / 77.7   216 rows 88.6 / 88.1   288 rows 96.9 / 93.5   576 rows 132.3 / 128.5
bool qkv_rope_applies(const Shape& s, int M_max) {
  if (s.dtype != BS_BF16 || s.D != kD) return false;
  if (M_max > kFewRows) return true;
  int cost;
  pick_rows(M_max, s.Hq + 2 * s.Hkv, s.d / kBK, true, cost);
  return cost + 300 <= gemm_slab_time(M_max, s.Nqkv(), s.d) + 440 + M_max * s.Nqkv() / 5760;
}

void launch_qkv_rope(const Shape& s, const Plan& p, int M_max, const void* A, const void* Wp,
                     const float* cos_t, const float* sin_t, void* q_out, void* k_pages, void* v_pages, hipStream_t st) {
  const int heads = s.Hq + 2 * s.Hkv;
  const QkvArgs g{M_max, s.d, s.Hq, s.Hkv, (const f16*)A, (const f16*)Wp, cos_t, sin_t, (f16*)q_out, (f16*)k_pages, (f16*)v_pages};
  if (M_max > kFewRows) {
    constexpr int a = qkv_lds<Rows64>(), b = qkv_lds<Rows128>(), c = qkv_lds<Rows192>(), d = qkv_lds<Rows32>(), ab = a > b ? a : b, cd = c > d ? c : d, lds = ab > cd ? ab : cd;
    static_assert(Rows64::THREADS == 512 && Rows128::THREADS == 512 && 2 * lds <= 160 * 1024, "two workgroups per CU");
    const int tiles = (M_max + 63) / 64 * heads;
    launch_one<qkv_rows_kernel>(tiles > kRows32Tiles ? tiles : kRows32Tiles, Rows192::THREADS, lds, st, p, g);
    return;
  }
  int cost;
#define BS_QKV(G_) do { const int mb = (M_max + G_::BM - 1) / G_::BM; launch_one<qkv_kernel<G_>>(mb * heads, G_::THREADS, qkv_lds<G_>(), st, p, g, mb); } while (0)
  switch (pick_rows(M_max, heads, s.d / kBK, true, cost)) {
    case 32: BS_QKV(Few32); break;
    case 64: BS_QKV(Few64); break;
    default: BS_QKV(Rows128);
  }
#undef BS_QKV
}
