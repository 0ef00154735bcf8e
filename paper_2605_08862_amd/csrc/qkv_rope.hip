// QKV projection fused with the rotary embedding and the tentative KV append (bf16 models, head size 128).
//
//   [M, d] x [ (Hq + 2 Hkv) * 128, d ]^T, then per head: q and k rotated at the row's absolute position
//   (pairs (j, j + 64)), q stored as float16 rows (attention operand), k and v rounded to bf16 and written
//   into the slot's KV page in the page layout.
//
// One workgroup = rows x one or two heads.  The partner of column j (< 64) of a head is two weight tiles further: a wave's 32-row weight tile is put
// together from 16 columns and their 16 partners by the addresses, so that both halves of a rotation are in one lane.
// The float32 projection never goes to memory and q, k, v are rounded exactly once, after the rotation.
#include "gemm_dma.h"
#include <initializer_list>

namespace {
constexpr int kD = 128;

struct QkvArgs {
  int M_max, K, Hq, Hkv;
  const f16 *A, *Wp;
  const float *cos_t, *sin_t;
  f16 *q_out, *k_pages, *v_pages;
};

template <typename G>
__device__ __forceinline__ void qkv_tile(const Plan& p, const QkvArgs& g, int m0, int head0, char* lds) {
  static_assert(G::CT % 4 == 0, "a workgroup's columns are heads");
  const int wave = G::wave_id(), wm = wave / G::WN, wn = wave % G::WN;
  const int lane = threadIdx.x & 63, heads = g.Hq + 2 * g.Hkv;
  const size_t tile_bytes = (size_t)(g.K / kBK) * 4096;
  // position t: columns 16 (t % 4) .. and 16 (t % 4) + 64 .. of head head0 + t / 4
  auto operands = [&](typename G::Operands& op) {
    G::make_operands(op, g.A, g.M_max, [&](int r) { return min(m0 + r, g.M_max - 1); }, g.Wp,
                     [&](int t) { return (size_t)(min(head0 + t / 4, heads - 1) * 4 + (t >> 1 & 1)) * tile_bytes + (t & 1) * kWHalf; }, 2u * (uint32_t)tile_bytes, 0);
  };
  auto finish = [&](f32x4 (&acc)[2 * G::MW][2 * G::NW]) {
    const int M = min(p.n_rows[0], g.M_max);
    // a wave's columns lie in one head
    static_assert(G::NW <= 4 && 4 % G::NW == 0, "");
    const int head = head0 + wn * G::NW / 4;
    if (G::CT > 4 && head >= heads) return;             // an odd number of heads
    const bool is_v = head >= g.Hq + g.Hkv;
    int place[2 * G::MW];                               // k or v head: the rows' cache places
#pragma unroll
    for (int a = 0; a < 2 * G::MW; ++a) place[a] = head >= g.Hq ? p.row_kv[min(m0 + (wm * 2 * G::MW + a) * 16 + acc_col(lane), g.M_max - 1)] : 0;
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
      for (int b = 0; b < G::NW; ++b) {
        const int d = 16 * ((wn * G::NW + b) % 4) + acc_row(lane);
        f32x4 c = f32x4{1.f, 1.f, 1.f, 1.f}, sn = f32x4{0.f, 0.f, 0.f, 0.f};
        if (!is_v) {
          c = *(const f32x4*)(g.cos_t + (size_t)m * 64 + d);
          sn = *(const f32x4*)(g.sin_t + (size_t)m * 64 + d);
        }
        float y[4], y2[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x1 = acc[a][2 * b][e], x2 = acc[a][2 * b + 1][e];
          y[e] = is_v ? x1 : x1 * c[e] - x2 * sn[e];
          y2[e] = is_v ? x2 : x2 * c[e] + x1 * sn[e];
        }
        store(d, y);
        store(d + 64, y2);
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
// Up to 640 rows the tile follows from the row limit: time of one K tile in 0.01 us when a launch fills the CUs once; the first stages, the
// epilogue and the launch's ragged start take as long as about 8 K tiles.  Measured, 16 heads, K 1536 / 36 heads, K 3584:
//   432 rows  32: 11.8 us, 64: 14.6, 128: 18.9     576 rows  32: 15.8, 64: 15.0, 128: 18.0
//   64 rows   32: 24, 64: 28.5     288 rows 32: 35, 64: 26.6
// 128 rows are eight waves of two accumulator tiles and 80 KB, so that two workgroups share a CU and one's epilogue runs beside the other's loop; the
// weights of the small tiles are in registers (StreamGemm).
typedef StreamGemm<1, 1, 4, 6> Few32;
typedef StreamGemm<2, 1, 4, 4> Few64;
typedef DmaGemm<1, 2, 4, 2, 5> Rows128;
inline int pick_rows(int M, int heads, int nk, int& cost) {
  auto time = [&](int bm, int t) { return ((M + bm - 1) / bm * heads + kCUs - 1) / kCUs * (nk + 8) * t; };
  int bm = 128;
  cost = time(128, 48);
  int c = time(64, 37);
  if (c < cost) { bm = 64; cost = c; }
  c = time(32, 31);
  if (c < cost) { bm = 32; cost = c; }
  return bm;
}
constexpr int kFewRows = 640;
// More rows: four waves, weights in registers, two workgroups per CU, rows and heads of a tile from the step's row count (TileRule).  Rows128 reads 1.5 fragments
// from LDS per product and is bound by that, these 0.6 .. 1.  Times of the kernels by themselves, weights that no cache holds, 32 / 64 / 96 / 128 / 160 / 192 rows of a
// head and 128 rows of two heads (the rule's times are fitted to 20 .. 4352 rows of 8 shapes, from 12 heads and K 512 to 48 heads and K 4096):
//   16 heads, K 1536   128 rows 11.6 / 13.9 / 14.4 / 19.3 / 19.7 / 19.8 / 29.8 us   505 rows 11.8 / 13.9 / 14.8 / 19.2 / 18.4 / 22.1 / 28.9   824 rows 16.2 / 13.9 / 15.7 / 17.2 / 18.6 / 21.6 / 28.8
//                      1200 rows 24.6 / 19.2 / 17.2 / 18.2 / 21.0 / 22.9 / 29.7   2720 rows 46.9 / 34.1 / 30.5 / 36.2 / 34.6 / 27.7 / 32.5
//   36 heads, K 3584   128 rows 22.8 / 27.0 / 26.5 / 37.4 / 38.0 / 37.9 / 55.4 us   281 rows 35.0 / 25.3 / 32.1 / 28.8 / 38.9 / 37.7 / 50.1   720 rows 62.8 / 42.4 / 47.0 / 35.2 / 36.4 / 42.1 / 51.5
//                      1200 rows 101 / 64.4 / 53.3 / 58.9 / 63.4 / 48.0 / 53.2   1632 rows 124 / 84.3 / 73.4 / 64.7 / 69.0 / 75.9 / 57.0
typedef StreamGemm<3, 1, 4, 3> Many96;
typedef StreamGemm<4, 1, 4, 3> Many128;
typedef StreamGemm<5, 1, 4, 3> Many160;
typedef StreamGemm<6, 1, 4, 4, 2> Many192;
typedef StreamGemm<4, 2, 4, 2> Many128x2;
// The tile at the place of the step's choice; HP heads per workgroup.
template <typename G, int HP = G::CT / 4>
__device__ __forceinline__ void qkv_many_tile(const Plan& p, const QkvArgs& g, int M, char* lds) {
  const int m_blocks = (M + G::BM - 1) / G::BM, id = xcd_flat(m_blocks * ((g.Hq + 2 * g.Hkv + HP - 1) / HP));
  if (id >= 0) qkv_tile<G>(p, g, id % m_blocks * G::BM, id / m_blocks * HP, lds);
}
__global__ void __launch_bounds__(256, 2) qkv_many_kernel(Plan p, QkvArgs g, int at) {
  extern __shared__ __align__(16) char lds[];
  const int M = min(p.n_rows[0], g.M_max);
  switch (p.n_rows[at]) {                                // places in qkv_rope_rule's list
    case 0: qkv_many_tile<Few32>(p, g, M, lds); break;
    case 1: qkv_many_tile<Few64>(p, g, M, lds); break;
    case 2: qkv_many_tile<Many96>(p, g, M, lds); break;
    case 3: qkv_many_tile<Many128>(p, g, M, lds); break;
    case 4: qkv_many_tile<Many160>(p, g, M, lds); break;
    case 5: qkv_many_tile<Many192>(p, g, M, lds); break;
    default: qkv_many_tile<Many128x2>(p, g, M, lds);
  }
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
  pick_rows(M_max, s.Hq + 2 * s.Hkv, s.d / kBK, cost);
  return cost + 300 <= gemm_slab_time(M_max, s.Nqkv(), s.d) + 440 + M_max * s.Nqkv() / 5760;
}

TileRule qkv_rope_rule(const Shape& s, int M_max) {
  const int heads = s.Hq + 2 * s.Hkv, pairs = (heads + 1) / 2;
  TileRule r;
  if (s.dtype != BS_BF16 || s.D != kD || M_max <= kFewRows) return r;
  // A further round also costs the change of workgroups, about two K tiles: counted without it, up to 6 K tiles took too many rounds (10 heads, K 256,
  // 2176 rows: 32 rows 10.1 us, 96 rows, taken now, 8.5; tiles taken with K below 512 were 3.4 % from the fastest, now 0.5; from 512 on 0.14 and 0.20).
  r = TileRule{CHOICE_QKV, 0, s.d / kBK + 2, 7, {{32, heads, 27, 246}, {64, heads, 33, 309}, {96, heads, 44, 361}, {128, heads, 51, 483}, {160, heads, 61, 445}, {192, heads, 61, 814},
                                                {128, pairs, 73, 1071}}};
  r.size_grid(M_max);
  return r;
}

void launch_qkv_rope(const Shape& s, const Plan& p, int M_max, const TileRule& rule, const void* A, const void* Wp,
                     const float* cos_t, const float* sin_t, void* q_out, void* k_pages, void* v_pages, hipStream_t st) {
  const int heads = s.Hq + 2 * s.Hkv;
  const QkvArgs g{M_max, s.d, s.Hq, s.Hkv, (const f16*)A, (const f16*)Wp, cos_t, sin_t, (f16*)q_out, (f16*)k_pages, (f16*)v_pages};
  constexpr auto most = [](std::initializer_list<int> v) { int m = 0; for (int x : v) m = x > m ? x : m; return m; };
  if (rule.at) {
    constexpr int lds = most({Few32::LDS_BYTES, Few64::LDS_BYTES, Many96::LDS_BYTES, Many128::LDS_BYTES, Many160::LDS_BYTES, Many192::LDS_BYTES, Many128x2::LDS_BYTES});
    static_assert(2 * lds <= 160 * 1024, "two workgroups per CU");
    launch_one<qkv_many_kernel>(rule.grid, 256, lds, st, p, g, rule.at);
    return;
  }
  int cost;
#define BS_QKV(G_) do { const int mb = (M_max + G_::BM - 1) / G_::BM; launch_one<qkv_kernel<G_>>(mb * heads, G_::THREADS, G_::LDS_BYTES, st, p, g, mb); } while (0)
  switch (pick_rows(M_max, heads, s.d / kBK, cost)) {
    case 32: BS_QKV(Few32); break;
    case 64: BS_QKV(Few64); break;
    default: BS_QKV(Rows128);
  }
#undef BS_QKV
}
