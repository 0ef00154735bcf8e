// Decoder layer for steps of few packed rows (at most 32: one to a few sequences, or plain decoding of a small batch).
//
// With so few rows a layer is bound by streaming its weights once, and the first obstacle is latency: 1.5B shape, nine
// rows, the weights of a layer are 94 MB = 15 us at the rate a streaming read reaches, and the tiled GEMMs took 62 us
// over six launches (normalisation, QKV, O, normalisation, gate/up, down), each with a pipeline fill, a tail and slabs.
// Here a layer is five launches besides attention (QKV, O, normalisation, gate/up, down), shaped for that:
//   * one workgroup = one or two 32-row weight tiles, its waves split K between them: every wave streams its own part of
//     the packed weights HBM -> registers, one contiguous KiB per load, and the partial tiles meet in LDS at the end.
//     Where that gives fewer workgroups than CUs, K is also split across workgroups and the last one to arrive adds the
//     partial tiles (publish_arrival: no slabs for another kernel to sum);
//   * activations are kept in MFMA fragment order too (act_index, h_frag_index), so a fragment is one contiguous
//     KiB from L2 straight into operand registers: no LDS staging, no swizzle, no barrier in the main loop;
//   * O and down add their result to the residual themselves and write the sum of squares of their 32 columns per row.  QKV
//     adds those up and normalises the residual as it reads it; in front of gate/up the normalisation is one small
//     element-wise kernel.  (A kernel costs about 2.4 us of launch besides its work.  In QKV the extra work is hidden, 1.5B shape,
//     launch subtracted: 8.1 us against 6.1 + 4.0.  Gate/up has a wave per tile and every wave would convert the whole residual: 7B shape, staged
//     in LDS once per workgroup, 56 us against 45 + 4.)
// Loads are issued in the order in which they are waited for (the memory counter is in order).
// A CU draws about 54 GB/s, so what it reads is what it costs, and a fragment of 32 rows is as many bytes as one of the weights: lanes
// of rows beyond the row limit read the last row again, which costs no line of its own (9 rows: half of the
// bytes; 1.5B shape, gate/up 14.9 -> 14.0 us, O and down 9.3 -> 8.6 on average; cutting K over more waves than now takes gate/up to 16).
#include "gemm_mfma.h"
#include <type_traits>

namespace {
__device__ __forceinline__ float silu_fast(float x) { return x * __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }

// The partial tiles of the workgroup's WS waves are summed through LDS.  After collect(), item i4 - accumulator registers
// 4 i4 .. 4 i4 + 3 of the tile, all 64 lanes - is the sum over s < HALF of s_part[s][i4][lane]; it is summed by whichever
// wave handles the item (sum_item).  The upper half of the waves first hands its tiles to the lower half.  The order of
// the sums is fixed.
template <int WS>
struct WaveSum {
  static constexpr int HALF = WS / 2;
  static constexpr int LDS_BYTES = HALF * 4096;
  __device__ static __forceinline__ void put(char* lds, int slot, const f32x16& acc, int lane) {
    f32x4* s = (f32x4*)lds;
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) s[(slot * 4 + i4) * 64 + lane] = f32x4{acc[4 * i4], acc[4 * i4 + 1], acc[4 * i4 + 2], acc[4 * i4 + 3]};
  }
  __device__ static __forceinline__ void collect(char* lds, f32x16& acc, int wave, int lane) {
    if (wave >= HALF) put(lds, wave - HALF, acc, lane);
    __syncthreads();
    if (wave < HALF) {
      const f32x4* s = (const f32x4*)lds;
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const f32x4 v = s[(wave * 4 + i4) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[4 * i4 + e] += v[e];
      }
      put(lds, wave, acc, lane);                         // its own slot: nobody else reads it before the barrier
    }
    __syncthreads();
  }
  __device__ static __forceinline__ f32x4 sum_item(const char* lds, int i4, int lane) {
    const f32x4* s = (const f32x4*)lds;
    f32x4 v = s[i4 * 64 + lane];
#pragma unroll
    for (int w = 1; w < HALF; ++w) {
      const f32x4 u = s[(w * 4 + i4) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += u[e];
    }
    return v;
  }
};

enum { SK_QKV = 0, SK_RESID = 1 };

struct QkvOut {        // SK_QKV: where the rotated q and the appended k / v go
  int Hq, Hkv;
  const float *cos_t, *sin_t;
  f16 *q, *k_pages, *v_pages;
};
struct NormIn {        // SK_QKV: float32 residual (fragment order), sums of squares [parts][32] and the gain
  const float *h, *ssq, *gain;
  int parts;
  float eps;
};
// eight residual elements k .. k + 7 of a row -> one float16 operand fragment element
__device__ __forceinline__ f16x8 norm8(const f32x4 a, const f32x4 b, const f32x4 ga, const f32x4 gb, float inv, int32_t* status) {
  const f16x4 lo = to_f16x4_guarded(a[0] * inv * ga[0], a[1] * inv * ga[1], a[2] * inv * ga[2], a[3] * inv * ga[3], status);
  const f16x4 hi = to_f16x4_guarded(b[0] * inv * gb[0], b[1] * inv * gb[1], b[2] * inv * gb[2], b[3] * inv * gb[3], status);
  return f16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
}
// Workgroup ids are dealt round-robin to the 8 XCDs; every XCD takes a contiguous range of the n pieces of work, so that its
// address translations and its L2 see one stretch of the weights.  -1: no work.
__device__ __forceinline__ int xcd_range(int n) {
  const int per = (n + 7) / 8, i = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
  return (int)(blockIdx.x / 8) < per && i < n ? i : -1;
}
// One 32-row weight tile x 32 activation rows x K / n_split, K split over eight waves.  The tile of a unit is
//   SK_RESID  32 rows of the matrix (output columns);
//   SK_QKV    16 columns of a head and the 16 columns 64 further (a rotation's partners), so that both land in the same lane,
//             in registers i and i + 8: the halves come from two packed tiles by the lanes' addresses (a load
//             instruction then reads four 256-byte runs).
// SK_QKV takes the float32 residual and normalises it, SK_RESID float16 rows in fragment order.
template <int KIND>
__global__ void __launch_bounds__(512, 2)
skinny_kernel(Plan p, int rows, int K, const f16* __restrict__ X, NormIn nin, const f16* __restrict__ Wp, float* h, float* __restrict__ ssq_out, int d,
              QkvOut qo, int units, int n_split, float* __restrict__ part, int32_t* __restrict__ counters) {
  constexpr int WS = 8;
  using R = WaveSum<WS>;
  constexpr bool NORM = KIND == SK_QKV;
  constexpr int RING = 3;                               // weight tiles in flight
  constexpr int RX = NORM ? 1 : RING;                   // activation tiles in flight (residual: two and three measured slower)
  constexpr int GROUPS = 64 * WS / 32;
  extern __shared__ __align__(16) char lds[];
  __shared__ float s_ss[GROUPS][32];
  __shared__ int s_last;
  float* s_gain = (float*)(lds + R::LDS_BYTES);         // NORM: [K]
  const int work = xcd_range(units * n_split);
  if (work < 0) return;
  const int tid = threadIdx.x, lane = tid & 63, ln = lane & 31, lg = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nk = K / kBK;
  const int unit = work / n_split, split = work % n_split;
  const int sw = split * WS + wave;                     // K is cut into n_split * WS ranges
  const int kt0 = nk * sw / (n_split * WS), kt1 = nk * (sw + 1) / (n_split * WS);
  const int half = unit & 1;                            // SK_QKV: upper or lower 16 rows of the tile pair
  const int tile0 = KIND == SK_RESID ? unit : (unit >> 2) * 4 + ((unit >> 1) & 1);
  uint32_t w_lane = lane * 16;
  if (KIND == SK_QKV) {
    w_lane = (lg * 32 + half * 16 + (ln & 15)) * 16;
    if (ln >= 16) w_lane += 2u * nk * (kWBlock * 2);
  }
  const int M = min(p.n_rows[0], 32);
  if (NORM) {                                           // sums of squares and the gain first (waited for first), then the streams
    float ss = 0.f;
    for (int i = tid >> 5; i < nin.parts; i += GROUPS) ss += nin.ssq[(size_t)i * 32 + ln];
    for (int i = tid * 4; i < K; i += 64 * WS * 4) *(f32x4*)(s_gain + i) = *(const f32x4_u*)(nin.gain + i);
    s_ss[tid >> 5][ln] = ss;
  }
  u32x4 w[RING][4], x[RX][NORM ? 8 : 4];                // NORM: [K-step][half] of the residual
  // Buffer loads: one lane offset and a scalar offset address everything.  Every request of the loop is unconditional (under a
  // condition the compiler would have to wait for all outstanding loads); beyond the wave's range its last tile is read again.
  const wt_buf wr = wt_buffer(Wp + (size_t)tile0 * nk * kWBlock), xr = wt_buffer(NORM ? (const void*)nin.h : (const void*)X);
  const int kl = max(kt1 - 1, 0);
  const uint32_t x_lane = (lg * 32 + min(ln, rows - 1)) * 16;
  auto load_x = [&](auto stage_tag, int kt) {
    constexpr int ST = decltype(stage_tag)::value, N = NORM ? 8 : 4;
    const int so = min(kt, kl) * (N * 1024);
#pragma unroll
    for (int s = 0; s < N; ++s) x[ST][s] = __builtin_amdgcn_raw_buffer_load_b128(xr, (int)x_lane + (s & 3) * 1024, so + (s >> 2) * 4096, 0);
  };
  auto load_w = [&](auto stage_tag, int kt) {
    constexpr int ST = decltype(stage_tag)::value;
    const int so = min(kt, kl) * (kWBlock * 2);
#pragma unroll
    for (int s = 0; s < 4; ++s) w[ST][s] = __builtin_amdgcn_raw_buffer_load_b128(wr, (int)w_lane + s * 1024, so, 0);
  };
  constexpr std::integral_constant<int, 0> S0{};
  constexpr std::integral_constant<int, 1> S1{};
  constexpr std::integral_constant<int, 2> S2{};
  load_x(S0, kt0);
  load_w(S0, kt0);
  if constexpr (!NORM) load_x(S1, kt0 + 1);
  load_w(S1, kt0 + 1);
  if constexpr (!NORM) load_x(S2, kt0 + 2);
  load_w(S2, kt0 + 2);
  // what the epilogue needs besides the products is looked up ahead
  size_t pbase = 0;                                     // SK_QKV, k and v heads: the row's cache slot
  int tok = 0;
  float inv = 0.f;
  f32x4 h_old = f32x4{0.f, 0.f, 0.f, 0.f};              // SK_RESID: the residual this wave will add to
  f32x4* h_at = nullptr;
  f32x4 rot_c = f32x4{0.f, 0.f, 0.f, 0.f}, rot_s = rot_c;   // SK_QKV: the rotation
  // SK_QKV: the four columns dc .. dc + 3 (and their partners dc + 64 ..) that this wave stores, if it stores any
  const int dc = 32 * ((unit >> 1) & 1) + half * 16 + 8 * (wave & 1) + 4 * lg;
  if constexpr (NORM) {
    rot_c = *(const f32x4*)(qo.cos_t + (size_t)min(ln, rows - 1) * 64 + dc);
    rot_s = *(const f32x4*)(qo.sin_t + (size_t)min(ln, rows - 1) * 64 + dc);
    if ((unit >> 2) >= qo.Hq && ln < M) {
      const int place = p.row_kv[ln];
      tok = place & (kPage - 1);
      pbase = (size_t)(place / kPage) * kv_page_elems(qo.Hkv, 128);
    }
    __syncthreads();
    float ss = 0.f;
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) ss += s_ss[g][ln];
    // rows beyond the count: their residual is zero (embed_frag_kernel) and stays zero
    inv = ln < M ? 1.0f / sqrtf(ss / (float)K + nin.eps) : 0.f;
  } else {
    h_at = (f32x4*)(h + h_frag_index(ln, unit * 32 + 8 * (wave & 3) + 4 * lg, d / kBK));
    h_old = *h_at;
  }
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;

  // one K tile, then the requests that take the place of what it used
  auto body = [&](auto stage_tag, int kt) {
    constexpr int ST = decltype(stage_tag)::value;
    if constexpr (NORM) {
      f16x8 xs[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const float* gp = s_gain + kt * kBK + lg * 32 + s * 8;
        xs[s] = norm8(__builtin_bit_cast(f32x4, x[0][2 * s]), __builtin_bit_cast(f32x4, x[0][2 * s + 1]), *(const f32x4*)gp,
                      *(const f32x4*)(gp + 4), inv, p.status);
      }
      __builtin_amdgcn_sched_barrier(0);
      load_x(S0, kt + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(w[ST][s]), xs[s], acc, 0, 0, 0);
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(w[ST][s]), as_f16x8(x[ST % RX][s]), acc, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      load_x(stage_tag, kt + RING);
    }
    __builtin_amdgcn_sched_barrier(0);
    load_w(stage_tag, kt + RING);
    __builtin_amdgcn_sched_barrier(0);
  };
  int kt = kt0;
  for (; kt + 3 <= kt1; kt += 3) { body(S0, kt); body(S1, kt + 1); body(S2, kt + 2); }
  if (kt < kt1) body(S0, kt);
  if (kt + 1 < kt1) body(S1, kt + 1);

  // ---- sum over the waves, then over the K splits
  R::collect(lds, acc, wave, lane);
  const wt_buf pb = wt_buffer(part + (size_t)unit * n_split * 1024);               // [split][i4][lane] x 4
  if (n_split > 1) {
    if (wave < 4) wt_store4(pb, ((split * 4 + wave) * 64 + lane) * 16, R::sum_item(lds, wave, lane));
    if (!publish_arrival(counters + unit, n_split, &s_last)) return;
  }
  auto total = [&](int i4) {                            // four consecutive columns of a row
    if (n_split == 1) return R::sum_item(lds, i4, lane);
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int sp0 = 0; sp0 < n_split; sp0 += 4) {         // four splits' loads in flight, summed in order
      f32x4 u4[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) u4[u] = wt_load4(pb, ((min(sp0 + u, n_split - 1) * 4 + i4) * 64 + lane) * 16);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (sp0 + u < n_split) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += u4[u][e];
        }
    }
    return v;
  };

  const int m = ln;
  if constexpr (KIND == SK_RESID) {
    if (wave < 4) {
      f32x4 v = total(wave);
      float ss = 0.f;
      if (m < M) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[e] += h_old[e]; ss += v[e] * v[e]; }
        *h_at = v;
      }
      ss += __shfl_xor(ss, 32);
      if (lg == 0) s_ss[wave][m] = ss;
    }
    __syncthreads();
    if (tid < 32) ssq_out[(size_t)unit * 32 + tid] = s_ss[0][tid] + s_ss[1][tid] + s_ss[2][tid] + s_ss[3][tid];
  } else if (wave < 2) {                                 // i4 = 0, 1: first half of the tile; i4 + 2: its partner
    constexpr int D = 128;
    const f32x4 a = total(wave), b = total(wave + 2);
    if (m >= M) return;
    const int head = unit >> 2;
    f32x4 y1 = a, y2 = b;
    if (head < qo.Hq + qo.Hkv) {
#pragma unroll
      for (int e = 0; e < 4; ++e) { y1[e] = a[e] * rot_c[e] - b[e] * rot_s[e]; y2[e] = b[e] * rot_c[e] + a[e] * rot_s[e]; }
    }
    if (head < qo.Hq) {
      f16* dst = qo.q + ((size_t)m * qo.Hq + head) * D + dc;
      *(f16x4*)dst = to_f16x4_guarded(y1[0], y1[1], y1[2], y1[3], p.status);
      *(f16x4*)(dst + 64) = to_f16x4_guarded(y2[0], y2[1], y2[2], y2[3], p.status);
    } else {
      // bf16-rounded values in float16 encoding (page format)
      const f16x4 v1 = to_f16x4_guarded((float)(bf16)y1[0], (float)(bf16)y1[1], (float)(bf16)y1[2], (float)(bf16)y1[3], p.status);
      const f16x4 v2 = to_f16x4_guarded((float)(bf16)y2[0], (float)(bf16)y2[1], (float)(bf16)y2[2], (float)(bf16)y2[3], p.status);
      if (head < qo.Hq + qo.Hkv) {
        *(f16x4*)(qo.k_pages + pbase + k_index_bf16(D, head - qo.Hq, tok, dc)) = v1;
        *(f16x4*)(qo.k_pages + pbase + k_index_bf16(D, head - qo.Hq, tok, dc + 64)) = v2;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          qo.v_pages[pbase + v_index_bf16(D, head - qo.Hq - qo.Hkv, tok, dc + e)] = v1[e];
          qo.v_pages[pbase + v_index_bf16(D, head - qo.Hq - qo.Hkv, tok, dc + 64 + e)] = v2[e];
        }
      }
    }
  }
}

// Gate/up projection + SwiGLU.  A unit is the gate tile and the up tile of 32 features, and ONE wave streams it over the
// whole K, three K tiles (24 KiB of weights) ahead: no sum over waves, no LDS, no barrier, and because every unit of the
// launch is resident at once and draws the same share of the memory bandwidth, no tail.
__global__ void __launch_bounds__(256, 2)
skinny_glu_kernel(Plan p, int rows, int K, const f16* __restrict__ X, const f16* __restrict__ Wp, int units, f16* __restrict__ act) {
  constexpr int RING = 3;
  const int waves = blockDim.x >> 6;
  const int wg = xcd_range((units + waves - 1) / waves);
  if (wg < 0) return;
  const int lane = threadIdx.x & 63, ln = lane & 31, lg = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int unit = wg * waves + wave, nk = K / kBK;
  if (unit >= units) return;
  const wt_buf xr = wt_buffer(X), w_gate = wt_buffer(Wp + (size_t)unit * nk * kWBlock), w_up = wt_buffer(Wp + (size_t)(unit + units) * nk * kWBlock);
  const uint32_t x_lane = (lg * 32 + min(ln, rows - 1)) * 16;
  u32x4 w[RING][2][4], x[RING][4];
  auto load = [&](auto stage_tag, int kt) {
    constexpr int ST = decltype(stage_tag)::value;
    const int so = min(kt, nk - 1) * (kWBlock * 2);     // unconditional, as above
#pragma unroll
    for (int s = 0; s < 4; ++s) x[ST][s] = __builtin_amdgcn_raw_buffer_load_b128(xr, (int)x_lane + s * 1024, so, 0);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      w[ST][0][s] = __builtin_amdgcn_raw_buffer_load_b128(w_gate, lane * 16 + s * 1024, so, 0);
      w[ST][1][s] = __builtin_amdgcn_raw_buffer_load_b128(w_up, lane * 16 + s * 1024, so, 0);
    }
  };
  constexpr std::integral_constant<int, 0> S0{};
  constexpr std::integral_constant<int, 1> S1{};
  constexpr std::integral_constant<int, 2> S2{};
  load(S0, 0);
  load(S1, 1);
  load(S2, 2);
  const int M = min(p.n_rows[0], 32);
  f32x16 acc[2];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[0][i] = acc[1][i] = 0.f;
  auto body = [&](auto stage_tag, int kt) {
    constexpr int ST = decltype(stage_tag)::value;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
        acc[ni] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(w[ST][ni][s]), as_f16x8(x[ST][s]), acc[ni], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    load(stage_tag, kt + RING);
    __builtin_amdgcn_sched_barrier(0);
  };
  int kt = 0;
  for (; kt + 3 <= nk; kt += 3) { body(S0, kt); body(S1, kt + 1); body(S2, kt + 2); }
  if (kt < nk) body(S0, kt);
  if (kt + 1 < nk) body(S1, kt + 1);
  if (ln >= M) return;
#pragma unroll
  for (int i4 = 0; i4 < 4; ++i4) {
    float y[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) y[j] = silu_fast(acc[0][4 * i4 + j]) * acc[1][4 * i4 + j];
    *(f16x4*)(act + act_index(ln, unit * 32 + 8 * i4 + 4 * lg, kSkinnyRows)) = to_f16x4_guarded(y[0], y[1], y[2], y[3], p.status);
  }
}

// RMSNorm of the fragment-ordered residual into float16 fragments, one workgroup per K tile.
__global__ void __launch_bounds__(256) norm_frag_kernel(Plan p, int K, float eps, const float* __restrict__ h,
                                                        const float* __restrict__ ssq, int parts, const float* __restrict__ gain,
                                                        f16* __restrict__ out) {
  __shared__ float s_ss[8][32];
  const int kt = blockIdx.x, tid = threadIdx.x, lane = tid & 63, s = tid >> 6, ln = lane & 31, lg = lane >> 5;
  const f32x4* hp = (const f32x4*)h + ((size_t)kt * 8 + 2 * s) * 64 + lane;
  const f32x4 a = hp[0], b = hp[64];
  const float* gp = gain + kt * kBK + lg * 32 + s * 8;
  const f32x4 ga = *(const f32x4_u*)gp, gb = *(const f32x4_u*)(gp + 4);
  float ss = 0.f;
  for (int i = tid >> 5; i < parts; i += 8) ss += ssq[(size_t)i * 32 + ln];
  s_ss[tid >> 5][ln] = ss;
  __syncthreads();
  ss = 0.f;
#pragma unroll
  for (int g = 0; g < 8; ++g) ss += s_ss[g][ln];
  // rows beyond the count: their residual is zero (embed_frag_kernel) and stays zero
  const float inv = ln < p.n_rows[0] ? 1.0f / sqrtf(ss / (float)K + eps) : 0.f;
  *(f16x8*)(out + ((size_t)kt * 4 + s) * 512 + lane * 8) = norm8(a, b, ga, gb, inv, p.status);
}

template <int KIND>
void launch_t(int rows, int units, int n_split, int K, const Shape& s, const Plan& p, const void* X, const NormIn& nin, const void* W, float* h, float* ssq,
              const QkvOut& qo, const SkinnyBufs& sk, hipStream_t st) {
  const int lds = WaveSum<8>::LDS_BYTES + (KIND == SK_QKV ? K * 4 : 0);
  hipLaunchKernelGGL((skinny_kernel<KIND>), dim3((units * n_split + 7) / 8 * 8), dim3(512), lds, st, p, rows, K, (const f16*)X, nin, (const f16*)W, h, ssq, s.d, qo, units, n_split, sk.part, sk.counters);
}

// Token embedding into the fragment-ordered residual; rows beyond the step's count become zero rows.  Also the row's sum
// of squares (part 0) and rotary table entries.
__global__ void __launch_bounds__(256) embed_frag_kernel(Plan p, KvView kv, int d, const bf16* __restrict__ embed, float* __restrict__ h,
                                                         float* __restrict__ ssq, int D, const double* __restrict__ inv_freq,
                                                         float* __restrict__ cos_t, float* __restrict__ sin_t) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4), aligned(2)));   // a caller's array: aligned to its elements only
  __shared__ float red[4];
  const int r = blockIdx.x;
  const bool live = r < p.n_rows[0];
  const bf16* src = embed + (live ? (size_t)p.row_tok[r] * d : 0);
  float ss = 0.f;
  for (int i = threadIdx.x * 4; i < d; i += 1024) {
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
    if (live) {
      const bf16x4 e = *(const bf16x4*)(src + i);
#pragma unroll
      for (int j = 0; j < 4; ++j) { v[j] = (float)e[j]; ss += v[j] * v[j]; }
    }
    *(f32x4*)(h + h_frag_index(r, i, d / kBK)) = v;
  }
  if (!live) return;
  if (threadIdx.x == 255) row_place(p, kv, r);
  if ((int)threadIdx.x < D / 2) rope_angle(p, r, threadIdx.x, D / 2, inv_freq, cos_t, sin_t);
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0) ssq[r] = red[0] + red[1] + red[2] + red[3];
}

// Final RMSNorm: fragment-ordered residual -> float16 rows in chunk order (operand of the LM head).
__global__ void __launch_bounds__(256) final_norm_frag_kernel(Plan p, int d, float eps, const float* __restrict__ h,
                                                              const float* __restrict__ ssq, int ssq_parts,
                                                              const float* __restrict__ gain, f16* __restrict__ out, int ld) {
  __shared__ float red[4];
  const int r = blockIdx.x;
  if (r >= p.n_rows[0]) return;
  float ss = 0.f;
  for (int i = threadIdx.x; i < ssq_parts; i += 256) ss += ssq[(size_t)i * 32 + r];
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float inv = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / (float)d + eps);
  for (int i = threadIdx.x * 4; i < d; i += 1024) {
    const f32x4 v = *(const f32x4*)(h + h_frag_index(r, i, d / kBK)), g = *(const f32x4_u*)(gain + i);
    *(f16x4*)(out + act_index(r, i, ld)) = to_f16x4_guarded(v[0] * inv * g[0], v[1] * inv * g[1], v[2] * inv * g[2], v[3] * inv * g[3], p.status);
  }
}
}  // namespace

bool skinny_applies(const Shape& s, int M_max) { return s.dtype == BS_BF16 && s.D == 128 && M_max <= kSkinnyRows && s.d <= 8192; }

void launch_skinny_embed(const Shape& s, const Plan& p, const KvView& kv, const void* embed, float* h, float* ssq, const double* inv_freq,
                         float* cos_t, float* sin_t, hipStream_t st) {
  hipLaunchKernelGGL(embed_frag_kernel, dim3(kSkinnyRows), dim3(256), 0, st, p, kv, s.d, (const bf16*)embed, h, ssq, s.D,
                     inv_freq, cos_t, sin_t);
}
void launch_skinny_final_norm(const Shape& s, const Plan& p, int M_max, const float* h, const float* ssq, const float* gain,
                              void* out, hipStream_t st) {
  hipLaunchKernelGGL(final_norm_frag_kernel, dim3(M_max), dim3(256), 0, st, p, s.d, s.eps, h, ssq, s.d / 32, gain, (f16*)out, M_max);
}
void launch_skinny_qkv(const Shape& s, const Plan& p, int M_max, const float* h, const float* ssq, int ssq_parts,
                       const float* gain, const void* W, const float* cos_t, const float* sin_t, void* q_out, void* k_pages, void* v_pages, const SkinnyBufs& sk, hipStream_t st) {
  const QkvOut qo{s.Hq, s.Hkv, cos_t, sin_t, (f16*)q_out, (f16*)k_pages, (f16*)v_pages};
  launch_t<SK_QKV>(M_max, 4 * (s.Hq + 2 * s.Hkv), 1, s.d, s, p, nullptr, NormIn{h, ssq, gain, ssq_parts, s.eps}, W, nullptr, nullptr, qo, sk, st);
}
void launch_skinny_gate_up(const Shape& s, const Plan& p, int M_max, const float* h, const float* ssq, int ssq_parts, const float* gain, void* a,
                           const void* W, void* act, hipStream_t st) {
  hipLaunchKernelGGL(norm_frag_kernel, dim3(s.d / kBK), dim3(256), 0, st, p, s.d, s.eps, h, ssq, ssq_parts, gain, (f16*)a);
  const int units = s.F / 32;
  int waves = (units + 255) / 256;                       // one workgroup per CU while the units last
  if (waves > 4) waves = 4;
  hipLaunchKernelGGL(skinny_glu_kernel, dim3(((units + waves - 1) / waves + 7) / 8 * 8), dim3(64 * waves), 0, st, p, M_max, s.d, (const f16*)a,
                     (const f16*)W, units, (f16*)act);
}
void launch_skinny_resid(const Shape& s, const Plan& p, int M_max, int K, const void* X, const void* W, float* h, float* ssq,
                         const SkinnyBufs& sk, hipStream_t st) {
  // A CU draws at most ~54 GB/s from HBM (measured: 48 streaming workgroups reach 2.6 TB/s, 128 reach 5.5), so K is also
  // split across workgroups where few column tiles meet a long K (1.5B shape, down projection: 48 tiles of 573 KB); the
  // last-arriver merge costs about 4 us of latency, which is what 200 KB per CU take
  const int units = s.d / 32, nk = K / kBK;
  int n_split = nk >= 96 ? (192 + units / 2) / units : 1;
  if (n_split > kMaxGemmSplit) n_split = kMaxGemmSplit;
  if (n_split < 1) n_split = 1;
  launch_t<SK_RESID>(M_max, units, n_split, K, s, p, X, NormIn{}, W, h, ssq, QkvOut{}, sk, st);
}
