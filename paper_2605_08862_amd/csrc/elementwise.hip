// Token-wise, bandwidth-trivial kernels of the verify pass (Sec. 3.3 "token-wise operations"):
// embedding gather, RMSNorm, rotary + tentative KV append, and the cache import/export copies.
// Each moves O(M*d) bytes per layer (<1 % of a step's traffic); they are written for clarity and
// coalesced row access, one workgroup per packed row.
#include "common.h"
#include <type_traits>

constexpr int kRuleGroups = 5;
// Token embedding of every packed row and, in the same launch, the row's rotary cos / sin table entries (the table
// [M_max][D/2] is shared by all layers of the step).
template <typename T>
__global__ void __launch_bounds__(256) embed_kernel(Plan p, KvView kv, int M_max, StepRules rules, int d, const T* __restrict__ embed, float* __restrict__ h,
                                                    int D, const double* __restrict__ inv_freq,
                                                    float* __restrict__ cos_t, float* __restrict__ sin_t) {
  int r = blockIdx.x;
  if (r >= M_max) {                                      // kRuleGroups more workgroups: one rule each
    if (threadIdx.x > 0) return;
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (r == M_max + i && rules.slab[i].at) p.n_rows[rules.slab[i].at] = pack_choice(rules.slab[i].choice(p.n_rows[0]));
    if (r == M_max + 3 && rules.qkv.at) p.n_rows[rules.qkv.at] = rules.qkv.choice(p.n_rows[0]);
    if (r == M_max + 4 && rules.glu.at) p.n_rows[rules.glu.at] = rules.glu.choice(p.n_rows[0]);
    return;
  }
  if (r >= p.n_rows[0]) return;
  const T* src = embed + (size_t)p.row_tok[r] * d;
  float* dst = h + (size_t)r * d;
  for (int i = threadIdx.x; i < d; i += blockDim.x) dst[i] = to_f32<T>(src[i]);
  if (threadIdx.x == 255) row_place(p, kv, r);
  if ((int)threadIdx.x < D / 2) rope_angle(p, r, threadIdx.x, D / 2, inv_freq, cos_t, sin_t);
}

__device__ __forceinline__ float block_sum_256(float v, float* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// out[r] = h[r] * gain / sqrt(mean(h[r]^2) + eps), float32 in; out is the GEMM operand type
// (float32 for float32 models: row-major; float16 for bf16 models: chunk order with ld rows).
// With n_slabs > 0 the row first absorbs the K-split slabs of the preceding residual projection:
// h[r] += sum_s slabs[s][r] (the updated residual is written back).
// One workgroup per row; the row (d <= 1024 * NV floats) stays in registers between the sum of squares
// and the scaling, so every operand is read once and the kernel has a single barrier.
template <typename T> struct Vec4;
template <> struct Vec4<float> { typedef float type __attribute__((ext_vector_type(4))); };
template <> struct Vec4<f16> { typedef _Float16 type __attribute__((ext_vector_type(4))); };

template <typename T, int NV, int NT = 256>
__global__ void __launch_bounds__(NT) rmsnorm_kernel(Plan p, int d, float eps, float* __restrict__ h,
                                                      const float* __restrict__ slabs, SlabCount rule, size_t slab_stride,
                                                      const float* __restrict__ gain, T* __restrict__ out, int ld) {
  constexpr bool CHUNKS = std::is_same<T, f16>::value;
  __shared__ float red[NT / 64];
  // Workgroup ids are dealt round-robin to the 8 XCDs.  In chunk order a 128-byte line holds eight rows' chunks: eight consecutive
  // rows go to one XCD, whose L2 then puts the line together.
  const int id = blockIdx.x, r = CHUNKS ? (id & ~63) + (id & 7) * 8 + ((id >> 3) & 7) : id;
  if (CHUNKS && r >= ld) return;
  const int n_rows = p.n_rows[0];                        // a fixed slab count leaves this wait until the row's loads are in flight
  // With the device rule the slab count needs the row count before the first slab load anyway, so the rows beyond
  // the count leave here instead of loading what they never store (a step with 1185 of at most 2176 rows fetched
  // 123 MB per launch for 68 MB of live operands).
  if (rule.at != 0 && r >= n_rows) return;
  const int n_slabs = rule.of(p.n_rows);
  typedef float f4 __attribute__((ext_vector_type(4)));
  float* x = h + (size_t)r * d;
  const float* sl = slabs + (size_t)r * d;
  f4 v[NV], gn[NV];
#pragma unroll
  for (int it = 0; it < NV; ++it) {
    const int i = (it * NT + threadIdx.x) * 4;          // d is a multiple of 64: 16-byte accesses throughout
    v[it] = f4{0.f, 0.f, 0.f, 0.f};
    gn[it] = v[it];
    if (i < d) {
      v[it] = *(const f4*)(x + i);
      gn[it] = *(const f4*)(gain + i);
    }
  }
  // slabs are added in index order; four slabs' loads (eight with few rows) are issued together (a slab index past the end is clamped
  // and its value dropped), so that a row costs one memory round trip instead of one per slab
  constexpr int GS = NT > 256 ? 8 : NV <= 4 ? 4 : 1;
  for (int s0 = 0; s0 < n_slabs; s0 += GS) {
    f4 t[GS][NV];
#pragma unroll
    for (int u = 0; u < GS; ++u) {
      const int s = min(s0 + u, n_slabs - 1);
#pragma unroll
      for (int it = 0; it < NV; ++it) {
        const int i = (it * NT + threadIdx.x) * 4;
        t[u][it] = f4{0.f, 0.f, 0.f, 0.f};
        if (i < d) t[u][it] = *(const f4*)(sl + (size_t)s * slab_stride + i);
      }
    }
#pragma unroll
    for (int u = 0; u < GS; ++u)
      if (s0 + u < n_slabs) {
#pragma unroll
        for (int it = 0; it < NV; ++it) v[it] += t[u][it];
      }
  }
  if (r >= n_rows) return;                               // rows beyond the count: loaded (in bounds), never stored
  float ss = 0.f;
#pragma unroll
  for (int it = 0; it < NV; ++it) {
    const int i = (it * NT + threadIdx.x) * 4;
    if (n_slabs > 0 && i < d) *(f4*)(x + i) = v[it];
    ss += v[it][0] * v[it][0] + v[it][1] * v[it][1] + v[it][2] * v[it][2] + v[it][3] * v[it][3];
  }
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  ss = 0.f;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) ss += red[w];
  const float inv = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
  for (int it = 0; it < NV; ++it) {
    const int i = (it * NT + threadIdx.x) * 4;
    if (i < d) {
      if constexpr (CHUNKS) {
        *(f16x4*)(out + act_index(r, i, ld)) = to_f16x4_guarded(v[it][0] * inv * gn[it][0], v[it][1] * inv * gn[it][1],
                                                                v[it][2] * inv * gn[it][2], v[it][3] * inv * gn[it][3], p.status);
      } else {
        typename Vec4<T>::type w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = from_f32<T>(v[it][e] * inv * gn[it][e]);
        *(typename Vec4<T>::type*)(out + (size_t)r * d + i) = w;
      }
    }
  }
}

// Many rows, chunk order: four rows per workgroup, two waves each, put together in LDS so that a store instruction writes the four
// rows' chunks of 16 k as runs of 64 bytes; two groups of four (a 128-byte line) go to one XCD.  Row per workgroup, 16-byte
// pieces: 23.2 us at 3700 rows of 1536 and one slab, 18.6 here.
__global__ void __launch_bounds__(512) rmsnorm_rows_kernel(Plan p, int d, float eps, float* __restrict__ h, const float* __restrict__ slabs,
                                                           SlabCount rule, size_t slab_stride, const float* __restrict__ gain,
                                                           f16* __restrict__ out, int ld) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  extern __shared__ __align__(16) char lds[];            // [4][d] float16, rows 32 bytes apart in the banks
  __shared__ float red[8];
  const int id = blockIdx.x, r0 = ((id & ~15) + (id & 7) * 2 + ((id >> 3) & 1)) * 4;
  const int n_rows = min(p.n_rows[0], ld);
  if (r0 >= n_rows) return;
  const int n_slabs = rule.of(p.n_rows);
  const int wave = threadIdx.x >> 6, rr = wave >> 1, t128 = threadIdx.x & 127, lds_row = 2 * d + 32;
  const int r = min(r0 + rr, n_rows - 1);                // a row past the end is computed again and stored by nobody
  float* x = h + (size_t)r * d;
  const float* sl = slabs + (size_t)r * d;
  constexpr int NV = 4;                                  // d <= 2048
  f4 v[NV], gn[NV];
#pragma unroll
  for (int it = 0; it < NV; ++it) {
    const int i = (it * 128 + t128) * 4;
    v[it] = f4{0.f, 0.f, 0.f, 0.f};
    gn[it] = v[it];
    if (i < d) {
      v[it] = *(const f4*)(x + i);
      gn[it] = *(const f4*)(gain + i);
    }
  }
  constexpr int GS = 4;                                  // slabs in flight together
  for (int s0 = 0; s0 < n_slabs; s0 += GS) {
    f4 t[GS][NV];
#pragma unroll
    for (int u = 0; u < GS; ++u) {
      const int s = s0 + u;
#pragma unroll
      for (int it = 0; it < NV; ++it) {
        const int i = (it * 128 + t128) * 4;
        t[u][it] = f4{0.f, 0.f, 0.f, 0.f};
        if (i < d && s < n_slabs) t[u][it] = *(const f4*)(sl + (size_t)s * slab_stride + i);
      }
    }
#pragma unroll
    for (int u = 0; u < GS; ++u)
      if (s0 + u < n_slabs) {
#pragma unroll
        for (int it = 0; it < NV; ++it) v[it] += t[u][it];
      }
  }
  float ss = 0.f;
#pragma unroll
  for (int it = 0; it < NV; ++it) {
    const int i = (it * 128 + t128) * 4;
    if (n_slabs > 0 && i < d && r0 + rr < n_rows) *(f4*)(x + i) = v[it];
    ss += v[it][0] * v[it][0] + v[it][1] * v[it][1] + v[it][2] * v[it][2] + v[it][3] * v[it][3];
  }
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if ((threadIdx.x & 63) == 0) red[wave] = ss;
  __syncthreads();
  ss = red[wave & 6] + red[wave | 1];
  const float inv = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
  for (int it = 0; it < NV; ++it) {
    const int i = (it * 128 + t128) * 4;
    if (i < d && r0 + rr < n_rows)
      *(f16x4*)(lds + rr * lds_row + i * 2) = to_f16x4_guarded(v[it][0] * inv * gn[it][0], v[it][1] * inv * gn[it][1],
                                                               v[it][2] * inv * gn[it][2], v[it][3] * inv * gn[it][3], p.status);
  }
  __syncthreads();
  const int row = r0 + (threadIdx.x & 3);
  if (row < n_rows)
    for (int c = threadIdx.x >> 2; c < d / 8; c += 128)
      *(f4*)(out + act_index(row, c * 8, ld)) = *(const f4*)(lds + (threadIdx.x & 3) * lds_row + c * 16);
}

// Inverse rotary frequencies theta^(-2j/D), j < D/2, in float64 (filled once per context).
__global__ void rope_table_kernel(int D, float theta, double* __restrict__ inv_freq) {
  const int j = threadIdx.x;
  if (j < D / 2) inv_freq[j] = exp2(-2.0 * (double)j / (double)D * log2((double)theta));
}

// Rotary (pairs (j, j + D/2), angle = position * theta^(-2j/D)) on q and k of packed row r at
// absolute position c_b + i, with the cos / sin table filled by embed_kernel.  The QKV projection arrives in
// float32, as n_slabs K-split slabs that are summed here (so each of q, k, v is rounded exactly once, after
// the rotation): q goes to the query buffer (float16 for bf16 models: it is an attention operand, not
// cache data), k and v to the slot's page in the cache dtype.
// A work item is four consecutive rotation pairs of one head (two 16-byte loads per slab, 8-byte stores) or four consecutive v
// elements; a thread has one, a row several workgroups.  Latency bound: the loads of four slabs go out together, before the row is
// known to be live or its page is known (64 .. 136 rows of the 7B shape, 5 .. 7 slabs one after the other and three items a thread: 8.4 .. 11.8 us).
template <typename T, typename TQ, typename TP>
__global__ void __launch_bounds__(256) rope_append_kernel(Plan p, int Hq, int Hkv, int D,
                                                          const float* __restrict__ cos_t, const float* __restrict__ sin_t,
                                                          const float* __restrict__ qkv, SlabCount rule, size_t slab_stride,
                                                          TQ* __restrict__ q_out, TP* __restrict__ k_pages,
                                                          TP* __restrict__ v_pages) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  const int r = blockIdx.x, idx = blockIdx.y * 256 + threadIdx.x;
  const int n_rows = p.n_rows[0];
  if (rule.at != 0 && r >= n_rows) return;               // the device rule needs the row count before the first slab load anyway
  const int n_slabs = max(rule.of(p.n_rows), 1);
  const int half = D / 2, groups = half / 4;
  const int n_rot = (Hq + Hkv) * groups, n_items = n_rot + Hkv * D / 4;
  if (idx >= n_items) return;
  const bool rot = idx < n_rot;
  const int hh = rot ? idx / groups : 0, j = rot ? (idx % groups) * 4 : 0;
  const int e0 = rot ? 0 : (idx - n_rot) * 4;            // four consecutive v elements of one head
  const float* x = qkv + (size_t)r * (Hq + 2 * Hkv) * D + (rot ? hh * D + j : (Hq + Hkv) * D + e0);
  const int x2_at = rot ? half : 0;
  const int place = p.row_kv[r];                         // (of a row beyond the count: never used)
  f4 x1 = f4{0.f, 0.f, 0.f, 0.f}, x2 = x1, c = x1, sn = x1;
  if (rot) { c = *(const f4*)(cos_t + (size_t)r * half + j); sn = *(const f4*)(sin_t + (size_t)r * half + j); }
  for (int s0 = 0; s0 < n_slabs; s0 += 4) {              // added in index order; an index past the end is clamped and its value dropped
    f4 t1[4], t2[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float* xs = x + (size_t)min(s0 + u, n_slabs - 1) * slab_stride;
      t1[u] = *(const f4*)xs;
      t2[u] = *(const f4*)(xs + x2_at);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (s0 + u < n_slabs) { x1 += t1[u]; x2 += t2[u]; }
  }
  if (r >= n_rows) return;                               // rows beyond the count: loaded (in bounds), never stored
  float y1[4], y2[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    y1[e] = x1[e] * c[e] - x2[e] * sn[e];
    y2[e] = x2[e] * c[e] + x1[e] * sn[e];
  }
  if (rot && hh < Hq) {
    TQ* qrow = q_out + (size_t)r * Hq * D;
    if constexpr (std::is_same<TQ, f16>::value) {
      *(f16x4*)(qrow + hh * D + j) = to_f16x4_guarded(y1[0], y1[1], y1[2], y1[3], p.status);
      *(f16x4*)(qrow + hh * D + j + half) = to_f16x4_guarded(y2[0], y2[1], y2[2], y2[3], p.status);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        qrow[hh * D + j + e] = from_f32<TQ>(y1[e]);
        qrow[hh * D + j + half + e] = from_f32<TQ>(y2[e]);
      }
    }
    return;
  }
  const int tok = place & (kPage - 1);
  const size_t pbase = (size_t)(place / kPage) * kv_page_elems(Hkv, D);
  // rounded to the cache dtype T, stored in the page encoding TP
  auto rt = [](float v) { return to_f32<T>(from_f32<T>(v)); };
  if (rot) {
    const int kh = hh - Hq;
    TP* k1 = k_pages + pbase + k_index<TP>(D, kh, tok, j);   // four consecutive d are contiguous in both page layouts
    TP* k2 = k_pages + pbase + k_index<TP>(D, kh, tok, j + half);
    if constexpr (std::is_same<TP, f16>::value) {
      *(f16x4*)k1 = to_f16x4_guarded(rt(y1[0]), rt(y1[1]), rt(y1[2]), rt(y1[3]), p.status);
      *(f16x4*)k2 = to_f16x4_guarded(rt(y2[0]), rt(y2[1]), rt(y2[2]), rt(y2[3]), p.status);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        k1[e] = from_f32<TP>(rt(y1[e]));
        k2[e] = from_f32<TP>(rt(y2[e]));
      }
    }
  } else {
    const int kh = e0 / D, dd = e0 % D;
    if constexpr (std::is_same<TP, f16>::value) {
      const f16x4 w = to_f16x4_guarded(rt(x1[0]), rt(x1[1]), rt(x1[2]), rt(x1[3]), p.status);
#pragma unroll
      for (int e = 0; e < 4; ++e) v_pages[pbase + v_index<TP>(D, kh, tok, dd + e)] = w[e];
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v_pages[pbase + v_index<TP>(D, kh, tok, dd + e)] = from_f32<TP>(rt(x1[e]));
    }
  }
}

// Export / import of cached rows, float32 pages: they are row-major, so a row is one contiguous run.
__global__ void __launch_bounds__(256) kv_copy_f32_kernel(KvView kv, int Hkv, int D, int slot, int pos0, float* __restrict__ k_pages,
                                                          float* __restrict__ v_pages, float* __restrict__ k_rows,
                                                          float* __restrict__ v_rows, int to_pages) {
  int i = blockIdx.x, pos = pos0 + i;
  int page = kv.block_table[(size_t)slot * kv.max_pages + pos / kPage];
  if (page < 0 || page >= kv.n_pages) return;
  int tok = pos % kPage;
  size_t pbase = (size_t)page * kv_page_elems(Hkv, D);
  for (int idx = threadIdx.x; idx < Hkv * D; idx += blockDim.x) {
    int kh = idx / D, dd = idx % D;
    size_t ki = pbase + k_index<float>(D, kh, tok, dd), vi = pbase + v_index<float>(D, kh, tok, dd);
    size_t ri = (size_t)i * Hkv * D + idx;
    if (to_pages) { k_pages[ki] = k_rows[ri]; v_pages[vi] = v_rows[ri]; }
    else          { k_rows[ri] = k_pages[ki]; v_rows[ri] = v_pages[vi]; }
  }
}

// Export / import of cached rows, float16 pages <-> bf16 rows.  One workgroup per (tile of 32 tokens, KV head, K or V); a thread
// moves the sixteen bytes that are contiguous in the page: eight dims of one token (K) or one dim of eight tokens (V).  Latency
// bound at these sizes (1900 rows x 2 heads x 128: 3.9 MB; one workgroup per row with two-byte accesses took 5.3 us, this takes 4.9, three dependent memory trips), hence every
// load of a thread before its first store.  vec: the rows start on sixteen bytes.
__global__ void __launch_bounds__(256) kv_copy_f16_kernel(KvView kv, int Hkv, int D, int slot, int pos0, int n, f16* __restrict__ k_pages,
                                                          f16* __restrict__ v_pages, bf16* __restrict__ k_rows,
                                                          bf16* __restrict__ v_rows, int to_pages, int vec, int32_t* __restrict__ status) {
  typedef f16 h8 __attribute__((ext_vector_type(8)));
  typedef bf16 b8 __attribute__((ext_vector_type(8)));
  const int t0 = (pos0 / kTile + blockIdx.x) * kTile;            // first token of the tile
  const int kh = blockIdx.y >> 1, is_v = blockIdx.y & 1;
  const int page = kv.block_table[(size_t)slot * kv.max_pages + t0 / kPage];
  if (page < 0 || page >= kv.n_pages) return;
  f16* pg = (is_v ? v_pages : k_pages) + (size_t)page * kv_page_elems(Hkv, D);
  bf16* rows = (is_v ? v_rows : k_rows) + kh * D;
  const int ld = Hkv * D, lo = pos0 - t0, hi = pos0 + n - t0;     // tokens [lo, hi) of the tile are the caller's
  const int nchunk = kTile * D / 8;
  bool out_of_range = false;
  auto enc = [&](bf16 x) {
    float f = to_f32<bf16>(x);
    if (!(fabsf(f) <= 65504.f)) { f = f16_saturate(f); out_of_range = true; }   // imported bf16 values beyond the float16 range
    return from_f32<f16>(f);
  };
  auto dec = [](f16 x) { return from_f32<bf16>(to_f32<f16>(x)); };
  for (int c = threadIdx.x; c < nchunk; c += 256) {
    if (!is_v) {                                         // consecutive threads: consecutive dims of a token
      const int t = c / (D / 8), d = c % (D / 8) * 8;
      if (t < lo || t >= hi) continue;
      h8* pp = (h8*)(pg + k_index<f16>(D, kh, (t0 + t) % kPage, d));
      bf16* rp = rows + (size_t)(t - lo) * ld + d;
      if (to_pages) {
        b8 x; h8 y;
        if (vec) x = *(const b8*)rp;
        else {
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] = rp[e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] = enc(x[e]);
        *pp = y;
      } else {
        const h8 y = *pp;
        b8 x;
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = dec(y[e]);
        if (vec) *(b8*)rp = x;
        else {
#pragma unroll
          for (int e = 0; e < 8; ++e) rp[e] = x[e];
        }
      }
    } else {                                             // consecutive threads: consecutive dims of eight tokens
      const int t = c / D * 8, d = c % D;
      if (t + 8 <= lo || t >= hi) continue;
      f16* pp = pg + v_index<f16>(D, kh, (t0 + t) % kPage, d);
      bf16* rp = rows + ((ptrdiff_t)t - lo) * ld + d;    // only rows in [lo, hi) are touched
      if (to_pages) {
        bf16 x[8]; h8 y;
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = rp[(ptrdiff_t)(min(max(t + e, lo), hi - 1) - t) * ld];
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] = enc(x[e]);
        if (t >= lo && t + 8 <= hi) *(h8*)pp = y;
        else {
#pragma unroll
          for (int e = 0; e < 8; ++e) if (t + e >= lo && t + e < hi) pp[e] = y[e];
        }
      } else {
        const h8 y = *(const h8*)pp;
#pragma unroll
        for (int e = 0; e < 8; ++e) if (t + e >= lo && t + e < hi) rp[(ptrdiff_t)e * ld] = dec(y[e]);
      }
    }
  }
  if (out_of_range) atomicOr(status, BS_FAULT_RANGE);
}

void launch_embed(const Shape& s, const Plan& p, const KvView& kv, int M_max, const StepRules& rules, const void* embed, float* h, const double* inv_freq,
                  float* cos_t, float* sin_t, hipStream_t st) {
  const int grid = M_max + (rules.slab[0].at || rules.qkv.at || rules.glu.at ? kRuleGroups : 0);
  if (s.dtype == BS_F32)
    hipLaunchKernelGGL(embed_kernel<float>, dim3(grid), dim3(256), 0, st, p, kv, M_max, rules, s.d, (const float*)embed, h, s.D, inv_freq, cos_t, sin_t);
  else
    hipLaunchKernelGGL(embed_kernel<bf16>, dim3(grid), dim3(256), 0, st, p, kv, M_max, rules, s.d, (const bf16*)embed, h, s.D, inv_freq, cos_t, sin_t);
}
void launch_rmsnorm(const Shape& s, const Plan& p, int M_max, float* h, const float* slabs, const SlabCount& n_slabs,
                    const float* gain, void* out, hipStream_t st) {
  const size_t stride = (size_t)M_max * s.d;
#define BS_RMS(T_, NV_, NT_) hipLaunchKernelGGL((rmsnorm_kernel<T_, NV_, NT_>), dim3(s.dtype == BS_F32 ? M_max : (M_max + 63) / 64 * 64), dim3(NT_), 0, st, p, s.d, s.eps, h, slabs, n_slabs, stride, gain, (T_*)out, M_max)
  if (s.dtype == BS_F32) { if (s.d <= 2048) BS_RMS(float, 2, 256); else if (s.d <= 4096) BS_RMS(float, 4, 256); else BS_RMS(float, 16, 256); }
  else if (s.d > 4096) BS_RMS(f16, 16, 256);
  // Few rows are one round of workgroups at most, and up to 8 slabs of them: all of a row's loads in one trip.
  else if (M_max <= 640) { if (s.d <= 2048) BS_RMS(f16, 1, 512); else BS_RMS(f16, 2, 512); }
  // Four rows per workgroup need several rounds of workgroups: 3700 rows of 1536 23.2 -> 18.6 us; 976 rows 8.6 -> 9.2; 1185 rows of
  // 3584 (28 floats a thread) 17.4 -> 25.8.
  else if (s.d <= 2048 && M_max > 2048)
    hipLaunchKernelGGL(rmsnorm_rows_kernel, dim3((M_max + 63) / 64 * 16), dim3(512), 4 * (2 * s.d + 32), st, p, s.d, s.eps, h, slabs, n_slabs, stride, gain, (f16*)out, M_max);
  else { if (s.d <= 2048) BS_RMS(f16, 2, 256); else BS_RMS(f16, 4, 256); }
#undef BS_RMS
}
void launch_rope_table(const Shape& s, double* inv_freq, hipStream_t st) {
  hipLaunchKernelGGL(rope_table_kernel, dim3(1), dim3(64), 0, st, s.D, s.theta, inv_freq);
}
void launch_rope_append(const Shape& s, const Plan& p, int M_max, const float* cos_t, const float* sin_t,
                        const float* qkv, const SlabCount& n_slabs, void* q_out, void* k_pages, void* v_pages, hipStream_t st) {
  const size_t stride = (size_t)M_max * s.Nqkv();
  const int y = ((s.Hq + s.Hkv) * s.D / 8 + s.Hkv * s.D / 4 + 255) / 256;
  if (s.dtype == BS_F32)
    hipLaunchKernelGGL((rope_append_kernel<float, float, float>), dim3(M_max, y), dim3(256), 0, st, p, s.Hq, s.Hkv, s.D, cos_t, sin_t,
                       qkv, n_slabs, stride, (float*)q_out, (float*)k_pages, (float*)v_pages);
  else
    hipLaunchKernelGGL((rope_append_kernel<bf16, f16, f16>), dim3(M_max, y), dim3(256), 0, st, p, s.Hq, s.Hkv, s.D, cos_t, sin_t,
                       qkv, n_slabs, stride, (f16*)q_out, (f16*)k_pages, (f16*)v_pages);
}
void launch_kv_copy(const Shape& s, const KvView& kv, int slot, int pos0, int n, void* k_pages, void* v_pages,
                    void* k_rows, void* v_rows, bool to_pages, int32_t* status, hipStream_t st) {
  if (n <= 0) return;
  if (s.dtype == BS_F32) {
    hipLaunchKernelGGL(kv_copy_f32_kernel, dim3(n), dim3(256), 0, st, kv, s.Hkv, s.D, slot, pos0, (float*)k_pages, (float*)v_pages,
                       (float*)k_rows, (float*)v_rows, to_pages ? 1 : 0);
    return;
  }
  const int tiles = (pos0 + n - 1) / kTile - pos0 / kTile + 1;
  const int vec = (((uintptr_t)k_rows | (uintptr_t)v_rows) & 15) == 0;
  hipLaunchKernelGGL(kv_copy_f16_kernel, dim3(tiles, 2 * s.Hkv), dim3(256), 0, st, kv, s.Hkv, s.D, slot, pos0, n, (f16*)k_pages,
                     (f16*)v_pages, (bf16*)k_rows, (bf16*)v_rows, to_pages ? 1 : 0, vec, status);
}
