// Plain (non-MFMA) verify attention on row-major pages: one workgroup per (packed row, query
// head), 256 tokens per pass.  Latency bound (few, small workgroups): pages of a pass come from LDS and a thread
// requests sixteen tokens' elements before it uses the first (20 rows x 4 heads, about 200 tokens: 16.5 us with a
// page lookup per load and one load at a time, 9.9 us).  Used by float32 models (the tiny parity configuration).  Sec. 3.3: every query
// length 1..k_max+1 is served by this one launch; row i of sequence b attends to cache
// positions 0 .. c_b + i (committed context plus the tentative rows up to itself).
#pragma once
#include "common.h"

template <typename T, typename TO>
__global__ void __launch_bounds__(256) attn_simple_kernel(Plan p, KvView kv, int Hq, int Hkv, int D, float scale,
                                                          const TO* __restrict__ q, const T* __restrict__ k_pages,
                                                          const T* __restrict__ v_pages, TO* __restrict__ out) {
  static_assert(std::is_same<T, float>::value, "the dot product below loads four row-major floats at a time");
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef float f4_u __attribute__((ext_vector_type(4), aligned(4)));   // the caller's pages: aligned to their elements only
  __shared__ __align__(16) float s_q[128];
  __shared__ float s_p[256], s_red[4], s_acc[256];
  __shared__ int s_pg[256 / kPage];                     // pages of the 256 tokens of a chunk
  const int r = blockIdx.x, hq = blockIdx.y;
  if (r >= p.n_rows[0]) return;
  const int b = p.row_seq[r];
  const int n_tok = p.seq_c[b] + p.row_pos[r] + 1;
  const int kvh = hq / (Hq / Hkv);
  const int tid = threadIdx.x;
  const int32_t* bt = kv.block_table + (size_t)p.seq_slot[b] * kv.max_pages;
  const size_t page_elems = kv_page_elems(Hkv, D);
  if (tid < D) s_q[tid] = to_f32<TO>(q[(size_t)r * Hq * D + (size_t)hq * D + tid]);
  float m_run = -INFINITY, l_run = 0.f, acc = 0.f;      // acc: thread (tid%D, tid/D) partial of out[d]
  const int dd = tid % D, part = tid / D, nparts = 256 / D;
  for (int t0 = 0; t0 < n_tok; t0 += 256) {
    if (tid < 256 / kPage) s_pg[tid] = min(max(bt[min(t0 + tid * kPage, n_tok - 1) / kPage], 0), kv.n_pages - 1);
    __syncthreads();
    const int t = t0 + tid;
    float s = -INFINITY;
    if (t < n_tok) {
      const int page = s_pg[tid / kPage];
      const T* kp = k_pages + (size_t)page * page_elems + k_index<T>(D, kvh, t % kPage, 0);   // row-major: D contiguous elements
      float dot[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 16
      for (int d = 0; d < D; d += 4) {
        const f4 kv4 = *(const f4_u*)(kp + d), q4 = *(const f4*)(s_q + d);
#pragma unroll
        for (int e = 0; e < 4; ++e) dot[e] += q4[e] * kv4[e];
      }
      s = ((dot[0] + dot[1]) + (dot[2] + dot[3])) * scale;
    }
    float mx = s;
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    if ((tid & 63) == 0) s_red[tid >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3]));
    const float m_new = fmaxf(m_run, mx);
    const float pr = (t < n_tok) ? __expf(s - m_new) : 0.f;
    s_p[tid] = pr;
    float ps = pr;
    for (int o = 32; o > 0; o >>= 1) ps += __shfl_xor(ps, o);
    __syncthreads();                                   // s_red reads done, s_p visible
    if ((tid & 63) == 0) s_red[tid >> 6] = ps;
    __syncthreads();
    const float alpha = __expf(m_run - m_new);         // exp(-inf) = 0 on the first chunk
    l_run = l_run * alpha + (s_red[0] + s_red[1] + s_red[2] + s_red[3]);
    m_run = m_new;
    acc *= alpha;
    const int cnt = min(256, n_tok - t0);
    for (int j0 = part; j0 < cnt; j0 += 16 * nparts) {   // sixteen tokens' V elements in flight
      float v[16], w[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int j = min(j0 + u * nparts, cnt - 1);
        v[u] = to_f32<T>(v_pages[(size_t)s_pg[j / kPage] * page_elems + v_index<T>(D, kvh, j % kPage, dd)]);
        w[u] = s_p[j];
      }
#pragma unroll
      for (int u = 0; u < 16; ++u)                       // beyond the end: the last token read again, not added (0 * inf is NaN)
        acc += j0 + u * nparts < cnt ? w[u] * v[u] : 0.f;
    }
    __syncthreads();
  }
  s_acc[tid] = acc;                                      // nparts partial sums per d
  __syncthreads();
  if (tid < D) {
    float o = s_acc[tid];
    for (int pp = 1; pp < nparts; ++pp) o += s_acc[pp * D + tid];
    out[(size_t)r * Hq * D + (size_t)hq * D + tid] = from_f32<TO>(o / l_run);
  }
}
