// LM head fused with softmax statistics, the accept scan of Alg. 1 and the residual / bonus
// sampling of Eq. 2-3.  The [M, V] probabilities are never formed in HBM, and the logits only where phase 2 costs more than
// writing them (up to lmhead_logit_rows rows):
//   phase 1  LM-head GEMM over all M rows whose epilogue keeps, per (row, vocabulary tile), only
//            (max, sum exp, arg max) of z/T and the logit of the draft token judged by the row;
//   scan     per sequence, the first rejected draft (Eq. 2, general form min(1, p/q));
//   phase 2  the one row per sequence that is sampled from (recovered, bonus or plain token) is read back, or
//            recomputed by the same MFMA loop (bit-identical logits), and sampled by inverse CDF in
//            vocabulary order with float64 running sums (Eq. 3 / max(0, p - q)).
#include "gemm_dma.h"

enum { MODE_NONE = 0, MODE_PLAIN = 1, MODE_RESID_ONEHOT = 2, MODE_RESID_DENSE = 3 };

constexpr int kLmNT = 2;                            // LM-head wave tile: 32*MT rows x 64 vocab entries
constexpr int kLmVtile = kLmNT * 32;                // vocab entries per statistics tile (bf16 path)
constexpr int kSampleChunks = 32;                   // vocabulary chunks per sequence in the sampling kernels

// Factor that carries a sum of exponentials from an old running maximum to a new, larger one.  The sum is still empty while the
// maximum is -inf, and (-inf) * inv_temp is NaN at infinite temperature (inv_temp = 0): the factor is 0 there.
__device__ __forceinline__ float rescale_exp(float from, float to, float inv_temp) {
  return from == -INFINITY ? 0.f : __expf((from - to) * inv_temp);
}

int lmhead_vtiles(int V) {
  const int a = (V + kLmVtile - 1) / kLmVtile;
  return a > kMaxRowSegs ? a : kMaxRowSegs;
}

// Row limit up to which phase 1 stores all logits (float32, 4 V bytes per row) instead of recomputing the sampled row of
// every sequence, which reads the 2 d V bytes of weights again.  Measured, phase 1 with stores against the second pass it
// saves: 7B shape, 64 rows + 10 us / 210, 288 rows + 38 / 203, 576 rows + 87 / 205, 1152 rows no gain; 1.5B shape, 9 rows
// + 4 / 85, 288 rows + 38 / 95, 432 rows no gain, 576 rows + 97 / 100.  (Storing whole lines by way of LDS changed nothing:
// the writes compete with the weight stream, not with the issue slots.)  The rows lie on top of the layers' activations
// and enlarge a workspace by what they exceed those: 7B shape, 288 rows (175 MB of logits) by 116 MB, 2176 rows (545 MB) by 95.
int lmhead_logit_rows(const Shape& s) { return s.dtype == BS_BF16 ? s.d / 4 : 0; }

// ------------------------------------------------------------------ phase 1 / phase 2 GEMM (bf16)
// STATS = true : rows are the packed query rows; epilogue writes statistics (+ optional debug logits).
// STATS = false: rows are the gathered ones (one per sequence); epilogue stores float32 logits to sel_logits [B, V].
template <typename G, bool STATS>
__global__ void __launch_bounds__(G::THREADS, (G::WGS * G::WAVES + 3) / 4) lmhead_kernel(const int32_t* __restrict__ n_rows_dev, int M_max, int V, int K,
                                                     const f16* __restrict__ X, int ld, const f16* __restrict__ W, float inv_temp,
                                                     const int32_t* __restrict__ row_target, SamplerBufs sb,
                                                     float* __restrict__ store, int n_blocks) {
  constexpr int kLmMT = G::MW;
  static_assert(G::NW == kLmNT, "a wave's columns are one statistics tile");
  extern __shared__ __align__(16) char lds[];
  const int M = n_rows_dev ? min(*n_rows_dev, M_max) : M_max;
  const int m_blocks = (M + G::BM - 1) / G::BM;
  const int id = xcd_flat(m_blocks * n_blocks);
  if (id < 0) return;
  const int wave = G::wave_id(), lane = threadIdx.x & 63;
  const size_t tile_bytes = (size_t)(K / kBK) * 4096;
  const int t_last = (V + 31) / 32 - 1;
  auto operands = [&](typename G::Operands& op) {
    const int m0 = id % m_blocks * G::BM, t0 = id / m_blocks * G::CT;
    G::make_operands(op, X, ld, [&](int r) { return min(m0 + r, M - 1); }, W, [&](int t) { return min(t0 + t, t_last) * tile_bytes; }, kWHalf, 0);
  };
  auto finish = [&](f32x4 (&acc)[2 * G::MW][2 * G::NW]) {
  const int m0 = id % m_blocks * G::BM + wave / G::WN * kLmMT * 32;      // first row of this wave
  const int vt = id / m_blocks * G::WN + wave % G::WN;           // statistics tile of this wave
  const int n_wave0 = vt * kLmVtile;
  if (n_wave0 >= V) return;

  // accumulator: acc[a][b][e] = vocabulary entry n_wave0 + 16 b + acc_row + e of token m0 + 16 a + acc_col
  const int n0 = n_wave0 + acc_row(lane);
  const bool store_vec = (V & 3) == 0 && ((uintptr_t)store & 15) == 0;   // V % 4 == 0: groups of four never straddle V
#pragma unroll
  for (int a = 0; a < 2 * kLmMT; ++a) {
    const int m = m0 + a * 16 + acc_col(lane);
    const bool valid = m < M;
    if (STATS) {
      const int tgt = valid ? row_target[m] : -1;
      float mx = -INFINITY, zt = 0.f;
      int arg = 0x7fffffff;
      bool hit = false;
      // no store inside this loop: the draft token's logit is picked up by a select (a conditional store at each of
      // the 32 positions cost 13 us of the 277 us launch)
#pragma unroll
      for (int b = 0; b < 2 * kLmNT; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int n = n0 + 16 * b + e;
          const float z = acc[a][b][e];
          if (n < V) {
            if (z > mx) { mx = z; arg = n; }
            if (n == tgt) { zt = z; hit = true; }
          }
        }
      if (hit) sb.z_target[m] = zt;                    // tgt >= 0 only for valid rows
      if (valid && store && !store_vec) {
#pragma unroll
        for (int b = 0; b < 2 * kLmNT; ++b)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int n = n0 + 16 * b + e;
            if (n < V) store[(size_t)m * V + n] = acc[a][b][e];
          }
      }
      if (valid && store && store_vec) {
        // four consecutive vocabulary entries of a lane: 16-byte stores
#pragma unroll
        for (int b = 0; b < 2 * kLmNT; ++b) {
          const int n = n0 + 16 * b;
          if (n + 3 < V) *(f32x4*)(store + (size_t)m * V + n) = acc[a][b];
        }
      }
#pragma unroll
      for (int o = 16; o <= 32; o += 16) {
        const float mx_o = __shfl_xor(mx, o);
        const int arg_o = __shfl_xor(arg, o);
        if (mx_o > mx || (mx_o == mx && arg_o < arg)) { mx = mx_o; arg = arg_o; }
      }
      float sum = 0.f;
#pragma unroll
      for (int b = 0; b < 2 * kLmNT; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n0 + 16 * b + e < V) sum += __expf((acc[a][b][e] - mx) * inv_temp);
      sum += __shfl_xor(sum, 16);
      sum += __shfl_xor(sum, 32);
      if (valid && lane < 16) {
        const size_t o = (size_t)vt * M_max + m;
        sb.part_max[o] = mx;
        sb.part_sum[o] = sum;
        sb.part_arg[o] = arg;
      }
    } else {
      if (!valid) continue;
      // four consecutive vocabulary entries of a lane: 16-byte stores when the row pitch keeps them aligned
      const bool vec = (V & 3) == 0;
#pragma unroll
      for (int b = 0; b < 2 * kLmNT; ++b) {
        const int n = n0 + 16 * b;
        if (vec && n + 3 < V) {
          *(f32x4*)(store + (size_t)m * V + n) = acc[a][b];
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (n + e < V) store[(size_t)m * V + n + e] = acc[a][b][e];
        }
      }
    }
  }
  };
  G::run(K / 32, lds, operands, finish);
}

// ------------------------------------------------------------------ statistics of given float32 logits
// One workgroup per (row, vocabulary segment), one entry of (max, sum exp, arg max) each; HBM bound: the row is read once,
// sixteen bytes per load, four loads in flight per thread, maximum and rescaled sum kept online; len: entries per segment (batch 128 x 9 rows of 151936
// logits, 700 MB: 232 us with one workgroup per 1024 entries and four-byte loads, 114 us).
__global__ void __launch_bounds__(256) logit_stats_kernel(Plan p, int M_max, int V, int len, const float* __restrict__ logits,
                                                          float inv_temp, SamplerBufs sb) {
  __shared__ float s_mx[4], s_sum[4];
  __shared__ int s_arg[4];
  const int m = blockIdx.y, seg = blockIdx.x, tid = threadIdx.x;
  if (m >= p.n_rows[0]) return;
  const int tgt = p.row_target[m];
  const float* z = logits + (size_t)m * V;
  const int j0 = min(seg * len, V), j1 = min(j0 + len, V);
  float mx = -INFINITY, sum[4] = {0.f, 0.f, 0.f, 0.f};
  int arg = 0x7fffffff;
  auto absorb = [&](const float* x, int n, int cnt) {    // cnt values of indices n ..
    float vm = x[0];
#pragma unroll
    for (int e = 1; e < 4; ++e) vm = e < cnt ? fmaxf(vm, x[e]) : vm;
    if (vm > mx) {
      const float f = rescale_exp(mx, vm, inv_temp);     // 0 on the first values
#pragma unroll
      for (int e = 0; e < 4; ++e) sum[e] *= f;
      mx = vm;
#pragma unroll
      for (int e = 3; e >= 0; --e) if (e < cnt && x[e] == vm) arg = n + e;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) if (e < cnt) sum[e] += x[e] == -INFINITY ? 0.f : __expf((x[e] - mx) * inv_temp);
  };
  const int v0 = min(j0 + (int)((16 - ((uintptr_t)(z + j0) & 15)) & 15) / 4, j1);   // first token of an aligned group of four
  const int n4 = (j1 - v0) / 4;
  int i = tid;
  for (; i + 3 * 256 < n4; i += 4 * 256) {
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = *(const f32x4*)(z + v0 + 4 * (i + u * 256));
#pragma unroll
    for (int u = 0; u < 4; ++u) { const float x[4] = {v[u][0], v[u][1], v[u][2], v[u][3]}; absorb(x, v0 + 4 * (i + u * 256), 4); }
  }
  for (; i < n4; i += 256) {
    const f32x4 v = *(const f32x4*)(z + v0 + 4 * i);
    const float x[4] = {v[0], v[1], v[2], v[3]};
    absorb(x, v0 + 4 * i, 4);
  }
  // up to three tokens before and after the groups; the first threads take them last, so compare indices of equal maxima
  for (int e = tid; e < 6; e += 256) {
    const int n = e < 3 ? j0 + e : v0 + 4 * n4 + e - 3;
    if (e < 3 ? n >= v0 : n >= j1) continue;
    const float x[4] = {z[n], 0.f, 0.f, 0.f};
    if (x[0] == mx && mx > -INFINITY && n < arg) arg = n;
    absorb(x, n, 1);
  }
  if (tid == 0 && tgt >= j0 && tgt < j1) sb.z_target[m] = z[tgt];
  float s = (sum[0] + sum[1]) + (sum[2] + sum[3]);
  for (int o = 32; o > 0; o >>= 1) {
    const float mo = __shfl_xor(mx, o), so = __shfl_xor(s, o);
    const int ao = __shfl_xor(arg, o);
    if (mo > mx) { s = s * rescale_exp(mx, mo, inv_temp) + so; mx = mo; arg = ao; }
    else if (mo > -INFINITY) { s += so * __expf((mo - mx) * inv_temp); if (mo == mx && ao < arg) arg = ao; }
  }
  if ((tid & 63) == 0) { s_mx[tid >> 6] = mx; s_sum[tid >> 6] = s; s_arg[tid >> 6] = arg; }
  __syncthreads();
  if (tid == 0) {
    float mt = s_mx[0], st = s_sum[0];
    int at = s_arg[0];
    for (int w = 1; w < 4; ++w) {
      const float mo = s_mx[w];
      if (mo > mt) { st = st * rescale_exp(mt, mo, inv_temp) + s_sum[w]; mt = mo; at = s_arg[w]; }
      else if (mo > -INFINITY) { st += s_sum[w] * __expf((mo - mt) * inv_temp); if (mo == mt && s_arg[w] < at) at = s_arg[w]; }
    }
    const size_t o = (size_t)seg * M_max + m;
    sb.part_max[o] = mt;
    sb.part_sum[o] = st;
    sb.part_arg[o] = at;
  }
}

// ------------------------------------------------------------------ per-row statistics
// Stage 1 folds the per-tile (max, sum exp, arg max) entries of 32 consecutive rows over one of kStatChunks
// ranges of vocabulary tiles into one entry per (row, range) with the same meaning.  Tile entries of a row
// are M_max apart, so a workgroup reads 32 rows x 8 tiles at a time: every 128-byte line it touches is used
// completely (one workgroup per row touched a new line for every 4-byte entry: 175 MB fetched for 16 MB).
constexpr int kStatChunks = 16;
__global__ void __launch_bounds__(256) row_stats_fold_kernel(Plan p, int M_max, int n_vtiles, float inv_temp, SamplerBufs sb) {
  __shared__ float s_mx[8][32], s_sum[8][32];
  __shared__ int s_arg[8][32];
  const int rr = threadIdx.x & 31, vl = threadIdx.x >> 5;
  const int r = blockIdx.x * 32 + rr, ch = blockIdx.y;
  const int per = (n_vtiles + kStatChunks - 1) / kStatChunks;
  const int v0 = min(ch * per, n_vtiles), v1 = min(v0 + per, n_vtiles);
  const bool valid = r < min(p.n_rows[0], M_max);
  float mx = -INFINITY, sum = 0.f;
  int arg = 0x7fffffff;
  auto fold = [&](float m2, float s2, int a2) {
    if (m2 > mx) { sum = sum * rescale_exp(mx, m2, inv_temp) + s2; mx = m2; arg = a2; }
    else if (m2 > -INFINITY) { sum += s2 * __expf((m2 - mx) * inv_temp); if (m2 == mx && a2 < arg) arg = a2; }
  };
  if (valid) {
    // four tile entries are requested before the first is folded (same order of folding): one memory round trip
    // per four entries instead of one per entry
    int vt = v0 + vl;
    for (; vt + 24 < v1; vt += 32) {
      float m4[4], s4[4];
      int a4[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const size_t o = (size_t)(vt + 8 * u) * M_max + r;
        m4[u] = sb.part_max[o]; s4[u] = sb.part_sum[o]; a4[u] = sb.part_arg[o];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) fold(m4[u], s4[u], a4[u]);
    }
    for (; vt < v1; vt += 8) {
      const size_t o = (size_t)vt * M_max + r;
      fold(sb.part_max[o], sb.part_sum[o], sb.part_arg[o]);
    }
  }
  s_mx[vl][rr] = mx; s_sum[vl][rr] = sum; s_arg[vl][rr] = arg;
  __syncthreads();
  if (vl == 0 && valid) {
    for (int w = 1; w < 8; ++w) fold(s_mx[w][rr], s_sum[w][rr], s_arg[w][rr]);
    const size_t o = (size_t)ch * M_max + r;
    sb.fold_max[o] = mx; sb.fold_sum[o] = sum; sb.fold_arg[o] = arg;
  }
}

// Stage 2 (also the only stage for the few segments of the plain-logits path):
__global__ void __launch_bounds__(256) row_stats_kernel(Plan p, int M_max, int n_vtiles, float inv_temp, SamplerBufs sb,
                                                        const float* __restrict__ t_max, const float* __restrict__ t_sum,
                                                        const int32_t* __restrict__ t_arg) {
  __shared__ float s_mx[4], s_sum[4];
  __shared__ int s_arg[4];
  const int r = blockIdx.x, tid = threadIdx.x;
  if (r >= p.n_rows[0]) return;
  float mx = -INFINITY;
  int arg = 0x7fffffff;
  for (int vt = tid; vt < n_vtiles; vt += 256) {
    const float m2 = t_max[(size_t)vt * M_max + r];
    const int a2 = t_arg[(size_t)vt * M_max + r];
    if (m2 > mx || (m2 == mx && a2 < arg)) { mx = m2; arg = a2; }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const float mo = __shfl_xor(mx, o);
    const int ao = __shfl_xor(arg, o);
    if (mo > mx || (mo == mx && ao < arg)) { mx = mo; arg = ao; }
  }
  if ((tid & 63) == 0) { s_mx[tid >> 6] = mx; s_arg[tid >> 6] = arg; }
  __syncthreads();
  mx = s_mx[0]; arg = s_arg[0];
  for (int w = 1; w < 4; ++w)
    if (s_mx[w] > mx || (s_mx[w] == mx && s_arg[w] < arg)) { mx = s_mx[w]; arg = s_arg[w]; }
  float sum = 0.f;
  for (int vt = tid; vt < n_vtiles; vt += 256) {
    const float m2 = t_max[(size_t)vt * M_max + r];
    if (m2 > -INFINITY) sum += t_sum[(size_t)vt * M_max + r] * __expf((m2 - mx) * inv_temp);
  }
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  if ((tid & 63) == 0) s_sum[tid >> 6] = sum;
  __syncthreads();
  if (tid == 0) {
    sb.row_max[r] = mx;
    sb.row_lse[r] = mx * inv_temp + logf(s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3]);
    sb.row_arg[r] = arg;
  }
}

// ------------------------------------------------------------------ proposal statistics
// For every query row that judges a draft: max and log-sum-exp of its q_logits row and q_logits[draft].
// One pass (online max / rescaled sum), 16-byte loads.
template <typename Q> struct QVec;
template <> struct QVec<float> { static constexpr int N = 4; };
template <> struct QVec<bf16> { static constexpr int N = 8; };

template <typename Q>
__global__ void __launch_bounds__(256) q_stats_kernel(Plan p, int V, const Q* __restrict__ q_logits, SamplerBufs sb) {
  __shared__ float s_m[4], s_s[4];
  const int r = blockIdx.x, tid = threadIdx.x;
  if (r >= p.n_rows[0]) return;
  const int tgt = p.row_target[r];
  if (tgt < 0) return;
  const int b = p.row_seq[r];
  const Q* q = q_logits + (size_t)(p.draft_start[b] + p.row_pos[r]) * V;
  constexpr int N = QVec<Q>::N;
  float m = -INFINITY, sum = 0.f;
  auto absorb = [&](float x) {
    if (x > m) { sum = sum * __expf(m - x) + 1.0f; m = x; }   // exp(-inf) = 0 on the first element
    else sum += __expf(x - m);
  };
  // U 16-byte vectors: a single rescale for their maximum, then the exponentials
  auto absorb_vecs = [&](auto count, const u32x4* raw) {
    constexpr int U = decltype(count)::value;
    float x[U][N], vm = -INFINITY;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (N == 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[u][j] = __uint_as_float(raw[u][j]);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) { x[u][2 * j] = __uint_as_float(raw[u][j] << 16); x[u][2 * j + 1] = __uint_as_float(raw[u][j] & 0xffff0000u); }
      }
#pragma unroll
      for (int j = 0; j < N; ++j) vm = fmaxf(vm, x[u][j]);
    }
    if (vm == -INFINITY) {                                    // masked tokens; a vector of NaN alone is none and makes the sum NaN
#pragma unroll
      for (int u = 0; u < U; ++u) {
        bool number = false;
#pragma unroll
        for (int j = 0; j < N; ++j) number |= x[u][j] == x[u][j];
        if (!number) sum = __builtin_nanf("");
      }
      return;
    }
    if (vm > m) { sum *= __expf(m - vm); m = vm; }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < N; ++j) sum += __expf(x[u][j] - m);
  };
  constexpr std::integral_constant<int, 1> One{};
  constexpr int B = 4;
  constexpr std::integral_constant<int, B> Batch{};
  const bool aligned = (((uintptr_t)q) & 15) == 0;
  const int nvec = aligned ? V / N : 0;
  // With one workgroup per row the bytes in flight, not HBM, set the rate: while four vectors per thread are absorbed the
  // next four are on their way (1024 rows of 151936: 68 -> 64 us).
  const int n_batches = nvec / (B * 256);
  u32x4 v[2][B];
  auto fetch = [&](u32x4* r, int batch) {
    batch = min(batch, n_batches - 1);
#pragma unroll
    for (int u = 0; u < B; ++u) r[u] = *(const u32x4*)(q + (size_t)((batch * B + u) * 256 + tid) * N);
  };
  if (n_batches > 0) {
    fetch(v[0], 0);
    int i = 0;
    for (; i + 2 <= n_batches; i += 2) {
      fetch(v[1], i + 1);
      absorb_vecs(Batch, v[0]);
      fetch(v[0], i + 2);
      absorb_vecs(Batch, v[1]);
    }
    if (i < n_batches) absorb_vecs(Batch, v[0]);
  }
  for (int i = n_batches * B * 256 + tid; i < nvec; i += 256) {
    const u32x4 one = *(const u32x4*)(q + (size_t)i * N);
    absorb_vecs(One, &one);
  }
  for (int n = nvec * N + tid; n < V; n += 256) absorb(to_f32<Q>(q[n]));
  for (int o = 32; o > 0; o >>= 1) {
    const float mo = __shfl_xor(m, o), so = __shfl_xor(sum, o);
    const float mn = fmaxf(m, mo);
    sum = (m == -INFINITY ? 0.f : sum * __expf(m - mn)) + (mo == -INFINITY ? 0.f : so * __expf(mo - mn));
    m = mn;
  }
  if ((tid & 63) == 0) { s_m[tid >> 6] = m; s_s[tid >> 6] = sum; }
  __syncthreads();
  if (tid == 0) {
    float mt = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3])), st = 0.f;
    for (int w = 0; w < 4; ++w) if (s_m[w] > -INFINITY) st += s_s[w] * __expf(s_m[w] - mt);
    sb.q_max[r] = mt;
    sb.q_lse[r] = mt + logf(st);
    sb.q_target[r] = to_f32<Q>(q[tgt]);
  }
}

// ------------------------------------------------------------------ accept scan (Alg. 1 inner loop, Eq. 2)
// One thread per sequence: the first rejected draft, the row that will be sampled from and how.
__global__ void __launch_bounds__(64) accept_scan_kernel(Plan p, int B, int k_max, int dense_q, float temperature,
                                                         int eos_id, int emit_bonus, int filter_on,
                                                         const float* __restrict__ u_accept,
                                                         SamplerBufs sb, int32_t* __restrict__ n_accepted,
                                                         int32_t* __restrict__ out_tokens, int32_t* __restrict__ n_emitted,
                                                         uint32_t* __restrict__ near_tie) {
  const int b = blockIdx.x * 64 + threadIdx.x;
  if (b >= B) return;
  const int k = p.seq_k[b];
  int32_t* out = out_tokens + (size_t)b * (k_max + 1);
  if (k < 0) {                                      // sequence skipped by the plan
    n_accepted[b] = 0; n_emitted[b] = 0; near_tie[b] = 0; sb.sel_mode[b] = MODE_NONE; sb.sel_row[b] = 0;
    for (int i = 0; i <= k_max; ++i) out[i] = -1;
    return;
  }
  const int r0 = p.row_start[b];
  const float inv_temp = temperature > 0.f ? 1.0f / temperature : 1.0f;
  int n_acc = 0, mode = MODE_NONE, sel = r0, sel_tok = -1, n_out = 0;
  uint32_t tie = 0;
  bool stopped = false, eos = false;
  for (int i = 0; i < k && !stopped; ++i) {
    const int r = r0 + i;
    const int x = p.row_target[r];
    float px;
    if (temperature > 0.f && filter_on)             // filtered target: zero outside the kept set, renormalised inside
      px = filter_keeps(filter_key(sb.z_target[r]), x, sb.f_key[r], sb.f_idx[r])
               ? __expf(sb.z_target[r] * inv_temp - sb.f_lse[r]) : 0.0f;
    else if (temperature > 0.f) px = __expf(sb.z_target[r] * inv_temp - sb.row_lse[r]);
    else px = (x == sb.row_arg[r]) ? 1.0f : 0.0f;
    float rho = px;
    if (dense_q) {
      const float qx = __expf(sb.q_target[r] - sb.q_lse[r]);
      rho = (qx == 0.f) ? INFINITY : px / qx;
    }
    const float u = u_accept[(size_t)b * k_max + i];
    if (fabsf(rho - u) <= 1e-3f) tie |= 1u << i;
    if (u < fminf(1.0f, rho)) {
      out[n_out++] = x;
      ++n_acc;
      if (x == eos_id) { stopped = true; eos = true; }
    } else {
      sel = r; sel_tok = x;
      mode = dense_q ? MODE_RESID_DENSE : MODE_RESID_ONEHOT;
      stopped = true;
    }
  }
  if (mode == MODE_NONE && !eos && (emit_bonus || k == 0)) {
    sel = r0 + k;
    mode = MODE_PLAIN;
  }
  if (mode != MODE_NONE && temperature == 0.f) {    // one-hot target: every sampled token is the arg-max
    out[n_out++] = sb.row_arg[sel];
    mode = MODE_NONE;
  }
  for (int i = n_out; i <= k_max; ++i) out[i] = -1;
  n_accepted[b] = n_acc;
  n_emitted[b] = n_out;
  near_tie[b] = tie;
  sb.sel_row[b] = sel;
  sb.sel_mode[b] = mode;
  sb.sel_tok[b] = sel_tok;
  sb.sel_qrow[b] = p.draft_start[b] + (sel - r0);
  sb.sel_pmax[b] = sb.row_max[sel];
  sb.sel_qmax[b] = (mode == MODE_RESID_DENSE) ? sb.q_max[sel] : 0.f;
}

// ------------------------------------------------------------------ inverse-CDF sampling (Eq. 3)
// The vocabulary of each sampled row is cut into kSampleChunks chunks so that B x 32 workgroups share
// the float64 exponentials.  Three small kernels: normaliser partials, chunk masses (dense proposals), pick.
//   p_j = exp(z_j/T - max) / sum_p ;  q_j likewise ;  w_j = p_j | p_j [j != draft] | max(0, p_j - q_j)
// Divisions by per-row constants (T, the two normalisers) are multiplications by their float64 reciprocals: a
// float64 division costs about as much as the exponential next to it, and the one-ulp difference is far below
// what the order of the running sums already leaves open.
// e^x in float64 for x <= 0 (the rows' maximum is subtracted), -inf -> 0 and NaN -> NaN.  x = n ln 2 + r with the remainder in two
// steps, e^r by a polynomial of degree 11 (minimax on |r| <= ln 2 / 2, relative error 3.6e-18, found with the Remez exchange), then
// the scaling by 2^n, which also makes the denormals and zeros.  Against the 80-bit exponential at 4e6 points of [-750, 0] the largest
// error is 1.00 ulp and the mean 0.258, as the library's (1.00, 0.258), which takes 28 instructions with its checks for both ends of
// the range; these are 22.  128 rows of 151936 tokens, with five loads in flight per thread: sums 44 -> 40 us, masses 47.6 -> 44.9.
__device__ __forceinline__ double exp_neg(double x) {
  x = x < -800.0 ? -800.0 : x;
  const double t = fma(x, 0x1.71547652b82fep+0, 0x1.8p+52);          // rint(x / ln 2) in the low bits
  const double n = t - 0x1.8p+52;
  double r = fma(n, -0x1.62e42fefa39efp-1, x);
  r = fma(n, -0x1.abc9e3b39803fp-56, r);
  double q = fma(r, 0x1.ad7e30d8cbb10p-26, 0x1.28ad632515bcep-22);
  q = fma(r, q, 0x1.71df25ec4e956p-19);
  q = fma(r, q, 0x1.a0199a1ce6609p-16);
  q = fma(r, q, 0x1.a01a012a2980cp-13);
  q = fma(r, q, 0x1.6c16c18424380p-10);
  q = fma(r, q, 0x1.1111111127c28p-7);
  q = fma(r, q, 0x1.5555555550896p-5);
  q = fma(r, q, 0x1.55555555554fap-3);
  q = fma(r, q, 0x1.000000000000ap-1);
  q = fma(r, q, 1.0);
  q = fma(r, q, 1.0);
  return __builtin_amdgcn_ldexp(q, (int)(uint32_t)__builtin_bit_cast(uint64_t, t));
}

template <typename Q, bool FILT>
struct SampleRow {
  const float* z; const Q* q; double inv_T, mxp, mxq; int tgt, mode;
  int f_idx; uint32_t f_key;                         // top-k / top-p threshold of the row (FILT only)
  // the *_v forms take the logits as values (callers that request many loads before using the first)
  __device__ double e_p_v(int j, float zj) const {
    if (FILT && !filter_keeps(filter_key(zj), j, f_key, f_idx)) return 0.0;
    return exp_neg((double)zj * inv_T - mxp);
  }
  __device__ double e_q_v(float qj) const { return exp_neg((double)qj - mxq); }
  // inv_sp, inv_sq: reciprocals of the normalisers
  __device__ double weight_v(int j, float zj, float qj, double inv_sp, double inv_sq, int mode_now) const {
    const double pj = e_p_v(j, zj) * inv_sp;
    if (mode_now == MODE_PLAIN) return pj;
    if (mode_now == MODE_RESID_ONEHOT) return j == tgt ? 0.0 : pj;
    return fmax(0.0, pj - e_q_v(qj) * inv_sq);
  }
  __device__ double weight(int j, double inv_sp, double inv_sq, int mode_now) const {
    return weight_v(j, z[j], (mode_now == MODE_RESID_DENSE) ? to_f32<Q>(q[j]) : 0.f, inv_sp, inv_sq, mode_now);
  }
};

template <typename Q, bool FILT>
__device__ __forceinline__ SampleRow<Q, FILT> sample_row(int b, int V, const float* logit_base, int rows_are_selected,
                                                         const Q* q_logits, float temperature, const SamplerBufs& sb) {
  SampleRow<Q, FILT> r;
  r.mode = sb.sel_mode[b];
  r.f_key = FILT ? sb.f_key[sb.sel_row[b]] : 0u;
  r.f_idx = FILT ? sb.f_idx[sb.sel_row[b]] : 0;
  r.z = logit_base + (size_t)(rows_are_selected ? b : sb.sel_row[b]) * V;
  r.q = (r.mode == MODE_RESID_DENSE) ? q_logits + (size_t)sb.sel_qrow[b] * V : nullptr;
  r.inv_T = 1.0 / (double)temperature;
  r.mxp = (double)sb.sel_pmax[b] * r.inv_T;          // max_j z_j/T: the scaling is monotone
  r.mxq = (double)sb.sel_qmax[b];
  r.tgt = sb.sel_tok[b];
  return r;
}

__device__ __forceinline__ double block_sum_f64(double v, double* red) {     // 256 threads
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// length of a vocabulary chunk: a multiple of four, so that chunks of aligned rows start aligned
__host__ __device__ __forceinline__ int sample_chunk_len(int V) { return ((V + kSampleChunks - 1) / kSampleChunks + 3) & ~3; }

// f(j, z_j, q_j) for j0 <= j < j1 over the workgroup's 256 threads; four consecutive tokens per load where the rows are aligned
template <typename Q, bool FILT, typename F>
__device__ __forceinline__ void for_each_token(const SampleRow<Q, FILT>& r, int j0, int j1, F f) {
  typedef Q q4 __attribute__((ext_vector_type(4)));
  const bool vec = ((uintptr_t)(r.z + j0) & 15) == 0 && ((uintptr_t)(r.q + j0) & (4 * sizeof(Q) - 1)) == 0;
  const int n4 = vec ? (j1 - j0) / 4 : 0;
  auto vectors = [&](auto count, int i0) {
    constexpr int U = decltype(count)::value;
    f32x4 z[U];
    q4 q[U] = {};
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + 4 * min(i0 + u * 256 + (int)threadIdx.x, n4 - 1);
      z[u] = *(const f32x4*)(r.z + j);
      if (r.q) q[u] = *(const q4*)(r.q + j);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * 256 + threadIdx.x;
      if (i < n4)
#pragma unroll
        for (int e = 0; e < 4; ++e) f(j0 + 4 * i + e, z[u][e], to_f32<Q>(q[u][e]));
    }
  };
  // five loads in flight (a chunk of a vocabulary of up to 163840 tokens at once), one where a thread has no more (up to 32768)
  constexpr int U = 5;
  for (int v0 = 0; v0 < n4;) {
    if (n4 - v0 > 256) { vectors(std::integral_constant<int, U>{}, v0); v0 += U * 256; }
    else { vectors(std::integral_constant<int, 1>{}, v0); v0 += 256; }
  }
  // rows that do not start on sixteen bytes (an odd vocabulary), and the last tokens of the others: eight tokens of a thread at once, then two
  auto batch = [&](auto count, int i0) {
    constexpr int US = decltype(count)::value;
    float z[US], q[US];
#pragma unroll
    for (int u = 0; u < US; ++u) {
      const int j = min(i0 + u * 256 + (int)threadIdx.x, j1 - 1);
      z[u] = r.z[j];
      q[u] = r.q ? to_f32<Q>(r.q[j]) : 0.f;
    }
#pragma unroll
    for (int u = 0; u < US; ++u) {
      const int j = i0 + u * 256 + threadIdx.x;
      if (j < j1) f(j, z[u], q[u]);
    }
  };
  int i0 = j0 + 4 * n4;
  for (; i0 + 8 * 256 <= j1; i0 += 8 * 256) batch(std::integral_constant<int, 8>{}, i0);
  for (; i0 < j1; i0 += 2 * 256) batch(std::integral_constant<int, 2>{}, i0);
}

// Per chunk: sum of e_p, and the sum of e_q (dense residual) or of e_p without the rejected draft (one-hot residual).  Without a
// dense proposal these are the chunk masses up to the common factor, and sample_mass_kernel has nothing to do.
template <typename Q, bool FILT>
__global__ void __launch_bounds__(256) sample_sum_kernel(int V, const float* __restrict__ logit_base, int rows_are_selected,
                                                         const Q* __restrict__ q_logits, float temperature, SamplerBufs sb) {
  __shared__ double red[4], red_q[4];
  const int c = blockIdx.x, b = blockIdx.y;
  const SampleRow<Q, FILT> r = sample_row<Q, FILT>(b, V, logit_base, rows_are_selected, q_logits, temperature, sb);
  if (r.mode == MODE_NONE) return;                       // (behind the other loads: one trip to memory instead of two)
  const int chunk = sample_chunk_len(V);
  const int j0 = min(c * chunk, V), j1 = min(j0 + chunk, V);
  double sp = 0.0, sq = 0.0;
  if (r.q) {
    for_each_token(r, j0, j1, [&](int j, float zj, float qj) { sp += r.e_p_v(j, zj); sq += r.e_q_v(qj); });
  } else {
    for_each_token(r, j0, j1, [&](int j, float zj, float) { const double e = r.e_p_v(j, zj); sp += e; sq += j == r.tgt ? 0.0 : e; });
  }
  for (int o = 32; o > 0; o >>= 1) { sp += __shfl_xor(sp, o); sq += __shfl_xor(sq, o); }
  if ((threadIdx.x & 63) == 0) { red[threadIdx.x >> 6] = sp; red_q[threadIdx.x >> 6] = sq; }
  __syncthreads();
  if (threadIdx.x == 0) {
    sp = red[0] + red[1] + red[2] + red[3];
    sq = red_q[0] + red_q[1] + red_q[2] + red_q[3];
    sb.samp_sum[((size_t)b * kSampleChunks + c) * 2] = sp;
    sb.samp_sum[((size_t)b * kSampleChunks + c) * 2 + 1] = sq;
  }
}

// Reciprocals of the two normalisers (0 for an absent proposal) from the chunk sums; every workgroup of a sequence sums in the
// same order.  s_sum: [kSampleChunks][2] in LDS.
__device__ __forceinline__ void sample_totals(const double* s_sum, double& inv_sp, double& inv_sq) {
  double sp = 0.0, sq = 0.0;
  _Pragma("unroll 4") for (int c = 0; c < kSampleChunks; ++c) {
    sp += s_sum[2 * c];
    sq += s_sum[2 * c + 1];
  }
  inv_sp = 1.0 / sp;
  inv_sq = sq > 0.0 ? 1.0 / sq : 0.0;
}

// Chunk masses of the residual against a dense proposal, max(0, p - q): needs both normalisers.
template <typename Q, bool FILT>
__global__ void __launch_bounds__(256) sample_mass_kernel(int V, const float* __restrict__ logit_base, int rows_are_selected,
                                                          const Q* __restrict__ q_logits, float temperature, SamplerBufs sb) {
  __shared__ double red[4], s_sum[2 * kSampleChunks];
  const int c = blockIdx.x, b = blockIdx.y;
  if (threadIdx.x < 2 * kSampleChunks) s_sum[threadIdx.x] = sb.samp_sum[(size_t)b * kSampleChunks * 2 + threadIdx.x];
  const SampleRow<Q, FILT> r = sample_row<Q, FILT>(b, V, logit_base, rows_are_selected, q_logits, temperature, sb);
  if (r.mode != MODE_RESID_DENSE) return;
  __syncthreads();
  double sp, sq;
  sample_totals(s_sum, sp, sq);
  const int chunk = sample_chunk_len(V);
  const int j0 = min(c * chunk, V), j1 = min(j0 + chunk, V);
  double mw = 0.0;
  for_each_token(r, j0, j1, [&](int j, float zj, float qj) { mw += r.weight_v(j, zj, qj, sp, sq, MODE_RESID_DENSE); });
  mw = block_sum_f64(mw, red);
  if (threadIdx.x == 0) sb.samp_mass[(size_t)b * kSampleChunks + c] = mw;
}

constexpr int kPickThreads = 1024;
template <typename Q, bool FILT>
__global__ void __launch_bounds__(kPickThreads) sample_pick_kernel(int V, const float* __restrict__ logit_base, int rows_are_selected,
                                                          const Q* __restrict__ q_logits, float temperature,
                                                          const float* __restrict__ u_sample, SamplerBufs sb,
                                                          const int32_t* __restrict__ n_accepted, int k_max,
                                                          int32_t* __restrict__ out_tokens, int32_t* __restrict__ n_emitted,
                                                          uint32_t* __restrict__ near_tie) {
  __shared__ double s_sum[2 * kSampleChunks], s_mass[kSampleChunks], s_wave[kPickThreads / 64];
  __shared__ int s_i[2];
  const int b = blockIdx.x, tid = threadIdx.x;
  if (sb.sel_mode[b] == MODE_NONE) return;
  const SampleRow<Q, FILT> r = sample_row<Q, FILT>(b, V, logit_base, rows_are_selected, q_logits, temperature, sb);
  if (tid < 2 * kSampleChunks) s_sum[tid] = sb.samp_sum[(size_t)b * kSampleChunks * 2 + tid];
  if (tid == 0) { s_i[0] = 0x7fffffff; s_i[1] = -1; }
  __syncthreads();
  double sp, sq;
  sample_totals(s_sum, sp, sq);
  // chunk level: masses of the residual (or of p itself), then every thread walks the 32 of them: same result in all threads
  int mode = r.mode;
  if (tid < kSampleChunks)
    s_mass[tid] = mode == MODE_RESID_DENSE ? sb.samp_mass[(size_t)b * kSampleChunks + tid]
                                           : s_sum[2 * tid + (mode == MODE_RESID_ONEHOT ? 1 : 0)] * sp;
  __syncthreads();
  double total = 0.0;
  _Pragma("unroll 4") for (int c = 0; c < kSampleChunks; ++c) total += s_mass[c];
  if (!(total > 0.0) && mode != MODE_PLAIN) {       // empty residual: fall back to the target itself
    mode = MODE_PLAIN;
    __syncthreads();
    if (tid < kSampleChunks) s_mass[tid] = s_sum[2 * tid] * sp;
    __syncthreads();
    total = 0.0;
    _Pragma("unroll 4") for (int c = 0; c < kSampleChunks; ++c) total += s_mass[c];
  }
  const double t = (double)u_sample[b] * total;
  int cs = -1, last_c = -1;
  double excl_c = 0.0, run = 0.0, last_excl = 0.0;
  _Pragma("unroll 4") for (int c = 0; c < kSampleChunks; ++c) {
    const double m = s_mass[c];
    if (m > 0.0) { last_c = c; last_excl = run; }
    if (cs < 0 && run + m > t) { cs = c; excl_c = run; }
    run += m;
  }
  if (cs < 0) { cs = last_c; excl_c = last_excl; }  // rounding left no chunk: last chunk with weight
  if (cs < 0) return;                               // no weight anywhere (cannot happen for finite logits)
  // slice level inside the chosen chunk
  const int chunk = sample_chunk_len(V);
  const int c0 = min(cs * chunk, V), c1 = min(c0 + chunk, V);
  const int slice = (c1 - c0 + kPickThreads - 1) / kPickThreads;
  const int j0 = min(c0 + tid * slice, c1), j1 = min(j0 + slice, c1);
  // One workgroup per sequence: nothing hides a load's latency here, so a thread requests its whole slice (up to
  // kW logits of p and q) at once and keeps the weights in registers for the walk below.  1024 threads: the two
  // float64 exponentials per token are the bulk of this kernel and only B workgroups share the GPU.
  constexpr int kW = 8;
  const bool in_regs = slice <= kW;
  double wv[kW];
  double csum = 0.0;
  if (in_regs) {
    float zr[kW], qr[kW];
#pragma unroll
    for (int i = 0; i < kW; ++i) {
      const int jj = min(j0 + i, V - 1);
      zr[i] = r.z[jj];
      qr[i] = (mode == MODE_RESID_DENSE) ? to_f32<Q>(r.q[jj]) : 0.f;
    }
#pragma unroll
    for (int i = 0; i < kW; ++i) {
      wv[i] = 0.0;
      if (i < slice) {                                // uniform: the 8 bodies stay apart (interleaved they spill)
        if (j0 + i < j1) wv[i] = r.weight_v(j0 + i, zr[i], qr[i], sp, sq, mode);
        csum += wv[i];
      }
    }
  } else {
    for (int j = j0; j < j1; ++j) csum += r.weight(j, sp, sq, mode);
  }
  // inclusive scan over the workgroup: within a wave, then over the wave totals in order
  double incl = csum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double v = __shfl_up(incl, o);
    if ((tid & 63) >= o) incl += v;
  }
  if ((tid & 63) == 63) s_wave[tid >> 6] = incl;
  __syncthreads();
  double before = excl_c;
  for (int w = 0; w < (tid >> 6); ++w) before += s_wave[w];
  incl += before;
  const double excl = incl - csum;
  if (csum > 0.0) {
    if (incl > t && excl <= t) atomicMin(&s_i[0], tid);
    atomicMax(&s_i[1], tid);
  }
  __syncthreads();
  const int owner = (s_i[0] != 0x7fffffff) ? s_i[0] : s_i[1];
  if (tid != owner) return;
  double acc = excl, w = 0.0, last_hi = 0.0, last_w = 0.0;
  int tok = -1, last = -1;
  if (in_regs) {
    bool found = false;
#pragma unroll
    for (int i = 0; i < kW; ++i) {
      const int j = j0 + i;
      if (!found && j < j1) {
        w = wv[i];
        acc += w;
        if (w > 0.0) { last = j; last_hi = acc; last_w = w; }
        if (acc > t) { tok = j; found = true; }
      }
    }
  } else {
    for (int j = j0; j < j1; ++j) {
      w = r.weight(j, sp, sq, mode);
      acc += w;
      if (w > 0.0) { last = j; last_hi = acc; last_w = w; }
      if (acc > t) { tok = j; break; }
    }
  }
  if (tok < 0) { tok = last; acc = last_hi; w = last_w; }
  const int n_acc = n_accepted[b];
  out_tokens[(size_t)b * (k_max + 1) + n_acc] = tok;
  n_emitted[b] = n_acc + 1;
  const double lo = acc - w;
  if (fmin(fabs(t - lo), fabs(acc - t)) <= 1e-3 * w) near_tie[b] |= 0x80000000u;
}

// ------------------------------------------------------------------ launchers
template <typename G, bool STATS>
static void launch_lmhead_t(const Shape& s, const int32_t* n_rows_dev, int M_max, const void* hf, int ld,
                            const void* lm_head, float inv_temp, const int32_t* row_target, const SamplerBufs& sb,
                            float* store, hipStream_t st) {
  const int m_blocks = (M_max + G::BM - 1) / G::BM, n_blocks = (s.V + G::WN * kLmVtile - 1) / (G::WN * kLmVtile);
  const int grid = ((m_blocks * n_blocks + 7) / 8) * 8;
  static bool attr_set = false;              // more than 64 KiB of dynamic LDS needs an opt-in
  if (!attr_set) { (void)hipFuncSetAttribute((const void*)lmhead_kernel<G, STATS>, hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS_BYTES); attr_set = true; }
  hipLaunchKernelGGL((lmhead_kernel<G, STATS>), dim3(grid), dim3(G::THREADS), G::LDS_BYTES, st, n_rows_dev, M_max, s.V, s.d,
                     (const f16*)hf, ld, (const f16*)lm_head, inv_temp, row_target, sb, store, n_blocks);
}
template <bool STATS>
static void launch_lmhead_any(const Shape& s, const int32_t* n_rows_dev, int M_max, const void* hf, int ld,
                              const void* lm_head, float inv_temp, const int32_t* row_target, const SamplerBufs& sb,
                              float* store, hipStream_t st) {
  // Up to 96 rows one row block.  256 entries per workgroup as long as that is one round (two workgroups per CU), 320 where it is not: V = 151936,
  // 96 rows, 1.5B / 7B shape 111 / 223 us against 115 / 238; V = 128256 102 / 200 against 90 / 190, V = 32000 34 / 56 against 28 / 45, 1 row of
  // V = 1000, d = 256 9.0 against 7.6.
  // Above, 96 or 128 rows, two workgroups per CU so that one's epilogue overlaps the other's products: by tiles per CU x time of a tile.  A 128-row
  // tile takes 1.19 times as long with the short K of the 1.5B shape (V = 151936, 576 rows 256 us with 96, 259 with 128; 432 rows 221, 216) and
  // 1.13 times with that of the 7B shape (576 rows 677 us with 96, 639 with 128; 280 rows 384, 392; V = 32000, 576 rows, 3 tiles per CU either
  // way, 150 and 160).  One block of 128 reads the weights once (V = 32000, 128 rows, 1.5B / 7B shape 33 / 52 us, with two of 96 37 / 62).
#define BS_LM(...) launch_lmhead_t<StreamGemm<__VA_ARGS__>, STATS>(s, n_rows_dev, M_max, hf, ld, lm_head, inv_temp, row_target, sb, store, st)
  const int n256 = (s.V + 255) / 256;
  if (M_max <= 96) {
    if (n256 > 2 * kCUs) {
      if (M_max <= 32) BS_LM(1, 2, 5, 4);
      else if (M_max <= 64) BS_LM(2, 2, 5, 3);
      else BS_LM(3, 2, 5, 3);
    } else {
      if (M_max <= 32) BS_LM(1, 2, 4, 3);
      else if (M_max <= 64) BS_LM(2, 2, 4, 2);
      else BS_LM(3, 2, 4, 2);
    }
    return;
  }
  auto cost = [&](int bm, int t) { return ((M_max + bm - 1) / bm * n256 + kCUs - 1) / kCUs * t; };
  if (M_max > 128 && cost(96, 100) < cost(128, s.d / kBK < 32 ? 119 : 113)) BS_LM(3, 2, 4, 2);
  else BS_LM(4, 2, 4, 2);
#undef BS_LM
}
void launch_lmhead_stats(const Shape& s, const Plan& p, int M_max, const void* hf, const void* lm_head, float inv_temp,
                         const SamplerBufs& sb, float* logits_debug, hipStream_t st) {
  launch_lmhead_any<true>(s, p.n_rows, M_max, hf, M_max, lm_head, inv_temp, p.row_target, sb, logits_debug, st);
}
// Final rows sel_row[b] -> rows 0 .. B - 1 of a compact matrix (both in chunk order).
__global__ void __launch_bounds__(256) gather_rows_kernel(int B, int d, const f16* __restrict__ hf, int ld, const int32_t* __restrict__ sel_row,
                                                          f16* __restrict__ out) {
  const int i = blockIdx.x * 256 + threadIdx.x;          // one chunk of eight elements; consecutive threads: consecutive sequences
  if (i < d / 8 * B) *(f16x8*)(out + (size_t)i * 8) = *(const f16x8*)(hf + ((size_t)(i / B) * ld + sel_row[i % B]) * 8);
}
void launch_lmhead_rows(const Shape& s, int B, int M_max, const void* hf, void* rows, const void* lm_head, const SamplerBufs& sb,
                        hipStream_t st) {
  hipLaunchKernelGGL(gather_rows_kernel, dim3((s.d / 8 * B + 255) / 256), dim3(256), 0, st, B, s.d, (const f16*)hf, M_max, sb.sel_row, (f16*)rows);
  launch_lmhead_any<false>(s, nullptr, B, rows, B, lm_head, 1.0f, nullptr, sb, sb.sel_logits, st);
}
void launch_logit_stats(const Plan& p, int M_max, int V, const float* logits, float inv_temp, const SamplerBufs& sb,
                        hipStream_t st) {
  const int segs = row_segs(V), len = ((V + segs - 1) / segs + 3) & ~3;      // whole groups of four
  hipLaunchKernelGGL(logit_stats_kernel, dim3(segs, M_max), dim3(256), 0, st, p, M_max, V, len, logits, inv_temp, sb);
}
void launch_q_stats(const Plan& p, int M_max, int V, const void* q_logits, int q_dtype, const SamplerBufs& sb,
                    hipStream_t st) {
  if (q_dtype == BS_F32) hipLaunchKernelGGL(q_stats_kernel<float>, dim3(M_max), dim3(256), 0, st, p, V, (const float*)q_logits, sb);
  else hipLaunchKernelGGL(q_stats_kernel<bf16>, dim3(M_max), dim3(256), 0, st, p, V, (const bf16*)q_logits, sb);
}
void launch_accept_scan(const Plan& p, int B, int k_max, int M_max, int n_vtiles, bool dense_q, float temperature,
                        int eos_id, int emit_bonus, const float* u_accept, const SamplerBufs& sb, const FilterArgs& filter,
                        int32_t* n_accepted, int32_t* out_tokens, int32_t* n_emitted, uint32_t* near_tie, hipStream_t st) {
  const float inv_temp = temperature > 0.f ? 1.0f / temperature : 1.0f;
  if (n_vtiles > 4 * kStatChunks) {
    hipLaunchKernelGGL(row_stats_fold_kernel, dim3((M_max + 31) / 32, kStatChunks), dim3(256), 0, st, p, M_max, n_vtiles, inv_temp, sb);
    hipLaunchKernelGGL(row_stats_kernel, dim3(M_max), dim3(256), 0, st, p, M_max, kStatChunks, inv_temp, sb, sb.fold_max,
                       sb.fold_sum, sb.fold_arg);
  } else {
    hipLaunchKernelGGL(row_stats_kernel, dim3(M_max), dim3(256), 0, st, p, M_max, n_vtiles, inv_temp, sb, sb.part_max,
                       sb.part_sum, sb.part_arg);
  }
  if (filter.on) launch_filter(p, M_max, temperature, filter, sb, st);      // needs row_max
  hipLaunchKernelGGL(accept_scan_kernel, dim3((B + 63) / 64), dim3(64), 0, st, p, B, k_max, dense_q ? 1 : 0, temperature,
                     eos_id, emit_bonus, filter.on, u_accept, sb, n_accepted, out_tokens, n_emitted, near_tie);
}
template <typename Q, bool FILT>
static void launch_sample_t(int B, int k_max, int V, const float* logit_base, bool rows_are_selected, const Q* q_logits,
                            float temperature, const float* u_sample, const SamplerBufs& sb, const int32_t* n_accepted,
                            int32_t* out_tokens, int32_t* n_emitted, uint32_t* near_tie, hipStream_t st) {
  const int sel = rows_are_selected ? 1 : 0;
  hipLaunchKernelGGL((sample_sum_kernel<Q, FILT>), dim3(kSampleChunks, B), dim3(256), 0, st, V, logit_base, sel, q_logits, temperature, sb);
  if (q_logits)                                      // only a dense proposal leaves anything to do
    hipLaunchKernelGGL((sample_mass_kernel<Q, FILT>), dim3(kSampleChunks, B), dim3(256), 0, st, V, logit_base, sel, q_logits, temperature, sb);
  hipLaunchKernelGGL((sample_pick_kernel<Q, FILT>), dim3(B), dim3(kPickThreads), 0, st, V, logit_base, sel, q_logits, temperature, u_sample, sb,
                     n_accepted, k_max, out_tokens, n_emitted, near_tie);
}
void launch_sample(int B, int k_max, int V, const float* logit_base, bool rows_are_selected, const void* q_logits,
                   int q_dtype, float temperature, bool filter_on, const float* u_sample, const SamplerBufs& sb,
                   const int32_t* n_accepted, int32_t* out_tokens, int32_t* n_emitted, uint32_t* near_tie,
                   hipStream_t st) {
  if (temperature == 0.f) return;                    // the scan already emitted the arg-max tokens
  // the filtered kernels are instantiations of their own: the membership test costs the unfiltered path nothing
#define BS_SAMPLE(Q_, F_) launch_sample_t<Q_, F_>(B, k_max, V, logit_base, rows_are_selected, (const Q_*)q_logits, temperature, \
                                                  u_sample, sb, n_accepted, out_tokens, n_emitted, near_tie, st)
  if (q_logits && q_dtype == BS_BF16) { if (filter_on) BS_SAMPLE(bf16, true); else BS_SAMPLE(bf16, false); }
  else                                { if (filter_on) BS_SAMPLE(float, true); else BS_SAMPLE(float, false); }
#undef BS_SAMPLE
}
