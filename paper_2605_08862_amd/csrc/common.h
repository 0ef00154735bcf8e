// Internal declarations shared by the translation units of libbubblespec (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "../../include/bubblespec.h"

typedef __bf16 bf16;
typedef _Float16 f16;

template <typename T> __device__ __forceinline__ float to_f32(T x);
template <> __device__ __forceinline__ float to_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ float to_f32<bf16>(bf16 x) { return (float)x; }
template <> __device__ __forceinline__ float to_f32<f16>(f16 x) { return (float)x; }
template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ f16 from_f32<f16>(float x) { return (f16)x; }             // RNE
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16 from_f32<bf16>(float x) { return (bf16)x; }  // RNE

// ---------------------------------------------------------------------------------------------
// float16 range guard.  bf16 models keep every matrix operand that is produced during the step
// (normalised rows, rotated queries, appended K/V, attention output, gated MLP activation) in IEEE
// float16, whose largest finite value is 65504.  A producer converts four values at a time and
// tests the packed result: a float16 is infinite or NaN iff its exponent field is all ones, i.e.
// iff (bits & 0x7fff) + 0x0400 carries into bit 15.  When that happens (never for sane models) the
// values are saturated to +-65504 (NaN becomes 0) and BS_FAULT_RANGE is set in the status word, so
// that no infinity or NaN enters a matrix product silently.
// ---------------------------------------------------------------------------------------------
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ bool f16x4_out_of_range(f16x4 v) {
  const u32x2 u = __builtin_bit_cast(u32x2, v);
  return ((((u[0] & 0x7fff7fffu) + 0x04000400u) | ((u[1] & 0x7fff7fffu) + 0x04000400u)) & 0x80008000u) != 0u;
}
__device__ __forceinline__ float f16_saturate(float x) { return x != x ? 0.f : fminf(fmaxf(x, -65504.f), 65504.f); }
// (a, b, c, d) -> four float16 values, saturated and flagged if any leaves the float16 range
__device__ __forceinline__ f16x4 to_f16x4_guarded(float a, float b, float c, float d, int32_t* __restrict__ status) {
  f16x4 v = f16x4{(f16)a, (f16)b, (f16)c, (f16)d};
  if (f16x4_out_of_range(v)) {
    v = f16x4{(f16)f16_saturate(a), (f16)f16_saturate(b), (f16)f16_saturate(c), (f16)f16_saturate(d)};
    atomicOr(status, BS_FAULT_RANGE);
  }
  return v;
}

// ---------------------------------------------------------------------------------------------
// Results that workgroups of ONE launch hand to each other (partial results merged by the last workgroup to arrive).
// The eight XCDs have an L2 each, so a plain store may sit in the writer's L2 and a plain load may hit a stale line of
// the reader's.  A device-scope fence repairs that by writing back and invalidating a whole L2: measured 40 us per
// launch in which 256 workgroups publish 4 KiB each.  The accesses below carry the coherence themselves (sc1: agent
// scope, written through, never served from a stale line): the same launch costs nothing measurable over an empty one.
//   writer:  wt_store*(...) by any threads; publish_arrival() by all threads of the workgroup
//   reader:  the workgroup for which publish_arrival() returned true reads everything with wt_load*
// ---------------------------------------------------------------------------------------------
typedef float wt_f32x4 __attribute__((ext_vector_type(4)));
typedef float wt_f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t wt_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t wt_u32x2 __attribute__((ext_vector_type(2)));
constexpr int kWriteThrough = 16;      // cache-policy bit sc1
typedef __amdgpu_buffer_rsrc_t wt_buf;
// `base` must be uniform within the wave; accesses are addressed by a 32-bit byte offset from it
__device__ __forceinline__ wt_buf wt_buffer(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0xffffffffu, 0x00020000);
}
__device__ __forceinline__ void wt_store4(wt_buf b, uint32_t off, wt_f32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(wt_u32x4, v), b, (int)off, 0, kWriteThrough);
}
__device__ __forceinline__ void wt_store2(wt_buf b, uint32_t off, float x, float y) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(wt_u32x2, wt_f32x2{x, y}), b, (int)off, 0, kWriteThrough);
}
__device__ __forceinline__ wt_f32x4 wt_load4(wt_buf b, uint32_t off) {
  return __builtin_bit_cast(wt_f32x4, __builtin_amdgcn_raw_buffer_load_b128(b, (int)off, 0, kWriteThrough));
}
__device__ __forceinline__ wt_f32x2 wt_load2(wt_buf b, uint32_t off) {
  return __builtin_bit_cast(wt_f32x2, __builtin_amdgcn_raw_buffer_load_b64(b, (int)off, 0, kWriteThrough));
}
// Called by every thread of the workgroup (uniformly) after its wt_stores; `flag` is a __shared__ int.  Counts the
// workgroup as arrived at `counter` and returns true in the one that completes the count n; the counter is then zero
// again for the next launch.  Nobody waits for anybody.
__device__ __forceinline__ bool publish_arrival(int32_t* counter, int n, int* flag) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this thread's stores have reached the coherence point
  __syncthreads();
  if (threadIdx.x == 0) {
    const bool last = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
    if (last) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *flag = last ? 1 : 0;
  }
  __syncthreads();
  const bool r = *flag != 0;
  __syncthreads();                                       // the flag may be reused
  return r;
}

constexpr int kPage = BS_PAGE_TOKENS;   // tokens per KV page
constexpr int kTile = 32;               // tokens per MFMA tile inside a page (bf16 layout)

// ---------------------------------------------------------------------------------------------
// Element order inside one KV page (all heads of one layer, kPage tokens).
//
// float32 pages are row-major [head][token][d] for both K and V.
//
// Pages of bf16 models hold bf16-rounded values (the cache dtype) ENCODED as IEEE float16 (same 16
// bits per element; exact for 6.1e-5 <= |x| <= 65504), so that they are operands of the f16 MFMA
// with no conversion in the attention loop.  They are stored in the operand order of the 32x32x16
// MFMA so that the attention kernel's wave-wide 16-byte-per-lane loads are 1 KiB contiguous and
// feed the matrix unit with no LDS staging and no shuffles.  Per head a page is two tiles of 32 tokens.
//   K tile: S^T = K Q^T uses K as the A operand.  A-row m of the tile holds token
//           tau = 16*(m%8/4) + 4*(m/8) + m%4  (so that accumulator register i of lane group g
//           is token 16g+i), and lane (m, g) needs, at K-step s, d = g*D/2 + 8s + j (j = 0..7;
//           the contraction index may be permuted freely as long as Q uses the same order).
//   V tile: O^T = V^T P^T uses V^T as the A operand, 32 d-values per d-tile; lane (d%32, g) at
//           step t needs tokens 16g + 8t + j.
// ---------------------------------------------------------------------------------------------
__host__ __device__ __forceinline__ size_t kv_page_elems(int Hkv, int D) { return (size_t)Hkv * kPage * D; }

__host__ __device__ __forceinline__ int k_index_f32(int D, int h, int tok, int d) { return (h * kPage + tok) * D + d; }
__host__ __device__ __forceinline__ int v_index_f32(int D, int h, int tok, int d) { return (h * kPage + tok) * D + d; }

__host__ __device__ __forceinline__ int k_tile_row(int tau) {   // token in tile -> A-row m
  return 4 * (tau / 16) + (tau % 4) + 8 * ((tau % 16) / 4);
}
__host__ __device__ __forceinline__ int k_index_bf16(int D, int h, int tok, int d) {
  int tile = tok / kTile, m = k_tile_row(tok % kTile);
  int g = d / (D / 2), r = d % (D / 2), s = r / 8, j = r % 8;
  return ((((h * 2 + tile) * (D / 16) + s) * 2 + g) * 32 + m) * 8 + j;
}
__host__ __device__ __forceinline__ int v_index_bf16(int D, int h, int tok, int d) {
  int tile = tok / kTile, tau = tok % kTile;
  int g = tau / 16, t = (tau % 16) / 8, j = tau % 8, dt = d / 32, dl = d % 32;
  return ((((((h * 2 + tile) * (D / 32) + dt) * 2 + t) * 2 + g) * 32 + dl) * 8) + j;
}
template <typename T> __host__ __device__ __forceinline__ int k_index(int D, int h, int tok, int d);
template <> __host__ __device__ __forceinline__ int k_index<float>(int D, int h, int tok, int d) { return k_index_f32(D, h, tok, d); }
template <> __host__ __device__ __forceinline__ int k_index<bf16>(int D, int h, int tok, int d) { return k_index_bf16(D, h, tok, d); }
template <> __host__ __device__ __forceinline__ int k_index<f16>(int D, int h, int tok, int d) { return k_index_bf16(D, h, tok, d); }
template <typename T> __host__ __device__ __forceinline__ int v_index(int D, int h, int tok, int d);
template <> __host__ __device__ __forceinline__ int v_index<f16>(int D, int h, int tok, int d) { return v_index_bf16(D, h, tok, d); }
template <> __host__ __device__ __forceinline__ int v_index<float>(int D, int h, int tok, int d) { return v_index_f32(D, h, tok, d); }
template <> __host__ __device__ __forceinline__ int v_index<bf16>(int D, int h, int tok, int d) { return v_index_bf16(D, h, tok, d); }

// ---------------------------------------------------------------------------------------------
// Device-side plan of one step (lives in the workspace; written by plan_kernel).
// ---------------------------------------------------------------------------------------------
struct Plan {
  int32_t* status;      // [1]   BS_FAULT_* bits (sticky until polled)
  int32_t* n_rows;      // [7]   M, T_d, choices of the slab GEMMs (SlabRule), the QKV and the gate/up projection (TileRule)
  int32_t* row_start;   // [B+1] first packed row of sequence b (k_b+1 rows each)
  int32_t* draft_start; // [B+1] first packed draft row of sequence b (k_b rows each)
  int32_t* seq_k;       // [B]   validated k_b (-1: sequence skipped)
  int32_t* seq_c;       // [B]   committed length c_b
  int32_t* seq_slot;    // [B]   validated slot
  int32_t* row_seq;     // [M_max] sequence of packed row r
  int32_t* row_pos;     // [M_max] i in 0..k_b
  int32_t* row_tok;     // [M_max] input token of row r
  int32_t* row_target;  // [M_max] draft token judged by row r (-1: none)
  int32_t* row_kv;      // [M_max] cache place of row r: page * kPage + token in the page (embedding kernel; on top of SamplerBufs::row_arg, which is
                        // written after the layers)
  // attention work list (bf16 models): every sequence's token range is cut into chunks of chunk_tiles 32-token
  // tiles; the item at list position i is (sequence item_seq[i], chunk item_chunk[i]) and the list is ordered by
  // decreasing size (full chunks, then the shorter last chunks).  Sequence b has item_start[b+1] - item_start[b]
  // chunks; its chunk c owns SLOT item_start[b] + c, by which partial results are addressed
  int32_t* attn_meta;   // [2]   chunk_tiles, number of items
  int32_t* item_start;  // [B+1]
  int32_t* item_seq;    // [item capacity]
  int32_t* item_chunk;  // [item capacity]
  int32_t* attn_queue;  // [n_layers][8] next position of every XCD's work queue (zeroed by plan_kernel)
};

// Capacity of the attention work list for B sequences when the launch wants at least s_min (sequence, chunk)
// items (see plan_kernel): sum_b chunks(b) <= B + S with S <= 4 max(B, s_min).
__host__ __device__ __forceinline__ int attn_item_capacity(int B, int s_min) { return 5 * (B > s_min ? B : s_min); }
constexpr int kAttnMaxSmin = 256;
constexpr int kAttnWorkgroups = 256;   // persistent workgroups of an attention launch (one per CU)

// How long an attention launch takes for a given chunk size: microseconds throughout, so that candidates of different branches
// of attn_chunk_cost can be compared (constants and what they were fitted to: attention.hip).  A task is one (item, KV head,
// query block); tasks running together take c_item + length * max(t_lat, t_full * tasks / workgroups).
struct AttnPlan {
  int s_min;            // 0: no work list; else items that fill the chip once (capacity of the list)
  int force_chunks;     // > 0 (tests): chunk size such that the longest sequence has that many chunks
  float pairs;          // tasks per item
  float c_item;         // fixed cost of a task: metadata, first loads, merge of its waves
  float t_scale;        // length of a task per 32-token tile
  float t_lat, t_full;  // time per unit of length: alone on the memory system, with every CU streaming
  float t_long, c_tail; // ragged batches of more tasks than workgroups: time per unit of length of the longest piece, end of the launch
  float c_merge, t_merge;   // merge of a sequence's chunks: fixed, per chunk
};
constexpr int kAttnCandidates = 128;
// Candidate i of the common chunk size (tiles) of a batch of T tiles whose longest sequence has mx: the longest sequence in
// 1 .. 64 equal parts, and 1/4 .. 9/4 of the fair share of one workgroup.
__host__ __device__ __forceinline__ int attn_chunk_candidate(const AttnPlan& a, int i, int T, int mx, int floor_cht) {
  const float fair = (float)T * a.pairs / (float)kAttnWorkgroups;
  int cht = i < 64 ? (mx + i) / (i + 1) : (int)(fair * (0.25f + (i - 64) * 0.03125f)) + 1;
  cht = cht < (mx > 1 ? mx : 1) ? cht : (mx > 1 ? mx : 1);
  return cht > floor_cht ? cht : floor_cht;
}
// Modelled time of the launch when a batch of nv sequences with T tiles, the longest mx, is cut into `items` chunks of cht tiles.
__host__ __device__ __forceinline__ float attn_chunk_cost(const AttnPlan& a, int cht, int items, int T, int mx, int nv) {
  const float slots = (float)kAttnWorkgroups, tasks = (float)items * a.pairs, len = cht * a.t_scale;
  float cost;
  if (tasks <= slots) {                                  // all tasks at once
    cost = a.c_item + len * fmaxf(a.t_lat, a.t_full * tasks / slots);
  } else if (4LL * mx * nv <= 5LL * T) {                 // equal tasks: whole rounds and a last one
    const float full = floorf(tasks / slots), rem = tasks - full * slots;
    cost = full * (a.c_item + len * a.t_full);
    if (rem > 0.f) cost += a.c_item + len * fmaxf(a.t_lat, a.t_full * rem / slots);
  } else {                                               // ragged: handed out longest first
    const float avg = (tasks * a.c_item + (float)T * a.pairs * a.t_scale * a.t_full) / slots;
    cost = fmaxf(avg, a.c_item + len * a.t_long) + a.c_tail;
  }
  if (cht < mx) cost += a.c_merge + a.t_merge * (float)((mx + cht - 1) / cht);
  return cost;
}
// Constants for launches whose workgroups hold `tiles_wg` query tiles (1, 2: four waves, a tile each, length in rows of four
// tiles; 4: the wide kernel, eight waves on two or four phases), q_blocks workgroups per (item, KV head).
inline void attn_plan_constants(AttnPlan& a, int tiles_wg, int q_blocks, int Hkv, int D) {
  const float bytes = D / 128.0f;                        // a tile's bytes against head size 128
  a.pairs = (float)(Hkv * q_blocks);
  if (tiles_wg <= 2) {
    a.c_item = 8.0f; a.t_scale = 0.25f; a.t_lat = 1.1f; a.t_full = 2.7f * bytes / q_blocks;
    a.t_long = a.t_full; a.c_tail = 4.0f; a.c_merge = 0.f; a.t_merge = 0.15f;
  } else {
    a.c_item = 14.0f; a.t_scale = 1.0f; a.t_lat = 0.6f; a.t_full = 0.66f * bytes;
    a.t_long = 0.72f * bytes; a.c_tail = 6.0f; a.c_merge = 2.0f; a.t_merge = 1.2f;
  }
}

struct KvView {
  int n_pages, n_slots, max_pages;
  const int32_t* block_table;
  int32_t* ctx_len;
};

// Cache place of a row, looked up once per step (block of a sequence -> slot -> page: three dependent loads that every append of every layer waited for).
__device__ __forceinline__ void row_place(const Plan& p, const KvView& kv, int r) {
  const int b = p.row_seq[r], pos = p.seq_c[b] + p.row_pos[r];
  p.row_kv[r] = kv.block_table[(size_t)p.seq_slot[b] * kv.max_pages + pos / kPage] * kPage + pos % kPage;
}

// cos / sin of the rotary angle of packed row r (absolute position c_b + i) and pair j.  The angle is formed in
// float64 (at positions of 3e4 a float32 angle is already off by ~2e-3 rad), reduced to [-pi, pi] in float64 and
// only then handed to the float32 sine / cosine.
__device__ __forceinline__ void rope_angle(const Plan& p, int r, int j, int half, const double* __restrict__ inv_freq,
                                           float* __restrict__ cos_t, float* __restrict__ sin_t) {
  const int pos = p.seq_c[p.row_seq[r]] + p.row_pos[r];
  const double ang = (double)pos * inv_freq[j];
  const double two_pi_hi = 6.283185307179586, two_pi_lo = 2.4492935982947064e-16;
  const double n = rint(ang * 0.15915494309189535);
  const double red = fma(-n, two_pi_lo, fma(-n, two_pi_hi, ang));
  float sn, cs;
  sincosf((float)red, &sn, &cs);
  cos_t[(size_t)r * half + j] = cs;
  sin_t[(size_t)r * half + j] = sn;
}

struct Shape {
  int L, d, Hq, Hkv, D, F, V, dtype;
  float eps, theta;
  int Nqkv() const { return (Hq + 2 * Hkv) * D; }
};

// ---- launchers (each .hip file defines its own kernels and these host wrappers) ---------------
// plan.hip
// attn.s_min > 0: also build the attention work list.
void launch_plan(const Plan& p, const KvView& kv, int B, int k_max, int vocab, const int32_t* seq_slot,
                 const int32_t* last_token, const int32_t* draft_tokens, const int32_t* draft_len,
                 bool need_kv, const AttnPlan& attn, int n_layers, hipStream_t st);
void launch_commit(const Plan& p, const KvView& kv, int B, const int32_t* seq_slot,
                   const int32_t* n_commit, hipStream_t st);
void launch_clear_status(int32_t* status, hipStream_t st);
void launch_kv_lengths(const KvView& kv, int B, const int32_t* seq_slot, int32_t* out, int32_t* status, hipStream_t st);
// elementwise.hip
// also fills the step's rotary tables cos_t / sin_t [M_max][D/2] (shared by all layers) and the rows' cache places
// rules: those of the step's GEMMs (step_rules); their choices are left behind the row count.
struct StepRules;
void launch_embed(const Shape& s, const Plan& p, const KvView& kv, int M_max, const StepRules& rules, const void* embed, float* h, const double* inv_freq,
                  float* cos_t, float* sin_t, hipStream_t st);
// h[r] += sum of n_slabs slabs [M_max, d] (n_slabs may be 0), then out[r] = RMSNorm(h[r]).
struct SlabCount;
// float32 models: out row-major; bf16 models: chunk order, ld = M_max
void launch_rmsnorm(const Shape& s, const Plan& p, int M_max, float* h, const float* slabs, const SlabCount& n_slabs,
                    const float* gain, void* out, hipStream_t st);
// qkv is the float32 projection, given as slabs [M_max, Nqkv] that are summed.
// inv_freq: [D/2] float64 table written by launch_rope_table.
void launch_rope_table(const Shape& s, double* inv_freq, hipStream_t st);
// cos_t / sin_t: [M_max][D/2] tables of the step's packed rows (filled by launch_embed, once per step).
void launch_rope_append(const Shape& s, const Plan& p, int M_max, const float* cos_t, const float* sin_t,
                        const float* qkv, const SlabCount& slabs, void* q_out, void* k_pages, void* v_pages, hipStream_t st);
void launch_kv_copy(const Shape& s, const KvView& kv, int slot, int pos0, int n, void* k_pages, void* v_pages,
                    void* k_rows, void* v_rows, bool to_pages, int32_t* status, hipStream_t st);
// qkv_rope.hip   QKV projection + rotary + KV append in one kernel (bf16 models with head size 128); A = normed
// rows (float16), Wp = packed wqkv.
bool qkv_rope_applies(const Shape& s, int M_max);
struct TileRule;
TileRule qkv_rope_rule(const Shape& s, int M_max);       // of the step; at == 0: the launch needs none
void launch_qkv_rope(const Shape& s, const Plan& p, int M_max, const TileRule& rule, const void* A, const void* Wp,
                     const float* cos_t, const float* sin_t, void* q_out, void* k_pages, void* v_pages, hipStream_t st);
// Float16 activations of bf16 models (normalised rows, attention output, gated activation, final rows), "chunk order": the eight
// elements k .. k + 7 (k % 8 == 0) of a row are one 16-byte chunk, and the chunks of one k of all rows are neighbours, ld chunks
// from one k to the next (ld: row limit of the step).  The order of the k is that of the packed weights, so a fragment of
// the MFMA (32 rows x 16 of K) is two runs of 512 bytes: GEMMs copy it to LDS as it is, no buffer needs padding rows, and an
// epilogue whose lanes are rows stores runs instead of pieces of rows.
__host__ __device__ __forceinline__ size_t act_index(int row, int k, int ld) {
  return ((size_t)((k >> 6) * 8 + ((k >> 3) & 3) * 2 + ((k >> 5) & 1)) * ld + row) * 8 + (k & 7);
}
// Stores columns 4 ch .. 4 ch + 3 (y0) and 4 (ch + n) .. (y1) of a row, n even: lanes 2 i and 2 i + 1 hold neighbouring ch and exchange
// halves, so that every store is a whole chunk.
__device__ __forceinline__ void store_chunk_pair(f16* out, int row, int col, int ch, int n, int ld, f16x4 y0, f16x4 y1) {
  const bool odd = ch & 1;
  typedef int i2 __attribute__((ext_vector_type(2)));
  const i2 own = __builtin_bit_cast(i2, odd ? y1 : y0), give = __builtin_bit_cast(i2, odd ? y0 : y1);
  const i2 got{__builtin_amdgcn_mov_dpp(give[0], 0xB1, 0xf, 0xf, true), __builtin_amdgcn_mov_dpp(give[1], 0xB1, 0xf, 0xf, true)};   // quad_perm 1 0 3 2
  typedef int i4 __attribute__((ext_vector_type(4)));
  const i4 v = odd ? i4{got[0], got[1], own[0], own[1]} : i4{own[0], own[1], got[0], got[1]};
  *(i4*)(out + act_index(row, col + 4 * (odd ? ch - 1 + n : ch), ld)) = v;
}
// gemm.hip   C[M,N] (+)= A[M,K] * W[N,K]^T with an epilogue.  float32 models: A, W float32 row-major.
// bf16 models: A float16 in chunk order with ld = M_max, W the packed float16 copy made by launch_pack_weight.
constexpr int kCUs = 256;
enum GemmEpilogue { EPI_RESID_ADD = 1, EPI_SWIGLU = 2, EPI_STORE_F32 = 3 };
constexpr int kMaxGemmSplit = 8;
// Time of a float32-result GEMM launch in units of 0.01 us, without its fixed part: rounds of the CUs (cap = two workgroups per CU)
// x K tiles per split x time of a K tile, and what a further slab costs its writer and its reader.
__host__ __device__ __forceinline__ int gemm_split_cost(int tiles, int nk, int cap, int s, int t_tile, int t_slab) {
  const int rounds = (int)ceilf((float)(tiles * s) * (2.0f / (float)cap));
  return (rounds > 0 ? rounds : 1) * ((nk + s - 1) / s) * t_tile + (s - 1) * t_slab;
}
// One slab of M x N float32 written and read at 4.5 TB/s.
__host__ __device__ __forceinline__ int gemm_slab_cost(int M, int N) { return (int)((float)M * (float)N * (1.0f / 5625.0f)); }
// Number of K splits: the one of least time, at most 6, at least 4 K tiles each, all workgroups resident at once.
__host__ __device__ __forceinline__ int gemm_adaptive_split(int tiles, int nk, int cap, int t_tile = 90, int t_slab = 0) {
  int best = 1, cost = gemm_split_cost(tiles, nk, cap, 1, t_tile, t_slab);
#pragma unroll
  for (int s = 2; s <= 6; ++s) {
    const int c = gemm_split_cost(tiles, nk, cap, s, t_tile, t_slab);
    if (4 * s <= nk && tiles * s <= cap && c < cost) { best = s; cost = c; }
  }
  return best;
}
// Number of K-split slabs a float32-epilogue GEMM writes: fixed on the host (bm == 0), or decided on the DEVICE from
// the step's row count M, which only the device knows (draft lengths may come straight from the lookup kernel): the
// launch is sized for the row limit.  The embedding kernel evaluates the rules of a step once, beside its rows, and leaves
// choice(M) behind the row count (Plan::n_rows[at]), where the GEMM and the consumer of its slabs read it with the row count.
// (Evaluated by every workgroup it was some 1500 instructions in front of a GEMM's first load, 650 in front of a normalisation's:
// two layers of d = 256 with 646 .. 1836 rows took 121 .. 168 us where they now take 99 .. 140.)
struct SlabRule {
  int fixed;                    // slab count when bm == 0 (0: the output was updated in place)
  int bm, n_blocks, nk, cap;    // device rule: row tile, column blocks, K tiles, resident workgroups
  int bm_alt;                   // second row tile the producer may choose on the device (0: none)
  int n_blocks_alt = 0;         // its column blocks (0: the same)
  int t = 90, t_alt = 90;       // time of a K tile (gemm_split_cost)
  int slab_cols = 0;            // columns of the output (0: slabs cost nothing)
  int at = 0;                   // device rule: where the choice is
  int tile = 0;                 // gemm.hip: the kernel
  __host__ __device__ int slab_cost(int M) const { return gemm_slab_cost(M, slab_cols); }
  __host__ __device__ int blocks(int b) const { return b == bm_alt && n_blocks_alt > 0 ? n_blocks_alt : n_blocks; }
  // Row tile and slabs of the step (device rule): with two candidates, the tile whose launch is shorter.
  struct Choice { int rows, slabs; };
  __host__ __device__ Choice choice(int M) const {
    Choice best{bm, 1};
    int least = 0;
    for (int i = 0; i < (bm_alt ? 2 : 1); ++i) {
      const int b = i ? bm_alt : bm, tiles = ((M + b - 1) / b) * blocks(b), tt = i ? t_alt : t;
      const int s = gemm_adaptive_split(tiles, nk, cap, tt, slab_cost(M)), cost = gemm_split_cost(tiles, nk, cap, s, tt, slab_cost(M));
      if (i == 0 || cost < least) { best = Choice{b, s}; least = cost; }
    }
    return best;
  }
  __host__ __device__ int tile_rows(int M) const { return choice(M).rows; }
  __host__ __device__ int slabs(int M) const { return bm == 0 ? fixed : choice(M).slabs; }
};
// A choice as one word, and the slab count of a launch as its consumer gets it.
__host__ __device__ __forceinline__ int pack_choice(SlabRule::Choice c) { return c.rows << 4 | c.slabs; }
struct SlabCount {
  int fixed, at;                // at == 0: fixed (0: the output was updated in place)
  __device__ int of(const int32_t* n_rows) const { return at ? n_rows[at] & 15 : fixed; }
};
// The GEMMs of a layer that write slabs.
enum SlabGemm { SLAB_QKV = 0, SLAB_O = 1, SLAB_DOWN = 2 };
// Tile of a launch whose best one depends on the step's row count, decided on the device like a slab choice (evaluated by every workgroup of every
// layer, a choice between six tiles had 283 instructions in front of the first load, 156 now): the tile of least time, rounds of the CUs x K tiles x time of one + what is not
// per K tile (fill, epilogue), 0.01 us.
struct TileRule {
  static constexpr int kMost = 8;
  struct Tile { int rows, blocks, t, fixed; };           // blocks: column blocks of the matrix
  int at = 0, grid = 0;                                  // where the choice is; most workgroups that any row count of the step takes
  int nk = 0, n = 0;
  Tile tile[kMost] = {};
  int waves = 4;                                         // of a workgroup
  int fixed = 0;                                         // at == 0: the launcher's tile for the row limit (0: one row block)
  __host__ __device__ int blocks(int i, int M) const { return (M + tile[i].rows - 1) / tile[i].rows * tile[i].blocks; }
  __host__ __device__ long long cost(int i, int M) const { return (long long)((blocks(i, M) + kCUs - 1) / kCUs) * (nk * tile[i].t) + tile[i].fixed; }
  __host__ __device__ int choice(int M) const {
    int best = 0;
    long long least = 0;
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
      if (i >= n) break;
      const long long c = cost(i, M);
      if (i == 0 || c < least) { best = i; least = c; }
    }
    return best;
  }
  // The choice changes only where the number of row blocks of some tile does: behind multiples of 32 rows.
  void size_grid(int M_max) {
    grid = 0;
    for (int M = 32; M < M_max + 32; M += 32) {
      const int m = M < M_max ? M : M_max, b = blocks(choice(m), m);
      grid = b > grid ? b : grid;
    }
  }
};
// The rules of a step, made once on the host, and the place of each choice behind the row count and the number of drafts (Plan::n_rows).
struct StepRules { SlabRule slab[3]; TileRule qkv, glu; };
enum StepChoice { CHOICE_SLABS = 2, CHOICE_QKV = CHOICE_SLABS + 3, CHOICE_GLU };
void gemm_slab_rules(const Shape& s, int M_max, SlabRule (&r)[3]);
TileRule gate_up_rule(const Shape& s, int M_max);        // at == 0: one row block, or a float32 model
inline StepRules step_rules(const Shape& s, int M_max) {
  StepRules r;
  gemm_slab_rules(s, M_max, r.slab);
  r.qkv = qkv_rope_rule(s, M_max);
  r.glu = gate_up_rule(s, M_max);
  return r;
}
// status: the step's device status word (float16-range faults of the float16 epilogues).  rule, glu: step_rules, made once per step
// (EPI_RESID_ADD / EPI_STORE_F32 and EPI_SWIGLU of bf16 models; made in each launch it kept steps of small models waiting for the host).  Returns the slabs written (these GEMMs: `out` is the slab buffer [split][M_max][N]
// and the consumer sums them), none where `out` was updated in place (float32 models).
SlabCount launch_gemm(int dtype, GemmEpilogue epi, const int32_t* n_rows_dev, int M_max, int N, int K, const void* A, const void* W, void* out,
                      int32_t* status, hipStream_t st, const SlabRule& rule = SlabRule{}, const TileRule& glu = TileRule{});
// time (0.01 us, without the fixed part of a launch) of an EPI_STORE_F32 launch of at most 640 rows
int gemm_slab_time(int M_max, int N, int K);
size_t packed_weight_elems(int N, int K);
void launch_pack_weight(const void* w_bf16, int N, int K, void* packed_f16, int32_t* status, hipStream_t st);
// skinny.hip   decoder layer of steps with at most kSkinnyRows packed rows (bf16 models with head size 128); activations in chunk
// order with ld = kSkinnyRows (a fragment is one contiguous KiB), the residual in fragment order.
constexpr int kSkinnyRows = 32;
// The float32 residual of these steps: a fragment (act_index) is two contiguous KiB, k .. k + 3 (k % 4 == 0) contiguous.
__host__ __device__ __forceinline__ size_t h_frag_index(int row, int k, int nk) {
  return ((size_t)((row >> 5) * nk + (k >> 6)) * 8 + ((k >> 3) & 3) * 2 + ((k >> 2) & 1)) * 256 + (((k >> 5) & 1) * 32 + (row & 31)) * 4 + (k & 3);
}
struct SkinnyBufs { float* part; int32_t* counters; };   // partial tiles of K splits; arrival counters (zero between launches)
bool skinny_applies(const Shape& s, int M_max);
// ssq: [parts][32] sums of squares of the residual's rows over column ranges (embed: 1 part, residual projections: d / 32)
void launch_skinny_embed(const Shape& s, const Plan& p, const KvView& kv, const void* embed, float* h, float* ssq, const double* inv_freq,
                         float* cos_t, float* sin_t, hipStream_t st);
void launch_skinny_final_norm(const Shape& s, const Plan& p, int M_max, const float* h, const float* ssq, const float* gain,
                              void* out, hipStream_t st);
void launch_skinny_qkv(const Shape& s, const Plan& p, int M_max, const float* h, const float* ssq, int ssq_parts,
                       const float* gain, const void* W, const float* cos_t, const float* sin_t, void* q_out, void* k_pages,
                       void* v_pages, const SkinnyBufs& sk, hipStream_t st);
void launch_skinny_gate_up(const Shape& s, const Plan& p, int M_max, const float* h, const float* ssq, int ssq_parts, const float* gain, void* a,
                           const void* W, void* act, hipStream_t st);      // a: scratch for the normalised rows
void launch_skinny_resid(const Shape& s, const Plan& p, int M_max, int K, const void* X, const void* W, float* h, float* ssq,
                         const SkinnyBufs& sk, hipStream_t st);
// attention.hip
// out_ld: ld of the output rows (bf16 models: chunk order, act_index).
// attention_plan_params gives the work-list parameters launch_plan needs for the same (B, k_max);
// launch_attention_init clears the completion counters once, at context creation.
// ahead: weights that the launches behind this one will stream, for workgroups that have no unit (attention.hip).
AttnPlan attention_plan_params(const Shape& s, int B, int k_max);
struct ReadAhead { const void* base; size_t bytes; };
void launch_attention_init(const Shape& s, int B_max, void* scratch, hipStream_t st);
void launch_zero_i32(int32_t* p, int n, hipStream_t st);
void launch_attention(const Shape& s, const Plan& p, const KvView& kv, int layer, int B, int B_max, int k_max, int M_max,
                      const void* q, const void* k_pages, const void* v_pages, void* out, int out_ld, void* scratch,
                      const ReadAhead& ahead, void* prof_token, hipStream_t st);
void attention_prof_mark(void* token, hipStream_t st, bool begin);   // api.hip: event pair around the main kernel
size_t attention_scratch_bytes(const Shape& s, int B_max, int k_max);
// sampler.hip
struct SamplerBufs {
  float* part_max; float* part_sum; int32_t* part_arg;   // [n_vtiles, M_max]
  float* fold_max; float* fold_sum; int32_t* fold_arg;   // [16, M_max] tile entries folded over 16 vocabulary ranges
  float* z_target;                                       // [M_max] logit of the judged draft token
  float* row_max; float* row_lse; int32_t* row_arg;      // [M_max] combined statistics of each packed row
  float* q_max; float* q_lse; float* q_target;           // [M_max] per query row that judges a draft
  int32_t* sel_row; int32_t* sel_mode; int32_t* sel_qrow; int32_t* sel_tok; // [B_max]
  float* sel_pmax; float* sel_qmax;                      // [B_max] raw maxima of the sampled row / its q row
  double* samp_sum; double* samp_mass;                   // [B_max, 32 chunks, 2], [B_max, 32] sampling partials
  float* sel_logits;                                     // [B_max, V]
  uint32_t* f_key; int32_t* f_idx; float* f_lse;         // [M_max] top-k / top-p threshold of each row (filter.hip)
};

// Ranking key of a logit for the top-k / top-p filter: unsigned order == numeric order (-0 counts as +0), so
// "token j of row r is kept" reads  key > f_key[r] || (key == f_key[r] && j <= f_idx[r]).
__device__ __forceinline__ uint32_t filter_key(float z) {
  if (z == 0.0f) z = 0.0f;
  const uint32_t u = __float_as_uint(z);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ bool filter_keeps(uint32_t key, int j, uint32_t f_key, int f_idx) {
  return key > f_key || (key == f_key && j <= f_idx);
}
struct FilterArgs { int on; int top_k; float top_p; const float* logits; int V; };
// Statistics entries per row of the plain-logits path: vocabulary segments, a workgroup each.  No shorter than 1024 entries (four
// per thread): with 16 segments whatever the length, 990 rows of 1000 entries took 69 us for the whole call, with one 59.
constexpr int kMaxRowSegs = 16;
inline int row_segs(int V) { return V >= kMaxRowSegs * 1024 ? kMaxRowSegs : (V + 1023) / 1024; }
int lmhead_vtiles(int V);
int lmhead_logit_rows(const Shape& s);
void launch_lmhead_stats(const Shape& s, const Plan& p, int M_max, const void* hf, const void* lm_head,
                         float inv_temp, const SamplerBufs& sb, float* logits_debug, hipStream_t st);
void launch_logit_stats(const Plan& p, int M_max, int V, const float* logits, float inv_temp,
                        const SamplerBufs& sb, hipStream_t st);
// rows: scratch for the B selected rows [d] of hf (chunk order, ld = M_max; sb.sel_row), float16
void launch_lmhead_rows(const Shape& s, int B, int M_max, const void* hf, void* rows, const void* lm_head, const SamplerBufs& sb,
                        hipStream_t st);
void launch_q_stats(const Plan& p, int M_max, int V, const void* q_logits, int q_dtype, const SamplerBufs& sb,
                    hipStream_t st);
void launch_accept_scan(const Plan& p, int B, int k_max, int M_max, int n_vtiles, bool dense_q, float temperature,
                        int eos_id, int emit_bonus, const float* u_accept, const SamplerBufs& sb, const FilterArgs& filter,
                        int32_t* n_accepted, int32_t* out_tokens, int32_t* n_emitted, uint32_t* near_tie, hipStream_t st);
void launch_sample(int B, int k_max, int V, const float* logit_base, bool rows_are_selected, const void* q_logits,
                   int q_dtype, float temperature, bool filter_on, const float* u_sample, const SamplerBufs& sb,
                   const int32_t* n_accepted, int32_t* out_tokens, int32_t* n_emitted, uint32_t* near_tie,
                   hipStream_t st);
// filter.hip   per-row threshold of the top-k / top-p filter (needs row_max of the same logits)
constexpr int kFilterMaxVocab = 262136;
void launch_filter(const Plan& p, int M_max, float temperature, const FilterArgs& filter, const SamplerBufs& sb,
                   hipStream_t st);
// index.hip   prebuilt suffix-automaton index: header check (host copy of the first 8 words) and the device walk
bool index_header_ok(const int32_t* header_host, size_t bytes, int* n_prompts);
void launch_index_lookup(const int32_t* blob, int n_prompts, const int32_t* seq_prompt, const int32_t* tail, int B,
                         int max_match, int min_match, int k_max, int32_t* draft_tokens, int32_t* draft_len,
                         hipStream_t st);
// lookup.hip
void launch_lookup(int B, int n_prompts, const int32_t* pool_tokens, const int64_t* rollout_offsets,
                   const int32_t* prompt_rollout_begin, const int32_t* seq_prompt, const int32_t* tail,
                   int max_match, int min_match, int k_max, int32_t* draft_tokens, int32_t* draft_len,
                   hipStream_t st);
