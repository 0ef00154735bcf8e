// Device-side planning of one verify step, KV commit, status word.
//
// draft_len may be produced on the device by the lookup kernel, so the packing of the ragged
// query rows (Alg. 1: every sequence verifies its own block of k_b drafts; Sec. 3.3: all query
// lengths ride in one batch) is computed here, on the device, with no host round trip.
#include "common.h"

constexpr int kPlanThreads = 1024;
constexpr int kPlanMaxB = 4096;                     // checked at context creation

// Exclusive prefix sum over the workgroup of one value per thread; `total` receives the sum.  s_part: kPlanThreads / 64
// words.  Called by all threads.
__device__ __forceinline__ int block_exclusive_scan(int v, int* s_part, int& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(incl, o);
    if (lane >= o) incl += t;
  }
  __syncthreads();                                  // s_part of an earlier scan is no longer read
  if (lane == 63) s_part[wave] = incl;
  __syncthreads();
  int before = 0, sum = 0;
#pragma unroll
  for (int w = 0; w < kPlanThreads / 64; ++w) {
    const int t = s_part[w];
    if (w < wave) before += t;
    sum += t;
  }
  total = sum;
  return before + incl - v;
}

// One workgroup plans the step, and every later kernel waits for it: what bounds it is the chain of dependent loads
// (slot -> committed length -> block table -> lists), so every phase spreads over 1024 threads and no phase is walked
// by one thread.  Measured, 7B shape: batch 8 (contexts near 20000) 33 -> 13 us, batch 128 (512 .. 32768) 48 -> 18 us.
__global__ void __launch_bounds__(kPlanThreads) plan_kernel(Plan p, KvView kv, int B, int k_max, int vocab,
                                                   const int32_t* __restrict__ seq_slot,
                                                   const int32_t* __restrict__ last_token,
                                                   const int32_t* __restrict__ draft_tokens,
                                                   const int32_t* __restrict__ draft_len, int need_kv, AttnPlan attn,
                                                   int n_layers) {
  __shared__ int s_fault;
  __shared__ int s_slot[kPlanMaxB];
  __shared__ int s_k[kPlanMaxB];                    // validated k_b (-1: skipped)
  __shared__ int s_c[kPlanMaxB];                    // c_b, later the sequence's number of tiles
  __shared__ int s_r[kPlanMaxB];                    // first packed row
  __shared__ int s_part[kPlanThreads / 64];
  const int tid = threadIdx.x;
  if (tid == 0) s_fault = 0;
  if (need_kv)
    for (int b = tid; b < B; b += kPlanThreads) s_slot[b] = seq_slot[b];
  if (need_kv && attn.s_min > 0)
    for (int i = tid; i < 8 * n_layers; i += kPlanThreads) p.attn_queue[i] = 0;
  __syncthreads();
  // phase 1: per-sequence validation.  16 lanes share a sequence: each repeats the scalar checks (same addresses: one
  // transaction) and takes a share of the duplicate-slot scan, of the block-table entries (four loads in flight) and of
  // the token ids.
  constexpr int SUBS = 16;
  for (int b = tid / SUBS; b < B; b += kPlanThreads / SUBS) {
    const int sub = tid % SUBS;
    int k = draft_len[b], fault = 0, c = 0, slot = 0;
    if (k < 0 || k > k_max) { fault |= BS_FAULT_DRAFT_LEN; }
    if (need_kv) {
      slot = s_slot[b];
      if (slot < 0 || slot >= kv.n_slots) {
        fault |= BS_FAULT_SLOT;
      } else {
        c = kv.ctx_len[slot];
        for (int b2 = sub; b2 < b; b2 += SUBS) if (s_slot[b2] == slot) fault |= BS_FAULT_SLOT;
        if (!(fault & BS_FAULT_DRAFT_LEN)) {
          if (c < 0 || (long)c + k + 1 > (long)kv.max_pages * kPage) {
            fault |= BS_FAULT_KV_PAGES;
          } else {
            const int32_t* bt = kv.block_table + (size_t)slot * kv.max_pages;
            const int last = (c + k) / kPage;
            for (int pg0 = sub; pg0 <= last; pg0 += 4 * SUBS) {
              int id[4];
#pragma unroll
              for (int u = 0; u < 4; ++u) id[u] = bt[min(pg0 + u * SUBS, last)];
#pragma unroll
              for (int u = 0; u < 4; ++u) if (id[u] < 0 || id[u] >= kv.n_pages) fault |= BS_FAULT_KV_PAGES;
            }
          }
        }
      }
    }
    // token ids of the sequence's rows (the last token and the k drafts): a sequence with an id outside the
    // vocabulary is skipped like one with a bad draft length (no row is embedded, appended or judged)
    if (!(fault & BS_FAULT_DRAFT_LEN)) {
      if (sub == 0 && last_token) {
        const int t = last_token[b];
        if (t < 0 || t >= vocab) fault |= BS_FAULT_TOKEN_ID;
      }
      for (int i = sub; i < k; i += SUBS) {
        const int t = draft_tokens[(size_t)b * k_max + i];
        if (t < 0 || t >= vocab) fault |= BS_FAULT_TOKEN_ID;
      }
    }
#pragma unroll
    for (int o = 1; o < SUBS; o <<= 1) fault |= __shfl_xor(fault, o);
    if (sub == 0) {
      p.seq_k[b] = fault ? -1 : k;
      s_k[b] = fault ? -1 : k;
      s_c[b] = c;
      p.seq_c[b] = c;
      p.seq_slot[b] = slot;
      if (fault) atomicOr(&s_fault, fault);
    }
  }
  __syncthreads();
  // phase 2: prefix sums over the sequences (each thread a contiguous range)
  const int per = (B + kPlanThreads - 1) / kPlanThreads;
  const int b_lo = min(tid * per, B), b_hi = min(b_lo + per, B);
  {
    int r = 0, t = 0, n_r, n_t;
    for (int b = b_lo; b < b_hi; ++b) if (s_k[b] >= 0) { r += s_k[b] + 1; t += s_k[b]; }
    r = block_exclusive_scan(r, s_part, n_r);
    t = block_exclusive_scan(t, s_part, n_t);
    for (int b = b_lo; b < b_hi; ++b) {
      p.row_start[b] = r;
      s_r[b] = r;
      p.draft_start[b] = t;
      if (s_k[b] >= 0) { r += s_k[b] + 1; t += s_k[b]; }
    }
    if (tid == 0) {
      p.row_start[B] = n_r;
      p.draft_start[B] = n_t;
      p.n_rows[0] = n_r;
      p.n_rows[1] = n_t;
      if (s_fault) atomicOr(p.status, s_fault);
    }
  }
  __syncthreads();
  // phase 3: per-row maps (parallel over sequences x positions)
  for (int idx = tid; idx < B * (k_max + 1); idx += kPlanThreads) {
    int b = idx / (k_max + 1), i = idx % (k_max + 1);
    int k = s_k[b];
    if (k < 0 || i > k) continue;
    int r = s_r[b] + i;
    // every id was validated in phase 1 (a sequence with a bad one has s_k[b] = -1 and is skipped above)
    const int tok = (i == 0) ? (last_token ? last_token[b] : 0) : draft_tokens[(size_t)b * k_max + i - 1];
    const int tgt = (i < k) ? draft_tokens[(size_t)b * k_max + i] : -1;
    p.row_seq[r] = b;
    p.row_pos[r] = i;
    p.row_tok[r] = tok;
    p.row_target[r] = tgt;
  }
  if (!need_kv || attn.s_min <= 0) return;

  // phase 4: attention work list.  The (sequence, KV head) streams of a ragged batch differ in length by
  // orders of magnitude (contexts of 512 .. 32768 tokens in one step), and a small batch has fewer streams than the
  // chip has CUs, so the token range of every sequence is cut into chunks of a common size; the attention kernel's
  // persistent workgroups walk the (sequence, chunk) items, of which each is `pairs` workgroup tasks (KV heads x query
  // blocks).  The size is the one that attn_chunk_cost says is fastest among kAttnCandidates (eight threads each).
  // sum_b chunks(b) <= B + 4 S, S = max(B, s_min), always (the work list's capacity).
  __shared__ float s_cost[kAttnCandidates];
  __shared__ int s_cand[kAttnCandidates];
  __shared__ int s_cht;
  int T, nv, mx = 0;
  {
    int t = 0, n_valid = 0;
    for (int b = b_lo; b < b_hi; ++b) {
      const int n = s_k[b] < 0 ? 0 : (s_c[b] + s_k[b] + 1 + kTile - 1) / kTile;
      s_c[b] = n;                                        // from here on: tiles of the sequence
      t += n; mx = max(mx, n); n_valid += n > 0;
    }
    block_exclusive_scan(t, s_part, T);
    block_exclusive_scan(n_valid, s_part, nv);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = max(mx, __shfl_xor(mx, o));
    __syncthreads();
    if ((tid & 63) == 0) s_part[tid >> 6] = mx;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kPlanThreads / 64; ++w) mx = max(mx, s_part[w]);
  }
  const int cap = attn_item_capacity(B, attn.s_min);
  // keeps sum_b ceil(n_b / cht) <= cap, and at most 512 chunks per sequence (32-bit offsets of the partial rows)
  const int floor_cht = max(max((T + (cap - B) - 1) / (cap - B), (mx + 511) / 512), 1);
  if (attn.force_chunks > 0) {
    if (tid == 0) s_cht = max((mx + attn.force_chunks - 1) / attn.force_chunks, floor_cht);
  } else {
    const int cand = tid >> 3, sub = tid & 7;            // eight threads share a candidate's count of items
    const int cht = attn_chunk_candidate(attn, cand, T, mx, floor_cht);
    const float inv = 1.0f / (float)cht;
    int items = 0;
    for (int b = sub; b < B; b += 8) items += (int)((float)(s_c[b] + cht - 1) * inv + 1e-4f);   // chunks (a model: +-1 is fine)
    items += __shfl_xor(items, 1);
    items += __shfl_xor(items, 2);
    items += __shfl_xor(items, 4);
    if (sub == 0) {
      s_cost[cand] = attn_chunk_cost(attn, cht, items, T, mx, nv);
      s_cand[cand] = cht;
    }
    __syncthreads();
    if (tid < 64) {                                      // cheapest candidate; equal cost: the larger chunk
      float c0 = s_cost[tid];
      int h0 = s_cand[tid];
      const float c1 = s_cost[tid + 64];
      const int h1 = s_cand[tid + 64];
      if (c1 < c0 || (c1 == c0 && h1 > h0)) { c0 = c1; h0 = h1; }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const float co = __shfl_xor(c0, o);
        const int ho = __shfl_xor(h0, o);
        if (co < c0 || (co == c0 && ho > h0)) { c0 = co; h0 = ho; }
      }
      if (tid == 0) s_cht = h0;
    }
  }
  __syncthreads();
  const int cht = s_cht;
  // Order of the list = order in which the persistent workgroups take the items: every chunk of full size first,
  // then the last (shorter) chunk of every sequence, longest first (64 size classes), so that the work still
  // handed out when the queues run dry is the smallest there is.  item_start[b] keeps numbering a sequence's
  // chunks contiguously (slot item_start[b] + chunk): the partial results are addressed by slot, not by position.
  __shared__ int s_hist[64], s_base[64];
  auto chunks_of = [&](int b) { return (s_c[b] + cht - 1) / cht; };
  auto size_class = [&](int rem) { return 63 - min(63, (int)(((long long)rem * 64 - 1) / cht)); };   // rem in 1 .. cht
  if (tid < 64) s_hist[tid] = 0;
  int n = 0, pf = 0, n_all, n_full;
  for (int b = b_lo; b < b_hi; ++b) { const int nc = chunks_of(b); n += nc; pf += max(nc - 1, 0); }
  n = block_exclusive_scan(n, s_part, n_all);
  pf = block_exclusive_scan(pf, s_part, n_full);
  if (tid == 0) {
    p.item_start[B] = n_all;
    p.attn_meta[0] = cht;
    p.attn_meta[1] = n_all;
  }
  for (int b = b_lo; b < b_hi; ++b) {
    p.item_start[b] = n;
    const int nc = chunks_of(b);
    for (int c = 0; c + 1 < nc; ++c, ++pf) { p.item_seq[pf] = b; p.item_chunk[pf] = c; }
    if (nc > 0) atomicAdd(&s_hist[size_class(s_c[b] - (nc - 1) * cht)], 1);
    n += nc;
  }
  __syncthreads();
  if (tid < 64) {
    const int v = s_hist[tid];
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(incl, o);
      if (tid >= o) incl += t;
    }
    s_base[tid] = n_full + incl - v;                     // after the full-size chunks
    s_hist[tid] = 0;
  }
  __syncthreads();
  for (int b = b_lo; b < b_hi; ++b) {
    const int nc = chunks_of(b);
    if (nc == 0) continue;
    const int cl = size_class(s_c[b] - (nc - 1) * cht);
    const int pos = s_base[cl] + atomicAdd(&s_hist[cl], 1);
    p.item_seq[pos] = b;
    p.item_chunk[pos] = nc - 1;
  }
}

__global__ void commit_kernel(Plan p, KvView kv, int B, const int32_t* __restrict__ seq_slot,
                              const int32_t* __restrict__ n_commit) {
  int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  int k = p.seq_k[b];
  if (k < 0) return;                       // sequence was skipped by the verify step
  int n = n_commit[b];
  if (n < 0 || n > k + 1 || seq_slot[b] != p.seq_slot[b]) { atomicOr(p.status, BS_FAULT_COMMIT); return; }
  kv.ctx_len[p.seq_slot[b]] = p.seq_c[b] + n;
}

__global__ void clear_status_kernel(int32_t* status) { *status = 0; }

// out[b] = committed length of slot seq_slot[b] (-1 and BS_FAULT_SLOT for a slot outside the cache)
__global__ void kv_lengths_kernel(KvView kv, int B, const int32_t* __restrict__ seq_slot, int32_t* __restrict__ out,
                                  int32_t* __restrict__ status) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const int slot = seq_slot[b];
  if (slot < 0 || slot >= kv.n_slots) { out[b] = -1; atomicOr(status, BS_FAULT_SLOT); return; }
  out[b] = kv.ctx_len[slot];
}

void launch_plan(const Plan& p, const KvView& kv, int B, int k_max, int vocab, const int32_t* seq_slot,
                 const int32_t* last_token, const int32_t* draft_tokens, const int32_t* draft_len,
                 bool need_kv, const AttnPlan& attn, int n_layers, hipStream_t st) {
  hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(kPlanThreads), 0, st, p, kv, B, k_max, vocab, seq_slot, last_token,
                     draft_tokens, draft_len, need_kv ? 1 : 0, attn, n_layers);
}
void launch_commit(const Plan& p, const KvView& kv, int B, const int32_t* seq_slot, const int32_t* n_commit,
                   hipStream_t st) {
  hipLaunchKernelGGL(commit_kernel, dim3((B + 255) / 256), dim3(256), 0, st, p, kv, B, seq_slot, n_commit);
}
void launch_kv_lengths(const KvView& kv, int B, const int32_t* seq_slot, int32_t* out, int32_t* status, hipStream_t st) {
  hipLaunchKernelGGL(kv_lengths_kernel, dim3((B + 255) / 256), dim3(256), 0, st, kv, B, seq_slot, out, status);
}
void launch_clear_status(int32_t* status, hipStream_t st) {
  hipLaunchKernelGGL(clear_status_kernel, dim3(1), dim3(1), 0, st, status);
}
