// Verify attention for batches in which a sequence may have three or four 32-row query tiles per KV head
// ((k_b + 1) * G > 64 query rows: long draft blocks on wide GQA groups, Sec. 3.3's "unified" launch at its
// widest).  Same work list, page layout, partial results and last-arriver merge (write-through, no fence) as attn_mfma_kernel in
// attention.hip; what differs is how a workgroup spends a CU.
//
// With four query tiles the step is no longer a pure stream: per 32-token K/V tile (16 KiB at head size 128) a
// CU owes 64 MFMAs and four softmax passes.  One wave per SIMD that owns two query tiles (the narrow kernel) issues
// ~21 vector instructions per MFMA and then waits for its own loads: measured on the long-tail batch, the matrix
// unit was busy 10 % of the time, the waves waited 36 % of it, and the kernel reached 2.5 TB/s although L2 served
// the second reader of every tile (fetched bytes 1.07 x algorithmic).  Here a workgroup has EIGHT waves, two per
// SIMD, so that one wave's softmax and LDS traffic overlap the other's MFMAs and waits, and every wave owns ONE
// query tile (64 accumulator registers), which is what lets two waves share a SIMD's 512 registers:
//   * wave w = (query tile qt = w % NQT, token phase ph = w / NQT), NQT = 2 or 4 query tiles per unit; the 8 / NQT
//     phases work on different token tiles of the chunk at the same time;
//   * the NQT waves of a phase share one K/V tile through LDS: each moves 1 / NQT of its 1 KiB fragments (the page layout is
//     already fragment order, so the LDS image is a straight copy and every LDS access is a conflict-free 1 KiB sweep), so K/V
//     leave HBM once per unit whatever the number of query tiles, with no reliance on L2;
//   * four query tiles: the memory pipeline copies the fragments (global -> LDS loads), four LDS buffers per phase, two to three tiles in
//     flight and one barrier per tile.  Through registers and two buffers (one tile in flight) launches took 97.8 us instead of 89.8
//     (7B heads, 8 sequences of 20000 tokens, 17 rows each), 422 instead of 414 (1.5B heads, 256 of 8192);
//   * two query tiles (four phases fill the LDS with two buffers): HBM -> registers -> LDS; in iteration i a wave writes its share of
//     tile i + 1 to the other buffer, requests its share of tile i + 2, computes on tile i, then all eight waves meet at one
//     barrier; loads are in flight for more than a full iteration;
//   * query fragments stay in registers (one tile: 32 registers at head size 128).
// What bounds it: K/V from memory and the ends of the units, not the loop's instructions.  With the score products of the next tile interleaved with the
// softmax of this one (no wait of a product for the other) launches stayed where they were: 128 ragged sequences of 16 drafts 327 .. 335 us and 328 .. 334,
// 256 of 8192 tokens (1.5B heads) 384 .. 389 and 390 .. 391, 8 of 20000 88 .. 89 and 88 .. 89; so they did with a higher wave priority for one wave of a SIMD.
// Units with one query tile run as NQT = 2 with the second wave of each pair only loading.
#pragma once
#include "attn_softmax.h"

// Waits until at most N of this wave's requests are in flight, then for the other waves.
template <int N> __device__ __forceinline__ void wait_shares() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
#endif
}

template <int D>
__global__ void __launch_bounds__(512) attn_wide_kernel(const int32_t* __restrict__ seq_k, const int32_t* __restrict__ seq_c,
                                                        const int32_t* __restrict__ row_start, const int32_t* __restrict__ seq_slot,
                                                        const int32_t* __restrict__ attn_meta, const int32_t* __restrict__ item_start,
                                                        const int32_t* __restrict__ item_seq, const int32_t* __restrict__ item_chunk,
                                                        const int32_t* __restrict__ block_table, int max_pages, int n_pages,
                                                        int n_units, int Hq, int Hkv, float scale_log2e,
                                                        const f16* __restrict__ q, const f16* __restrict__ k_pages,
                                                        const f16* __restrict__ v_pages, f16* __restrict__ out,
                                                        float* __restrict__ part_o, float* __restrict__ part_ml,
                                                        int32_t* __restrict__ counters, int32_t* __restrict__ queue,
                                                        int out_ld, int32_t* __restrict__ status) {
  constexpr int KS = D / 16;            // MFMA K-steps of the QK^T product = K fragments of a tile
  constexpr int DT = D / 32;            // 32-wide d tiles of the output; V fragments of a tile = 2 DT
  constexpr int NF = KS + 2 * DT;       // 1 KiB fragments of one K/V tile
  constexpr int RPT = 128;              // padded query rows of a unit (stride of the partial results)
  constexpr int LDO = D + 4;            // row stride (floats) of an accumulator in LDS: 4 banks of skew per row
  constexpr int THREADS = 512;
  extern __shared__ __align__(16) char lds_raw[];
  __shared__ int s_w, s_last;

  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, wgs_per_xcd = gridDim.x >> 3;
  const int n_live = min(attn_meta[1] * Hkv, n_units);
  const int total_w = n_live > xcd ? (n_live - xcd + 7) / 8 : 0;   // units of this XCD (unit u belongs to XCD u % 8)
  // the wave index is made scalar so that everything derived from it stays on the scalar unit
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int ln = lane & 31, lg = lane >> 5;
  const size_t page_elems = kv_page_elems(Hkv, D);

  // threadIdx.x as a value the compiler cannot move.  What the two epilogues derive from it would otherwise be computed once,
  // before the loop over the units, and live through the tile loop: 256 registers and 43 spilled ones instead of 206.  Measured
  // per launch (7B heads unless stated): 128 sequences of 512 .. 32768 tokens 347 -> 341 us, one of 1000 tokens 26.8 -> 21.6,
  // 1.5B heads, 61 prompts around 512 tokens 35.4 -> 30.3.
  auto thread_now = [&]() { int t = threadIdx.x; asm volatile("" : "+v"(t)); return t; };
  // Combines the n_ch chunks of one (sequence, KV head): called by the last workgroup to publish its partial rows.
  // Four threads per query row; four chunks' loads are in flight together, the sums run in chunk order.
  auto merge_unit = [&](const int b, const int h, const int n_ch) {
    constexpr int TPR = THREADS / RPT, CH = D / 4, CPT = CH / TPR, GC = 4;
    const size_t slot0 = ((size_t)item_start[b] * Hkv + h) * RPT;
    const wt_buf bo = wt_buffer(part_o + slot0 * D), bm = wt_buffer(part_ml + slot0 * 2);
    const int G = Hq / Hkv, R = (seq_k[b] + 1) * G;
    const int tid = thread_now(), qr = tid / TPR, sub = tid % TPR;
    if (qr >= R) return;
    const uint32_t step = (uint32_t)Hkv * RPT;             // partial rows from one chunk to the next
    // the first group of chunks is requested with the maxima: one trip to memory, not two
    wt_f32x2 ml[GC];
    f32x4 v[GC][CPT];
    auto load_group = [&](int c0) {
#pragma unroll
      for (int u = 0; u < GC; ++u) {
        const uint32_t r = min(c0 + u, n_ch - 1) * step + qr;
        ml[u] = wt_load2(bm, r * 8);
#pragma unroll
        for (int j = 0; j < CPT; ++j) v[u][j] = wt_load4(bo, (r * D + (sub + j * TPR) * 4) * 4);
      }
    };
    load_group(0);
    float mt = -INFINITY;
    for (int c0 = 0; c0 < n_ch; c0 += 8) {
      float m[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) m[u] = wt_load2(bm, (min(c0 + u, n_ch - 1) * step + qr) * 8)[0];
#pragma unroll
      for (int u = 0; u < 8; ++u) mt = fmaxf(mt, m[u]);
    }
    float lt = 0.f;
    f32x4 acc[CPT];
#pragma unroll
    for (int j = 0; j < CPT; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < n_ch; c0 += GC) {
      if (c0 > 0) load_group(c0);
#pragma unroll
      for (int u = 0; u < GC; ++u) {
        if (c0 + u >= n_ch || ml[u][0] == -INFINITY) continue;
        const float f = __builtin_amdgcn_exp2f(ml[u][0] - mt);
        lt += ml[u][1] * f;
#pragma unroll
        for (int j = 0; j < CPT; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[j][e] += v[u][j][e] * f;
      }
    }
    const int iq = qr / G, hg = qr % G;
    const float inv = 1.0f / lt;
    const int orow = row_start[b] + iq, ocol = (h * G + hg) * D;
#pragma unroll
    for (int j = 0; j < CPT; j += 2)
      store_chunk_pair(out, orow, ocol, sub + j * TPR, TPR, out_ld,
                       to_f16x4_guarded(acc[j][0] * inv, acc[j][1] * inv, acc[j][2] * inv, acc[j][3] * inv, status),
                       to_f16x4_guarded(acc[j + 1][0] * inv, acc[j + 1][1] * inv, acc[j + 1][2] * inv, acc[j + 1][3] * inv, status));
  };

  // One unit with NQT query tiles (2 or 4).
  auto run = [&](auto nqt_tag, const int unit) {
    constexpr int NQT = decltype(nqt_tag)::value;
    constexpr int NPH = 8 / NQT;        // token phases
    constexpr int LPW = NF / NQT;       // fragments a wave moves per tile
    const int item = unit / Hkv, h = unit % Hkv;
    const int b = item_seq[item], chunk = item_chunk[item];
    const int n_ch = item_start[b + 1] - item_start[b];
    const int k = seq_k[b];
    const int G = Hq / Hkv;
    const int c = seq_c[b];
    const int n_tok = c + k + 1;
    const int R = (k + 1) * G;
    const int row0 = row_start[b];
    const int32_t* __restrict__ bt = block_table + (size_t)seq_slot[b] * max_pages;
    const int qt = wave % NQT, ph = wave / NQT;
    const bool has_rows = qt * 32 < R;                   // wave-uniform: a wave without query rows only moves data
    const int n_tiles = (n_tok + kTile - 1) / kTile;
    const int cht = attn_meta[0];
    const int t_begin = min(chunk * cht, n_tiles), t_end = min(t_begin + cht, n_tiles);
    const int n_it = (t_end - t_begin + NPH - 1) / NPH;  // iterations of the workgroup (at least 1: chunks are not empty)
    auto tile_of = [&](int i) { return t_begin + ph + NPH * i; };
    auto tile_offset = [&](int t) -> size_t {            // element offset of fragment 0 of tile t
      const int tb = min(t, n_tiles - 1) * kTile;        // clamped: a phase without a tile re-reads the last one
      const int page = min(max(bt[tb / kPage], 0), n_pages - 1);
      return (size_t)page * page_elems + (size_t)(h * 2 + ((tb / kTile) & 1)) * (kTile * D);
    };
    char* const my_stage = lds_raw + (size_t)ph * NF * 1024 + lane * 16;      // buffer 0 of this phase
    constexpr int BUF_BYTES = NPH * NF * 1024;
    constexpr bool DMA = NQT == 4;
    constexpr int NB = DMA ? 4 : 2;                      // LDS buffers
    // DMA: this wave's share of tile t straight into buffer buf
    auto request_share = [&](int t, int buf) {
      const size_t off = tile_offset(t);
#pragma unroll
      for (int j = 0; j < LPW; ++j) {
        const int f = qt + NQT * j;
        const f16* src = f < KS ? k_pages + off + f * 512 : v_pages + off + (f - KS) * 512;
        char* dst = lds_raw + (size_t)buf * BUF_BYTES + (ph * NF + f) * 1024;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(wt_buffer(src), (__attribute__((address_space(3))) void*)dst, 16, lane * 16, 0, 0, 0);
      }
    };
    u32x4 stg[LPW];
    auto load_share = [&](int t) {
      const size_t off = tile_offset(t) + lane * 8;
#pragma unroll
      for (int j = 0; j < LPW; ++j) {
        const int f = qt + NQT * j;
        stg[j] = (f < KS) ? *(const u32x4*)(k_pages + off + f * 512) : *(const u32x4*)(v_pages + off + (f - KS) * 512);
      }
    };
    auto store_share = [&](int buf) {
#pragma unroll
      for (int j = 0; j < LPW; ++j) *(u32x4*)(my_stage + buf * BUF_BYTES + (qt + NQT * j) * 1024) = stg[j];
    };

    // query fragments of this wave's tile (B operand: lane (n, g) holds Q[row n][g*D/2 + 8s + j]); rows beyond R are
    // clamped and masked through lim
    const int qr = qt * 32 + ln;
    const int lim = (qr < R) ? c + qr / G : -1;
    u32x4 qf[KS];
    {
      const int qc = min(qr, R - 1);
      const int iq = qc / G, hg = qc % G;
      const f16* src = q + (size_t)(row0 + iq) * Hq * D + (size_t)(h * G + hg) * D + lg * (D / 2);
#pragma unroll
      for (int s = 0; s < KS; ++s) qf[s] = *(const u32x4*)(src + s * 8);
    }
    if constexpr (DMA) {
      // The query loads in front and the requests unconditional (clamped), so that the wait for the queries leaves the requests in
      // flight; and here, because in the loop it would be a wait for everything in every iteration.
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NB - 1; ++i) request_share(tile_of(i), i);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(qf[s]));
    } else {
      load_share(tile_of(0));
      store_share(0);
      load_share(tile_of(1));
    }
    f32x16 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    if constexpr (!DMA) __syncthreads();

    for (int i = 0; i < n_it; ++i) {
      if constexpr (DMA) {
        // this wave's share of tile i has arrived (those of up to two more tiles may be in flight), then everybody's; nobody reads
        // tile i - 1 any more, whose buffer takes tile i + 3
        if (i + 2 < n_it) wait_shares<2 * LPW>();
        else if (i + 1 < n_it) wait_shares<LPW>();
        else wait_shares<0>();
        __builtin_amdgcn_sched_barrier(0);
        if (i + NB - 1 < n_it) request_share(tile_of(i + NB - 1), (i + NB - 1) & (NB - 1));
        __builtin_amdgcn_sched_barrier(0);
      } else {
        store_share((i + 1) & 1);                        // tile i + 1 (requested one iteration ago) -> the other buffer
        if (i + 2 < n_it) load_share(tile_of(i + 2));    // workgroup-uniform
      }
      const int t = tile_of(i);
      if (has_rows && t < t_end) {
        const char* stage = my_stage + (i & (NB - 1)) * BUF_BYTES;
        const int tok0 = t * kTile + 16 * lg;            // accumulator register r <-> token tok0 + r
        const bool full = (t + 1) * kTile - 1 <= c;      // every token visible to every row: no masking
        // the K fragments are requested from LDS together, before the first product (left to itself the compiler
        // reuses one register quad and waits for every read in turn: eight exposed LDS latencies per product);
        // the V fragments are requested into the same registers once the score products are issued and arrive
        // while the softmax runs
        u32x4 kf[KS], vf[2 * DT];
#pragma unroll
        for (int s = 0; s < KS; ++s) kf[s] = *(const u32x4*)(stage + s * 1024);
        __builtin_amdgcn_sched_barrier(0);
        f32x16 st;
#pragma unroll
        for (int r = 0; r < 16; ++r) st[r] = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s)
          st = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(kf[s]), as_f16x8(qf[s]), st, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x2 = 0; x2 < 2 * DT; ++x2) vf[x2] = *(const u32x4*)(stage + (KS + x2) * 1024);
        __builtin_amdgcn_sched_barrier(0);
        float x[16];
        if (full) {
#pragma unroll
          for (int r = 0; r < 16; ++r) x[r] = st[r];
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) x[r] = (tok0 + r <= lim) ? st[r] : -INFINITY;
        }
        float mloc = x[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mloc = fmaxf(mloc, x[r]);
        mloc = max_halves(mloc) * scale_log2e;           // scale > 0 commutes with max
        if (__any(mloc > m_run + kLateRescale)) {
          const float m_new = fmaxf(m_run, mloc);
          const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
          l_run *= alpha;
          m_run = m_new;
#pragma unroll
          for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
        }
        const float m_safe = (m_run == -INFINITY) ? 0.f : m_run;
        float psum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          x[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[r], scale_log2e, -m_safe));   // exp2(-inf) = 0
          psum += x[r];
        }
        l_run += psum;                                   // per lane half; halves are added at the end
        f16x8 pf[2];
#pragma unroll
        for (int j = 0; j < 8; ++j) { pf[0][j] = (f16)x[j]; pf[1][j] = (f16)x[8 + j]; }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int t2 = 0; t2 < 2; ++t2)
            o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(vf[dt * 2 + t2]), pf[t2], o[dt], 0, 0, 0);
      }
      if constexpr (!DMA) __syncthreads();               // buffer i & 1 is free, buffer (i + 1) & 1 is complete
    }
    if constexpr (DMA) __syncthreads();

    // ---- merge the NPH phases of each query tile through LDS (the K/V buffers are free after the loop's last
    // barrier): every wave stores its unscaled accumulator and its per-row (max, sum); after one barrier the 512
    // threads combine them, TPR threads per query row.
    float* s_o = (float*)lds_raw;                        // [8 waves][32][LDO]
    float* s_m = s_o + 8 * 32 * LDO;                     // [8][32]
    float* s_l = s_m + 8 * 32;
    {
      float* mine = s_o + (size_t)wave * 32 * LDO;
      l_run = sum_halves(l_run);
      if (lg == 0) { s_m[wave * 32 + ln] = m_run; s_l[wave * 32 + ln] = l_run; }
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
          *(f32x4*)(mine + ln * LDO + dt * 32 + 8 * i4 + 4 * lg) =
              f32x4{o[dt][4 * i4], o[dt][4 * i4 + 1], o[dt][4 * i4 + 2], o[dt][4 * i4 + 3]};
    }
    __syncthreads();
    const size_t slot0 = ((size_t)item_start[b] * Hkv + h) * RPT;       // partial row 0 of chunk 0
    const wt_buf bo = wt_buffer(part_o + slot0 * D), bm = wt_buffer(part_ml + slot0 * 2);
    {
      constexpr int TPR = THREADS / (32 * NQT);          // threads per query row: 8 or 4
      constexpr int CH = D / 4;                          // 16-byte chunks per row
      const int tid = thread_now(), wr = tid / TPR, sub = tid % TPR;      // wr = query row of the unit, 0 .. 32 NQT - 1
      const int tq = wr / 32, lr = wr % 32;
      if (wr < R) {
        float mw[NPH], mt = -INFINITY;
#pragma unroll
        for (int w = 0; w < NPH; ++w) {
          mw[w] = s_m[(w * NQT + tq) * 32 + lr];
          mt = fmaxf(mt, mw[w]);
        }
        const float ms = (mt == -INFINITY) ? 0.f : mt;
        float lt = 0.f;
#pragma unroll
        for (int w = 0; w < NPH; ++w) {
          mw[w] = __builtin_amdgcn_exp2f(mw[w] - ms);    // weight of phase w (0 for a phase that saw no token)
          lt += s_l[(w * NQT + tq) * 32 + lr] * mw[w];
        }
        const int iq = wr / G, hg = wr % G;
        const float inv = 1.0f / lt;                     // a single-chunk row always sees position c + i: lt > 0
        const int orow = row0 + iq, ocol = (h * G + hg) * D;
        const uint32_t pr = (uint32_t)(chunk * Hkv) * RPT + wr;   // row of this chunk, counted from chunk 0 of (sequence, head)
#pragma unroll
        for (int j = 0; j < CH / TPR; j += 2) {
          f32x4 acc[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int ch = sub + (j + u) * TPR;
            acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < NPH; ++w) {
              const f32x4 v = *(const f32x4*)(s_o + ((size_t)(w * NQT + tq) * 32 + lr) * LDO + ch * 4);
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[u][e] += v[e] * mw[w];
            }
            if (n_ch > 1) wt_store4(bo, (pr * D + ch * 4) * 4, acc[u]);
          }
          if (n_ch == 1)
            store_chunk_pair(out, orow, ocol, sub + j * TPR, TPR, out_ld,
                             to_f16x4_guarded(acc[0][0] * inv, acc[0][1] * inv, acc[0][2] * inv, acc[0][3] * inv, status),
                             to_f16x4_guarded(acc[1][0] * inv, acc[1][1] * inv, acc[1][2] * inv, acc[1][3] * inv, status));
        }
        if (n_ch > 1 && sub == 0) wt_store2(bm, pr * 8, mt, lt);
      }
    }
  };   // run

  auto process = [&](const int unit) {
    const int b = item_seq[unit / Hkv];
    const int k = seq_k[b];
    if (k < 0) return;                                   // workgroup-uniform
    if ((k + 1) * (Hq / Hkv) > 64) run(std::integral_constant<int, 4>{}, unit);
    else run(std::integral_constant<int, 2>{}, unit);
    // several chunks: the last workgroup of (sequence, KV head) to arrive merges all of them
    const int h = unit % Hkv, n_ch = item_start[b + 1] - item_start[b];
    if (n_ch > 1 && publish_arrival(counters + ((size_t)b * Hkv + h) * 4, n_ch, &s_last)) merge_unit(b, h, n_ch);
  };

  int w = slot;                                         // position in this XCD's queue
  while (w < total_w) {
    __syncthreads();                                    // LDS of the previous unit is no longer read
    process(xcd + 8 * w);
    if (total_w <= wgs_per_xcd) break;                  // at most one unit per workgroup: nothing to take
    __syncthreads();
    if (threadIdx.x == 0) s_w = atomicAdd(queue + xcd, 1) + wgs_per_xcd;
    __syncthreads();
    w = __builtin_amdgcn_readfirstlane(s_w);
  }
}
