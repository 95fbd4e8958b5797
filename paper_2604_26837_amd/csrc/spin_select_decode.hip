// Stages 2, 3 and 4 in one launch (all-resident mode, partitions of whole pages, rows that fit a workgroup's
// registers or go by their tiles' maxima).
//
// A launch that depends on the one before it starts 2 to 3 us after that one's last wavefront has its result, and the
// page list goes out to memory and back in between.  Here every workgroup of a row, one per split of stage 4, selects
// and resolves the row for itself: the same device functions on the same scores, so that all of them hold the same
// list, in LDS, and no workgroup waits for another.  Split 0 stores it.  What is done more than once is a row's few KiB of
// scores and its leaf entries, on compute units that would have waited.  Whole steps, us, against the launch of stages
// 2+3 followed by that of stage 4: 128 rows of 2048 pages, 128 attended 52.6 -> 50.2; 24 rows of 512, 64 attended 23.0 ->
// 20.8; 8 rows of 8192 28.0 -> 24.7; 256 ragged rows of up to 16384 139.5 -> 137.6; 32 rows of 1024 blocks 31.5 -> 30.1;
// 512 rows of 500 and 1000 83.9 -> 72.4 and 143.5 -> 132.9 (also where the rows are more than the compute units, then);
// 8 rows of 62500, 256 attended 61.8 -> 58.3; 32 rows of 250 clusters, 32 of them attended 24.6 -> 23.1, and 22.7 with the
// windows' tables read four entries at a time, without branches.
//
// The row's always-attended pages are known before its scores are: each wavefront asks for the first of its own ahead of
// the selection and attends it when the first selected ones are under way.
#include <cstdio>

#include "spin_score_dev.h"
#include "spin_step_dev.h"

// the selection goes to LDS; memory has it from the row's first workgroup
struct step_sel {
  int32_t *__restrict__ out;
  int stride;
  spin_lds_i32 *lds;
  bool store;
  __device__ __forceinline__ void put(int pos, int32_t id) const {
    if (pos < stride) lds[pos] = id;
  }
  __device__ __forceinline__ void pad(int pos) const {
    if (store) out[pos] = -1;
  }
  __device__ __forceinline__ void count(int32_t *__restrict__ nsel, int row, int take) const {
    if (store) nsel[row] = take;
  }
};

// and so does the page list
struct step_pages {
  res_out out;
  spin_lds_i32 *slot;
  spin_lds_u16 *mask;
  bool store;
  __device__ __forceinline__ void put(int pos, int32_t s, int32_t page, uint32_t m) const {
    slot[pos] = s;
    mask[pos] = (uint16_t)m;
    if (store) out.put(pos, s, page, m);
  }
  __device__ __forceinline__ void count(int total) const {
    if (store) out.count(total);
  }
};

// The first of this wavefront's always-attended pages, number `first` of the row's: its leaf entry's index and whether there
// is one.  lane_dir: the row's directory, one entry per lane.
struct asked_page {
  int page;
  size_t leaf;
  bool there;
};
__device__ __forceinline__ asked_page page_ahead(bool mine, int first, const forced_span &fs, int32_t lane_dir, int dir_stride,
                                                 int64_t leaf_chunks, int leaf_entries, int leaf_log) {
  asked_page p;
  p.page = first < fs.nlo ? first : fs.recent_begin + (first - fs.nlo);
  const int ci = !mine ? 0 : (leaf_log >= 0 ? p.page >> leaf_log : p.page / leaf_entries);
  const int32_t chunk = __builtin_amdgcn_readlane(lane_dir, ci < dir_stride ? ci : 0);
  p.there = mine && ci < dir_stride && chunk >= 0 && (int64_t)chunk < leaf_chunks;
  p.leaf = p.there ? (size_t)chunk * leaf_entries + (p.page - ci * leaf_entries) : 0;
  return p;
}

// The selection of a row of partitions of one page, KPT of them per thread (`scores` gives a quad of theirs): the chosen
// pages in order to l_page, and with `with_leaf` their leaf entries, which came with the scores, to l_slot (a thread's pages
// are quads of one leaf).
template <int BLOCK, int KPT, typename SCORES, typename ASK>
__device__ __forceinline__ void select_pages(SCORES scores, const sel_plan &pl, bool with_leaf,
                                             int32_t lane_dir, int dir_stride, const spin_step_args &a, spin_lds_i32 *l_page,
                                             spin_lds_i32 *l_slot, reg_row_lds<BLOCK> &s, ASK ask_ahead) {
  typedef typename key_bits<KPT>::type M;
  constexpr int Q = KPT <= 8 ? KPT / 4 : 1;
  const int c0 = threadIdx.x * KPT;
  float f[KPT];
#pragma unroll
  for (int k4 = 0; k4 < KPT; k4 += 4) {
    const float4 v = scores(c0 + k4);
    f[k4] = v.x; f[k4 + 1] = v.y; f[k4 + 2] = v.z; f[k4 + 3] = v.w;
  }
  spin_i32x4_at4 leaf[Q];
  [[maybe_unused]] bool there[Q];
  if constexpr (KPT <= 8) {
    if (with_leaf) {
#pragma unroll
      for (int j = 0; j < Q; ++j) {
        const int p = c0 + 4 * j, ci = p >> a.leaf_log;
        const int32_t chunk = __shfl(lane_dir, min(ci, dir_stride - 1));
        there[j] = ci < dir_stride && chunk >= 0 && (int64_t)chunk < a.leaf_chunks;
        const size_t at = there[j] ? ((size_t)chunk << a.leaf_log) + (p & (a.leaf_entries - 1)) : 0;
        leaf[j] = *(const spin_i32x4_at4 *)(a.leaf_pool + at);
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  const M cand = range_bits<KPT>(c0, pl.nf_lo, pl.first_hi);
  const M forced = range_bits<KPT>(c0, 0, pl.P) & ~cand;
  ask_ahead();
  select_elements<BLOCK, KPT>(f, cand, forced, c0, pl.nf_lo, pl.first_hi, pl.kprime, s, [&](int pos, int k) {
    if (pos >= a.page_stride) return;
    l_page[pos] = c0 + k;
    if constexpr (KPT <= 8)
      if (with_leaf) l_slot[pos] = there[k / 4] ? leaf[k / 4][k & 3] : -1;
  });
}

// Stage 1 of a row by the calling workgroup of 8 wavefronts: the scores go to LDS (`cap` of them), and to `out` where that is
// there.  The arithmetic is consume_tile's, and so are the bits.
// Small contexts: a launch whose few workgroups have a tile or two per wavefront is over in the time that it takes to
// start, and so would be the wait for its end; and every workgroup of the row has its summaries in one trip.
template <bool MINMAX>
__device__ __forceinline__ void score_row(const spin_bf16x8 (&qf)[4], const uint4 *__restrict__ summ, size_t base, int PP,
                                          int reps, int G, int wave, int lane, float *lds, int cap, float *__restrict__ out) {
  constexpr int NJ = MINMAX ? 8 : 4, WAVES = 8;
  const int n = lane & 15, c = lane >> 4;
  spin_bf16x8 qs[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    uint4 v = __builtin_bit_cast(uint4, qf[j & 3]);
    if (MINMAX) v = make_uint4(relu_pack(v.x, j < 4), relu_pack(v.y, j < 4), relu_pack(v.z, j < 4), relu_pack(v.w, j < 4));
    qs[j] = __builtin_bit_cast(spin_bf16x8, v);
  }
  const int ntiles = PP * reps / 16, per_tile = 16 / reps;
  const uint4 *tiles = summ + base * reps * (NJ * 4);
  // (tile by tile, since a row beyond its context may have any number of them)
  auto load = [&](score_tile<NJ> &r, int t) {
    const __amdgpu_buffer_rsrc_t buf = spin_buffer(tiles + (size_t)(t < ntiles ? t : 0) * (NJ * 64), t < ntiles ? NJ * 1024 : 0);
#pragma unroll
    for (int j = 0; j < NJ; ++j) r.a[j] = spin_buffer_load_kept(buf, (uint32_t)(j * 64 + lane) * 16);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto consume = [&](const score_tile<NJ> &r, int t) {
    spin_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qs[j], __builtin_bit_cast(spin_bf16x8, r.a[j]), acc, 0, 0, 0);
    float m = spin_head_max(acc, c, G);
    if (!MINMAX) {
      if (reps >= 2) m = fmaxf(m, spin_dpp<SPIN_DPP_XOR1>(m));
      if (reps == 4) m = fmaxf(m, spin_dpp<SPIN_DPP_XOR2>(m));
    }
    if (c == 0 && (n & (reps - 1)) == 0) {
      const int at = t * per_tile + n / reps;
      if (at < cap) lds[at] = m;
      if (out) out[base + at] = m;
    }
  };
  score_tile<NJ> ra, rb;
  load(ra, wave);
  load(rb, wave + WAVES);
  for (int t = wave; t < ntiles; t += 2 * WAVES) {
    consume(ra, t);
    load(ra, t + 2 * WAVES);
    if (t + WAVES < ntiles) consume(rb, t + WAVES);
    load(rb, t + 3 * WAVES);
  }
}

// grid: splits x KV heads x requests.  PAGES: partitions of one page, 2^leaf_log >= 4 entries to a leaf; the selection is
// the page list, nothing is divided, a row takes as many scores per thread as its own length asks for, and with up to 8 a
// page's leaf entry comes with its score.
// TILES: rows beyond a workgroup's registers, selected from their tiles' maxima, KPT of them per thread; otherwise KPT is the
// scores per thread of the longest row.
// VAR: variable-length partitions.  Which pages their windows cover is known from the tables only: none is asked for ahead.
// SCORE: stage 1 as well (score_row), of the kind SCORE - 1.
template <int KPT, bool PAGES, bool TILES, bool VAR, int SCORE>
__global__ __launch_bounds__(512) void spin_select_decode_kernel(
    const float *__restrict__ scores, const int32_t *__restrict__ part_offsets, const int32_t *__restrict__ seq_lens,
    const int32_t *__restrict__ dir, const uint16_t *__restrict__ q, int Hkv, int nsplit, int G, int Hq, int dir_stride,
    spin_step_args a) {
  constexpr int WAVES = 8, BLOCK = 64 * WAVES;
  __shared__ typename std::conditional<TILES, int, reg_row_lds<BLOCK>>::type s;
  __shared__ int32_t held_words[PAGES ? RES_DIR_LDS : sizeof(held_row<true>) / sizeof(int32_t)];
  // VAR, rows of up to 4096: their tables, so that the selected entries are no trip to memory (32 rows of 250: 22.8 -> 22.0 us)
  constexpr int TABLES = VAR && KPT <= 8 ? BLOCK * KPT : 0;
  __shared__ __align__(16) int32_t s_tables[TABLES ? 2 * TABLES : 1];
  __shared__ __align__(16) float s_scores[SCORE ? BLOCK * KPT : 1];
  extern __shared__ __align__(16) float smem[];       // the merge buffers of decode_finish, then the row's page list
  spin_lds_i32 *l_slot = (spin_lds_i32 *)(smem + a.lists_at);
  spin_lds_i32 *l_page = l_slot + a.page_stride;      // PAGES: the pages
  spin_lds_u16 *l_mask = (spin_lds_u16 *)l_page;      // otherwise: the masks
  const int split = blockIdx.x, h = blockIdx.y, b = blockIdx.z, row = b * Hkv + h;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, c = lane >> 4;
  const bool store = split == 0;

  // Pages are dealt round-robin, the always-attended ones (first the sink, then the recent ones) ahead of the others:
  // page v goes to split v % nsplit, wavefront (v / nsplit) % WAVES.
  const int first = wave * nsplit + split, stride = WAVES * nsplit;
  const int32_t *rdir = dir + (size_t)row * dir_stride;
  // the directory one entry per lane (larger ones: no page is asked for ahead)
  const bool ahead = dir_stride <= 64;
  const int32_t lane_dir = rdir[min(lane, dir_stride - 1)];
  const int N = max(seq_lens[b], 0);
  const forced_span fs = VAR ? forced_span{0, 0, 0} : forced_pages_of(N, a.sink_pages, a.recent_pages);
  // (not where the trips to the page's entries would keep the maxima waiting, 8 rows of 62500 57.8 -> 58.3 us, or the scores)
  const bool asked = !TILES && !SCORE && ahead && first < fs.nlo + fs.nhi;
  spin_bf16x8 qf[4];
  page_regs rf;
  unsigned rf_mask = 0;
  int rf_slot = 0;
  auto ask_ahead = [&](const asked_page &p) {
    const int32_t slot = __builtin_amdgcn_readfirstlane(a.leaf_pool[p.leaf]);
    const bool ok = p.there && slot >= 0 && (int64_t)slot < a.pool_slots;
    rf_mask = ok ? page_mask(p.page, N) : 0u;
    rf_slot = ok ? slot : 0;
    load_k_tile(rf, a.pool, rf_slot, lane, rf_mask);
    load_v_tile(rf, a.pool, rf_slot, lane, rf_mask);
    __builtin_amdgcn_sched_barrier(0);
  };

  int np;                                             // pages of the row's list
  [[maybe_unused]] bool with_leaf = false;
  if constexpr (PAGES) {
    const int off = part_offsets[b], PP = part_offsets[b + 1] - off;
    const int32_t mydir = rdir[min(tid, dir_stride - 1)];
    load_queries(qf, q, b, h, G, Hq, n, c);
    __builtin_amdgcn_sched_barrier(0);
    auto ask = [&] {
      if constexpr (!SCORE)
        ask_ahead(page_ahead(asked, first, fs, lane_dir, dir_stride, a.leaf_chunks, a.leaf_entries, a.leaf_log));
      if (!with_leaf && tid < RES_DIR_LDS) held_words[tid] = mydir;
    };
    if constexpr (TILES) {
      const lds_sel rsel = {min(a.sel_stride, a.page_stride), l_page};
      np = select_tiles_row<BLOCK, KPT, STEP_CAP, true>(scores, a.maxima, a.max_stride, a.gs_log, part_offsets, seq_lens, Hkv,
                                                        SPIN_PAGE_TOKENS, a.topk, a.includes_forced, a.sink_pages,
                                                        a.recent_pages, a.sel, rsel, a.nsel, row, *(step_tiles_lds *)smem);
      if (tid < RES_DIR_LDS) held_words[tid] = mydir;
    } else {
      // the selection's plan: partitions are pages
      const int pages = min((N + 15) >> 4, PP), P = min(pages, BLOCK * KPT);
      // (of a row beyond the context's longest the first BLOCK * KPT pages are kept, but all its forced ones count, as in
      // stage 2)
      const int beyond = a.includes_forced ? pages - max(min(fs.recent_begin, pages), P) : 0;
      const sel_plan pl = plan_of(P, min(fs.nlo, P), min(fs.recent_begin, P), a.topk - beyond, a.includes_forced, a.sel_stride);
      with_leaf = ahead && P <= 8 * BLOCK;
      if constexpr (SCORE != 0) {
        score_row<SCORE == SPIN_SCORE_MINMAX + 1>(qf, a.summ, (size_t)Hkv * off + (size_t)h * PP, PP, a.reps, G, wave, lane,
                                                  s_scores, BLOCK * KPT, store ? a.scores_out : nullptr);
        __syncthreads();
        select_pages<BLOCK, KPT>([&](int at) { return *(const float4 *)(s_scores + at); }, pl, with_leaf, lane_dir, dir_stride, a,
                                 l_page, l_slot, s, ask);
      } else {
        // zeros past the row's end
        const __amdgpu_buffer_rsrc_t buf =
            spin_buffer(scores + (size_t)Hkv * off + (size_t)h * PP, (uint32_t)max(PP, 0) * sizeof(float));
        auto quad = [&](int at) { return __builtin_bit_cast(float4, spin_buffer_load_kept(buf, (uint32_t)at * sizeof(float))); };
        if (KPT == 4 || P <= 4 * BLOCK)
          select_pages<BLOCK, 4>(quad, pl, with_leaf, lane_dir, dir_stride, a, l_page, l_slot, s, ask);
        else if (KPT == 8 || P <= 8 * BLOCK)
          select_pages<BLOCK, 8>(quad, pl, with_leaf, lane_dir, dir_stride, a, l_page, l_slot, s, ask);
        else if (KPT == 16 || P <= 16 * BLOCK)
          select_pages<BLOCK, 16>(quad, pl, false, lane_dir, dir_stride, a, l_page, l_slot, s, ask);
        else
          select_pages<BLOCK, 32>(quad, pl, false, lane_dir, dir_stride, a, l_page, l_slot, s, ask);
      }
      np = min(pl.take, a.page_stride);
    }
  } else {
    load_queries(qf, q, b, h, G, Hq, n, c);
    held_row<true> &s_held = *(held_row<true> *)held_words;
    int32_t mydir;
    const step_sel rsel = {a.sel + (size_t)row * a.sel_stride, a.sel_stride, (spin_lds_i32 *)s_held.sel, store};
    auto ask = [&] {
      mydir = row_dir_entry(dir, dir_stride, row);
      if constexpr (!VAR && !TILES)
        ask_ahead(page_ahead(asked, first, fs, lane_dir, dir_stride, a.leaf_chunks, a.leaf_entries, a.leaf_log));
    };
    int take;
    spin_var_span span;
    if constexpr (TILES) {
      ask();
      take = select_tiles_row<BLOCK, KPT, STEP_CAP, true>(scores, a.maxima, a.max_stride, a.gs_log, part_offsets, seq_lens, Hkv,
                                                          a.tp, a.topk, a.includes_forced, a.sink_pages, a.recent_pages,
                                                          a.sel, rsel, a.nsel, row, *(step_tiles_lds *)smem);
    } else {
      take = select_reg_row<BLOCK, KPT, (TABLES > 0)>(scores, part_offsets, seq_lens, Hkv, a.tp, a.topk, a.includes_forced,
                                                      a.sink_pages, a.recent_pages, rsel, a.nsel, row,
                                                      VAR ? a.var : spin_var{}, span, s, ask, s_tables);
    }
    if (tid < RES_DIR_LDS) s_held.dir[tid] = mydir;
    __syncthreads();                   // the selection and the directory are whole
    if (store)
      for (int i = tid; i < take; i += BLOCK) rsel.out[i] = rsel.lds[i];
    const step_pages list = {res_row_out(a.slots, a.page_ids, a.valid_mask, a.npages, row, a.page_stride), l_slot, l_mask, store};
    np = resolve_row<BLOCK, true, true, true, TABLES>(row, take, a.sel, seq_lens, dir, a.leaf_pool, a.leaf_chunks, Hkv, a.tp,
                                                      a.sink_pages, a.recent_pages, a.sel_stride, a.page_stride, dir_stride,
                                                      a.leaf_entries, list, a.status, VAR ? a.var : spin_var{},
                                                      VAR ? &span : nullptr, &s_held, s_tables);
  }
  __syncthreads();

  // The sink pages open the list and the recent ones close it (but for a row longer than its partition table, whose list
  // may be without the recent ones).
  softmax_state st;
  softmax_reset(st);
  const bool whole = fs.nlo + fs.nhi <= np;
  const int nlo = whole ? fs.nlo : 0, nf = whole ? fs.nlo + fs.nhi : 0;
  const int cnt_all = np > first ? (np - first + stride - 1) / stride : 0;
  const res_out out = res_row_out(a.slots, a.page_ids, a.valid_mask, a.npages, row, a.page_stride);
  for (int base = 0; base == 0 || base < cnt_all; base += 64) {
    const int cnt = max(min(cnt_all - base, 64), 0);
    int myslot = 0;
    unsigned mymask = 0;
    [[maybe_unused]] int at = 0, page = -1, found = -1;
    [[maybe_unused]] unsigned found_mask = 0;
    if (lane < cnt) {
      const int v = first + (base + lane) * stride;
      at = v < nf ? (v < nlo ? v : np - nf + v) : nlo + (v - nf);
      if constexpr (PAGES) {
        page = l_page[at];
        if (with_leaf) {
          found = l_slot[at];
        } else {
          const int ci = page >> a.leaf_log;
          if (ci < dir_stride) {
            const int32_t chunk = dir_stride <= RES_DIR_LDS ? ((spin_lds_i32 *)held_words)[ci] : rdir[ci];
            if (chunk >= 0 && (int64_t)chunk < a.leaf_chunks)
              found = a.leaf_pool[((size_t)chunk << a.leaf_log) + (page & (a.leaf_entries - 1))];
          }
        }
        if (found < 0) {
          found = -1;
          spin_raise(a.status, SPIN_ERR_NOT_RESIDENT);
        }
        found_mask = found >= 0 ? page_mask(page, N) : 0u;
      } else {
        found = l_slot[at];
        found_mask = l_mask[at];
      }
      if (found >= 0 && (int64_t)found < a.pool_slots) {
        myslot = found;
        mymask = found_mask;
      } else if (found >= 0) {                            // (one that is missing has been reported)
        spin_raise(a.status, SPIN_ERR_SLOT_RANGE);        // attends to none of it
      }
    }
    // the first one was asked for already, if it is the listed one
    const int from = base == 0 && asked && __builtin_amdgcn_readlane(myslot, 0) == rf_slot &&
                     __builtin_amdgcn_readlane((int)mymask, 0) == (int)rf_mask ? 1 : 0;
    attend_lane_pages<2>(st, a.pool, myslot, mymask, from, cnt, lane, c, qf, a.scale_log2e, [&] {
      if (from && cnt > 0) tile_attend(st, tile_logits(rf, qf), rf, rf_mask, c, a.scale_log2e);
      if constexpr (PAGES) {                              // the row's lists: its own entries from every wavefront
        if (lane < cnt) out.put(at, found, page, found_mask);
        if (store && base == 0) {
          int32_t *rsel = a.sel + (size_t)row * a.sel_stride;
          for (int i = tid; i < a.sel_stride; i += BLOCK) rsel[i] = i < np ? l_page[i] : -1;
          for (int i = np + tid; i < a.page_stride; i += BLOCK) out.put(i, -1, -1, 0);
          if (tid == 0) {
            a.nsel[row] = np;
            out.count(np);
          }
        }
      }
    });
  }
  decode_finish<WAVES>(st, row, split, b, h, lane, wave, n, c, G, Hq, nsplit, nsplit, a.part_ml, a.part_acc, a.tickets, a.out,
                       a.lse);
}

// partitions of one page, leaves of four entries and more, in powers of two: the kernel's PAGES
static bool step_one_page(const spin_ctx *ctx) {
  const int32_t leaf = ctx->cfg.leaf_entries;
  return ctx->cfg.partition_tokens == SPIN_PAGE_TOKENS && leaf >= 4 && (leaf & (leaf - 1)) == 0;
}

// Contexts whose stage 1 the launch of stages 2 to 4 does as well (score_row): a row's summaries fill two tiles of 8 KiB per
// wavefront at most, or one where the rows are enough for a launch of stage 1 to stream.  Steps, us, two launches / one:
// MINMAX, 64 pages to a row: 2 rows 10.8 / 9.5, 32 rows 14.0 / 12.1, 256 rows 26.4 / 25.4; 128 pages 12.9 / 11.6, 14.6 / 13.3,
// 27.7 / 27.2; 256 pages 12.0 / 11.7, 14.2 / 13.4, 29.9 / 30.3; 512 pages 13.2 / 12.9, 14.5 / 15.6, 34.4 / 35.6; one
// representative per page, 24 rows of 256 / 512 / 1024 pages 14.6 / 12.2, 14.5 / 12.6, 14.4 / 14.2.
static bool score_in_step(const spin_ctx *ctx) {
  const spin_config &c = ctx->cfg;
  const int64_t row_bytes = (int64_t)((ctx->max_parts + 15) / 16 * 16) * ctx->rows_per_part * ctx->kd * 2;
  return step_one_page(ctx) && c.score_kind != SPIN_SCORE_SKETCH && !ctx->var.count && ctx->max_parts <= 2048 &&
         row_bytes <= (ctx->max_rows <= 128 ? 128 : 64) * 1024;
}

// maxima_ready: stage 1 of this step has left its tiles' maxima in the workspace.  summaries: stage 1 has not run, its scores
// go to scores_out (contexts that score_in_step says are small)
static int select_resolve_decode_impl(spin_ctx *ctx, int32_t batch, const float *scores, const int32_t *part_offsets,
                                      const int32_t *seq_lens, int32_t *sel, int32_t *nsel, const int32_t *dir,
                                      const int32_t *leaf_pool, int64_t leaf_chunks, int32_t *slots, int32_t *page_ids,
                                      uint16_t *valid_mask, int32_t *npages, const void *q, const void *kv_pool,
                                      int64_t pool_slots, void *out, float *lse, void *workspace, void *stream,
                                      bool maxima_ready, const void *summaries, float *scores_out) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch || leaf_chunks <= 0 || pool_slots <= 0) return SPIN_ERR_INVALID;
  if (ctx->fused_splits == 0) return SPIN_ERR_UNSUPPORTED;
  if (batch == 0) return SPIN_OK;
  if (!scores || !part_offsets || !seq_lens || !sel || !nsel || !dir || !leaf_pool || !slots || !page_ids ||
      !valid_mask || !npages || !q || !kv_pool || !out)
    return SPIN_ERR_INVALID;
  if (!workspace) return SPIN_ERR_WORKSPACE;
  const spin_config &c = ctx->cfg;
  char *ws = (char *)workspace;
  const int leaf_log = (c.leaf_entries & (c.leaf_entries - 1)) ? -1 : 31 - __builtin_clz((unsigned)c.leaf_entries);
  const bool tiles = ctx->step_tiles != 0;
  float *maxima = tiles ? (float *)(ws + ctx->ws_max_off) : nullptr;
  if (tiles && !maxima_ready) spin_take_maxima(ctx, batch * c.num_kv_heads, scores, part_offsets, maxima, stream);
  const spin_step_args a = {leaf_pool, leaf_chunks, sel, nsel, slots, page_ids, valid_mask, npages, (const uint4 *)kv_pool,
                            pool_slots, (uint16_t *)out, lse, (float *)(ws + ctx->ws_ml_off),
                            (float *)(ws + ctx->ws_acc_off), (int32_t *)(ws + ctx->ws_ticket_off), (int32_t *)workspace,
                            c.partition_tokens, c.topk, c.topk_includes_forced, c.sink_pages, c.recent_pages,
                            ctx->sel_stride, ctx->page_stride, c.leaf_entries, leaf_log,
                            (int)(spin_fused_front(ctx) / sizeof(float)), maxima, ctx->max_stride, ctx->tile_log, ctx->var,
                            (const uint4 *)summaries, scores_out, ctx->rows_per_part,
                            ctx->scale * 1.4426950408889634f};
  if (ctx->k_token_major) return spin_step_tokens_launch(ctx, batch, scores, part_offsets, seq_lens, dir, q, a, stream);
  const int per_thread = spin_step_per_thread(ctx);
  const bool one_page = step_one_page(ctx);
#define SPIN_SD_LAUNCH1(KPT, PAGES, TILES, VAR, SCORE)                                                                   \
  spin_launch(ctx, SPIN_K_SELECT_DECODE, spin_select_decode_kernel<KPT, PAGES, TILES, VAR, SCORE>,                           \
              dim3((unsigned)ctx->fused_splits, (unsigned)c.num_kv_heads, (unsigned)batch), dim3(512), spin_fused_lds(ctx), \
              (hipStream_t)stream, scores, part_offsets, seq_lens, dir, (const uint16_t *)q, c.num_kv_heads,      \
              ctx->fused_splits, ctx->group, c.num_q_heads, ctx->dir_stride, a)
#define SPIN_SD_LAUNCH(KPT, TILES)                                                                \
  do {                                                                                            \
    if (!TILES && ctx->var.count) SPIN_SD_LAUNCH1(KPT, false, false, true, 0);                       \
    else if (one_page) SPIN_SD_LAUNCH1(KPT, true, TILES, false, 0);                                  \
    else SPIN_SD_LAUNCH1(KPT, false, TILES, false, 0);                                               \
  } while (0)
  if (summaries) {
    if (c.score_kind == SPIN_SCORE_MINMAX) SPIN_SD_LAUNCH1(4, true, false, false, SPIN_SCORE_MINMAX + 1);
    else SPIN_SD_LAUNCH1(4, true, false, false, SPIN_SCORE_REPMAX + 1);
  } else if (tiles) {
    if (per_thread == 4) SPIN_SD_LAUNCH(4, true);
    else if (per_thread == 8) SPIN_SD_LAUNCH(8, true);
    else SPIN_SD_LAUNCH(16, true);
  } else if (per_thread == 4) SPIN_SD_LAUNCH(4, false);
  else if (per_thread == 8) SPIN_SD_LAUNCH(8, false);
  else if (per_thread == 16) SPIN_SD_LAUNCH(16, false);
  else SPIN_SD_LAUNCH(32, false);
#undef SPIN_SD_LAUNCH1
#undef SPIN_SD_LAUNCH
  return spin_launch_status();
}

extern "C" int spin_select_resolve_decode(spin_ctx *ctx, int32_t batch, const float *scores, const int32_t *part_offsets,
                                          const int32_t *seq_lens, int32_t *sel, int32_t *nsel, const int32_t *dir,
                                          const int32_t *leaf_pool, int64_t leaf_chunks, int32_t *slots, int32_t *page_ids,
                                          uint16_t *valid_mask, int32_t *npages, const void *q, const void *kv_pool,
                                          int64_t pool_slots, void *out, float *lse, void *workspace, void *stream) {
  return select_resolve_decode_impl(ctx, batch, scores, part_offsets, seq_lens, sel, nsel, dir, leaf_pool, leaf_chunks,
                                    slots, page_ids, valid_mask, npages, q, kv_pool, pool_slots, out, lse, workspace,
                                    stream, false, nullptr, nullptr);
}

// Stages 1 to 4 in one call, two launches (small contexts: one): stage 1 (with its tiles' maxima in contexts whose rows are
// selected by them, see step_tiles), then the above.
extern "C" int spin_decode_step(spin_ctx *ctx, int32_t batch, const void *q, const void *summaries, const int32_t *chan_idx,
                                const int32_t *part_offsets, const int32_t *seq_lens, float *scores, int32_t *sel,
                                int32_t *nsel, const int32_t *dir, const int32_t *leaf_pool, int64_t leaf_chunks,
                                int32_t *slots, int32_t *page_ids, uint16_t *valid_mask, int32_t *npages,
                                const void *kv_pool, int64_t pool_slots, void *out, float *lse, void *workspace,
                                void *stream) {
  // refuse before stage 1 is issued what the second launch would refuse
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch || leaf_chunks <= 0 || pool_slots <= 0) return SPIN_ERR_INVALID;
  if (ctx->fused_splits == 0) return SPIN_ERR_UNSUPPORTED;
  if (batch == 0) return SPIN_OK;
  if (!sel || !nsel || !dir || !leaf_pool || !slots || !page_ids || !valid_mask || !npages || !kv_pool || !out)
    return SPIN_ERR_INVALID;
  if (!workspace) return SPIN_ERR_WORKSPACE;
  if (score_in_step(ctx)) {
    if (!q || !summaries || !part_offsets || !seq_lens || !scores) return SPIN_ERR_INVALID;
    return select_resolve_decode_impl(ctx, batch, scores, part_offsets, seq_lens, sel, nsel, dir, leaf_pool, leaf_chunks,
                                      slots, page_ids, valid_mask, npages, q, kv_pool, pool_slots, out, lse, workspace,
                                      stream, false, summaries, scores);
  }
  const bool tiles = ctx->step_tiles != 0;
  const int st = spin_score_impl(ctx, batch, q, summaries, chan_idx, part_offsets, seq_lens, scores, workspace, stream,
                                 tiles ? (float *)((char *)workspace + ctx->ws_max_off) : nullptr);
  if (st != SPIN_OK) return st;
  return select_resolve_decode_impl(ctx, batch, scores, part_offsets, seq_lens, sel, nsel, dir, leaf_pool, leaf_chunks,
                                    slots, page_ids, valid_mask, npages, q, kv_pool, pool_slots, out, lse, workspace,
                                    stream, true, nullptr, nullptr);
}

extern "C" int32_t spin_fused_splits(const spin_ctx *c) { return c ? c->fused_splits : 0; }

extern "C" int32_t spin_step_kernel(const spin_ctx *ctx, char *name, int32_t size) {
  if (!ctx || !name || size < 1) return SPIN_ERR_INVALID;
  if (ctx->fused_splits == 0) return 0;
  const spin_config &c = ctx->cfg;
  const bool one = score_in_step(ctx), var = ctx->var.count != nullptr;
  const char *tiles = ctx->step_tiles ? "true" : "false";
  if (ctx->k_token_major)
    snprintf(name, size, "spin_select_decode_tokens_kernel<%d, %s>", spin_step_per_thread(ctx), tiles);
  else
    snprintf(name, size, "spin_select_decode_kernel<%d, %s, %s, %s, %d>", one ? 4 : spin_step_per_thread(ctx),
             step_one_page(ctx) && !var ? "true" : "false", tiles, var ? "true" : "false",
             one ? (c.score_kind == SPIN_SCORE_MINMAX ? SPIN_SCORE_MINMAX : SPIN_SCORE_REPMAX) + 1 : 0);
  return one ? 1 : 2;
}
