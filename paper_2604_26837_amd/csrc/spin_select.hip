// Stage 2: per row, forced partitions plus the k' best-scoring candidates
// (Table 1, "-> topk"; Section 4.2: the always-attended windows are filtered
// out of the candidates).
//
// One workgroup per row.  Scores become order-preserving 32-bit keys (NaN ->
// -inf, -0 -> +0); an MSB-first radix select (four 8-bit passes, LDS
// histogram, parallel suffix scan) finds the key T of the k'-th best
// candidate; then one index-ordered compaction emits every forced partition,
// every candidate with key > T and the lowest-index candidates with key == T
// that are still needed.  Because emission is in index order the output is
// ascending and ties go to the lower id without any sort.
#include "spin_select_resolve_dev.h"

#define SEL_BLOCK 512

__global__ __launch_bounds__(SEL_BLOCK) void spin_select_kernel(
    const float *__restrict__ scores, const int32_t *__restrict__ part_offsets,
    const int32_t *__restrict__ seq_lens, int Hkv, int tp, int topk, int includes_forced, int sink_pages,
    int recent_pages, int sel_stride, int32_t *__restrict__ sel, int32_t *__restrict__ nsel) {
  select_generic_row<SEL_BLOCK>(scores, part_offsets, seq_lens, Hkv, tp, topk, includes_forced, sink_pages,
                                recent_pages, sel_stride, sel, nsel, (int)blockIdx.x);
}

template <int BLOCK, int KPT>
__global__ __launch_bounds__(BLOCK) void spin_select_reg_kernel(
    const float *__restrict__ scores, const int32_t *__restrict__ part_offsets,
    const int32_t *__restrict__ seq_lens, int Hkv, int tp, int topk, int includes_forced, int sink_pages,
    int recent_pages, int sel_stride, int32_t *__restrict__ sel, int32_t *__restrict__ nsel, spin_var var) {
  __shared__ reg_row_lds<BLOCK> s;
  spin_var_span span;
  (void)select_reg_row<BLOCK, KPT>(scores, part_offsets, seq_lens, Hkv, tp, topk, includes_forced, sink_pages,
                                   recent_pages, sel_row<false>{sel + (size_t)blockIdx.x * sel_stride, sel_stride, nullptr},
                                   nsel, (int)blockIdx.x, var, span, s, [] {});
}

// ---------------------------------------------------------------------------
// Rows that go by their tiles' maxima (select_by_tile_maxima): contexts of 16385 to 131072 partitions, whose rows do not
// fit the workgroup's registers.  For scores that do not come from stage 1 of the same call this launch, many workgroups
// per row, takes the maxima first.
__global__ __launch_bounds__(256) void spin_tile_max_kernel(const float *__restrict__ scores,
                                                            const int32_t *__restrict__ part_offsets, int Hkv,
                                                            int gs_log, float *__restrict__ maxima, int max_stride) {
  const int row = blockIdx.y;
  const int b = row / Hkv, h = row - b * Hkv;
  const int PP = part_offsets[b + 1] - part_offsets[b];
  const float *rs = scores + (size_t)Hkv * part_offsets[b] + (size_t)h * PP;
  // a quad of scores per lane (one contiguous KiB per wavefront); a tile is 1, 2 or 4 neighbouring lanes
  const int p = ((int)blockIdx.x * 256 + (int)threadIdx.x) * 4;
  if (p >= PP) return;                                   // PP is a multiple of 16: whole tiles leave
  const float4 v = *(const float4 *)(rs + p);
  float m = fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w));     // NaN only where all four are: ranks as -inf
  if (gs_log >= 3) m = fmaxf(m, spin_dpp<SPIN_DPP_XOR1>(m));
  if (gs_log >= 4) m = fmaxf(m, spin_dpp<SPIN_DPP_XOR2>(m));
  const int t = p >> gs_log;
  if ((p & ((1 << gs_log) - 1)) == 0 && t < max_stride) maxima[(size_t)row * max_stride + t] = m;
}

// One workgroup per row.  MPT: maxima per thread.  RESOLVE: the workgroup goes on to stage 3 for its row (same device
// function as the stage call).
// Latency bounds it: a dependent load each for maxima, scores and leaf entries, about 14 barriers, and whatever every
// wavefront does for itself.  With a chip-wide histogram of the leading 12 key bits in its place one compute unit
// walked the row's scores, and rows with many scores in the threshold's bin were searched whole: stages 2+3, 8 rows
// of 62500, k' = 244: 28.8 -> 12.7 us; 64 rows of 65536, k' = 1024: 22.8 -> 20.0; and stage 1, which counted the
// histogram in LDS, 42.7 -> 39.5 us on 8 rows of 62500.
template <int BLOCK, int MPT, bool RESOLVE, bool HELD = false>
__global__ __launch_bounds__(BLOCK) void spin_select_tiles_kernel(
    const float *__restrict__ scores, const float *__restrict__ maxima, int max_stride, int gs_log,
    const int32_t *__restrict__ part_offsets, const int32_t *__restrict__ seq_lens, int Hkv, int tp, int topk,
    int includes_forced, int sink_pages, int recent_pages, int sel_stride, int32_t *sel, int32_t *__restrict__ nsel,
    spin_resolve_args ra, int page_stride, int dir_stride, int leaf_entries, int32_t *status) {
  constexpr int CAP = 4096;
  __shared__ tiles_row_lds<BLOCK, CAP> s;
  __shared__ int32_t held_words[RESOLVE ? sizeof(held_row<HELD>) / sizeof(int32_t) : 1];
  held_row<HELD> &s_held = *(held_row<HELD> *)held_words;
  const int row = blockIdx.x;
  [[maybe_unused]] int32_t mydir = 0;
  // (with 32 maxima per thread there is no register to hold it in)
  if (RESOLVE && MPT < 32) mydir = row_dir_entry(ra.dir, dir_stride, row);
  const sel_row<HELD> rsel = {sel + (size_t)row * sel_stride, sel_stride, (spin_lds_i32 *)s_held.sel};
  const int take = select_tiles_row<BLOCK, MPT, CAP, HELD>(scores, maxima, max_stride, gs_log, part_offsets, seq_lens, Hkv,
                                                           tp, topk, includes_forced, sink_pages, recent_pages, sel, rsel,
                                                           nsel, row, s);
  if (RESOLVE) {
    if (MPT >= 32) mydir = row_dir_entry(ra.dir, dir_stride, row);
    resolve_selected<BLOCK>(s_held, rsel, mydir, row, take, sel, seq_lens, ra.dir, ra.leaf_pool, ra.leaf_chunks, Hkv,
                            tp, sink_pages, recent_pages, page_stride, dir_stride, leaf_entries, ra.slots, ra.page_ids,
                            ra.valid_mask, ra.npages, status, spin_var{}, nullptr);
  }
}

void spin_take_maxima(spin_ctx *ctx, int rows, const float *scores, const int32_t *part_offsets, float *maxima, void *stream) {
  spin_launch(ctx, SPIN_K_SELECT_HIST, spin_tile_max_kernel,
              dim3((unsigned)((ctx->max_parts + 1023) / 1024), (unsigned)rows), dim3(256), 0, (hipStream_t)stream,
              scores, part_offsets, ctx->cfg.num_kv_heads, ctx->tile_log, maxima, ctx->max_stride);
}

int spin_select_impl(spin_ctx *ctx, int32_t batch, const float *scores, const int32_t *part_offsets,
                     const int32_t *seq_lens, int32_t *sel, int32_t *nsel, void *workspace, void *stream,
                     bool maxima_ready, const spin_resolve_args *res) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch) return SPIN_ERR_INVALID;
  if (batch == 0) return SPIN_OK;
  if (!scores || !part_offsets || !seq_lens || !sel || !nsel) return SPIN_ERR_INVALID;
  const spin_config &c = ctx->cfg;
  const int rows = batch * c.num_kv_heads;
  // (rows are the second dimension of the grid that takes the maxima)
  const bool by_maxima = ctx->ws_max_off && workspace && rows <= 65535 && ctx->max_parts > 16384;
  // stage 3 in the same launch exists for the path by the tiles' maxima only
  if (res && !by_maxima) return SPIN_ERR_UNSUPPORTED;
  if (by_maxima) {
    float *maxima = (float *)((char *)workspace + ctx->ws_max_off);
    const int stride = ctx->max_stride, gs_log = ctx->tile_log;
    if (!maxima_ready) spin_take_maxima(ctx, rows, scores, part_offsets, maxima, stream);
#define SPIN_TILES_LAUNCH1(BLOCK, MPT, RESOLVE, HELD, ARGS)                                                    \
  spin_launch(ctx, SPIN_K_SELECT, spin_select_tiles_kernel<BLOCK, MPT, RESOLVE, HELD>, dim3((unsigned)rows),   \
              dim3(BLOCK), 0, (hipStream_t)stream, scores, (const float *)maxima, stride, gs_log,              \
              part_offsets, seq_lens, c.num_kv_heads, c.partition_tokens, c.topk, c.topk_includes_forced,      \
              c.sink_pages, c.recent_pages, ctx->sel_stride, sel, nsel, ARGS, ctx->page_stride,                \
              ctx->dir_stride, c.leaf_entries, (int32_t *)workspace)
#define SPIN_TILES_LAUNCH(BLOCK, MPT)                                                                          \
  do {                                                                                                         \
    if (!res) SPIN_TILES_LAUNCH1(BLOCK, MPT, false, false, spin_resolve_args{});                               \
    else if (ctx->sel_stride <= SEL_HELD) SPIN_TILES_LAUNCH1(BLOCK, MPT, true, true, *res);                    \
    else SPIN_TILES_LAUNCH1(BLOCK, MPT, true, false, *res);                                                    \
  } while (0)
    // What every wavefront does for itself favours few of them, the lines of many tiles many: 512 against 1024
    // threads, 8 rows of 62500 and k' = 244: 12.7 / 13.4 us; 64 rows of 65536 and k' = 1024: 21.2 / 19.9 us.
    const bool few = c.topk <= 512;
    if (stride <= 4096 && few) SPIN_TILES_LAUNCH(512, 8);
    else if (stride <= 4096) SPIN_TILES_LAUNCH(1024, 4);
    else if (stride <= 8192 && few) SPIN_TILES_LAUNCH(512, 16);
    else if (stride <= 8192) SPIN_TILES_LAUNCH(1024, 8);
    else SPIN_TILES_LAUNCH(1024, 32);
#undef SPIN_TILES_LAUNCH
#undef SPIN_TILES_LAUNCH1
    return spin_launch_status();
  }
#define SPIN_SELECT_ARGS                                                                                      \
  0, (hipStream_t)stream, scores, part_offsets, seq_lens, c.num_kv_heads, c.partition_tokens, c.topk,         \
      c.topk_includes_forced, c.sink_pages, c.recent_pages, ctx->sel_stride, sel, nsel
  if (ctx->max_parts <= 2048)
    spin_launch(ctx, SPIN_K_SELECT, spin_select_reg_kernel<512, 4>, dim3((unsigned)rows), dim3(512), SPIN_SELECT_ARGS, ctx->var);
  else if (ctx->max_parts <= 4096)
    spin_launch(ctx, SPIN_K_SELECT, spin_select_reg_kernel<512, 8>, dim3((unsigned)rows), dim3(512), SPIN_SELECT_ARGS, ctx->var);
  else if (ctx->max_parts <= 8192)   // 512 x 16 against 1024 x 8 and 1024 x 16, stages 2+3 of 8 rows: 9.0 / 10.4 / 11.8 us
    spin_launch(ctx, SPIN_K_SELECT, spin_select_reg_kernel<512, 16>, dim3((unsigned)rows), dim3(512), SPIN_SELECT_ARGS, ctx->var);
  else if (ctx->max_parts <= 16384)
    spin_launch(ctx, SPIN_K_SELECT, spin_select_reg_kernel<1024, 16>, dim3((unsigned)rows), dim3(1024),
                SPIN_SELECT_ARGS, ctx->var);
  else if (ctx->max_parts <= 65536)
    spin_launch(ctx, SPIN_K_SELECT, spin_select_reg_kernel<1024, 64>, dim3((unsigned)rows), dim3(1024),
                SPIN_SELECT_ARGS, ctx->var);
  else if (ctx->var.count)
    return SPIN_ERR_UNSUPPORTED;   // variable-length partitions: rows of at most 65536 partitions
  else
    spin_launch(ctx, SPIN_K_SELECT, spin_select_kernel, dim3((unsigned)rows), dim3(SEL_BLOCK), SPIN_SELECT_ARGS);
#undef SPIN_SELECT_ARGS
  return spin_launch_status();
}

extern "C" int spin_select_topk(spin_ctx *ctx, int32_t batch, const float *scores, const int32_t *part_offsets,
                                const int32_t *seq_lens, int32_t *sel, int32_t *nsel, void *workspace,
                                void *stream) {
  return spin_select_impl(ctx, batch, scores, part_offsets, seq_lens, sel, nsel, workspace, stream, false, nullptr);
}

// Stages 1 and 2 in one call: for contexts of 16385 to 131072 partitions stage 1 leaves its tiles' maxima for stage 2;
// otherwise the two stages are simply issued one after the other.  Same results as the two calls, bit for bit.
extern "C" int spin_score_select_topk(spin_ctx *ctx, int32_t batch, const void *q, const void *summaries,
                                      const int32_t *chan_idx, const int32_t *part_offsets,
                                      const int32_t *seq_lens, float *scores, int32_t *sel, int32_t *nsel,
                                      void *workspace, void *stream) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch) return SPIN_ERR_INVALID;
  if (batch == 0) return SPIN_OK;
  if (!sel || !nsel) return SPIN_ERR_INVALID;
  // (same condition as in stage 2)
  const bool fuse = ctx->max_parts > 16384 && ctx->ws_max_off && workspace && batch * ctx->cfg.num_kv_heads <= 65535;
  float *maxima = fuse ? (float *)((char *)workspace + ctx->ws_max_off) : nullptr;
  const int st = spin_score_impl(ctx, batch, q, summaries, chan_idx, part_offsets, seq_lens, scores, workspace, stream,
                                 maxima);
  if (st != SPIN_OK) return st;
  return spin_select_impl(ctx, batch, scores, part_offsets, seq_lens, sel, nsel, workspace, stream, fuse, nullptr);
}
