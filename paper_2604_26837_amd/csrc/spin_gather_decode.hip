// Retrieve steps 3-4 and stage 4 in two launches (budget mode, partitions of whole pages): the launch that copies the
// missed pages attends the others meanwhile, and a second one attends the missed pages, starting from its partial.
//
// The host link bounds the copy, which a few workgroups keep busy; the rest of the chip waited for it, and all of stage 4
// came behind.  The workgroups that copy come first in the launch and wait for nothing; those that attend leave the row's
// merged partial, as the first of two passes over one page list does, and write down the masks of the row's missed pages,
// which the second launch has as a list of its own: a few pages to a row, not the whole list under masks.  Rows that miss
// none have their output from the first.
// Step of 64 rows, 128 pages attended, about 1010 pages missed in all: 207.6 -> 196.9 us (stage 4 behind the copy 16.7 ->
// 7.1; the copy as before, 160).  With the 64 copying wavefronts in 8 workgroups instead of 16 the copy took 165.
// 8 rows, 64 pages attended, 82 missed 39.0 -> 35.6; 8 rows, 128 attended, none missed 28.1 -> 28.1 (32.0 with a second pass
// over empty lists).
// Copy and stage 4 alone, replayed from a graph, us, one after the other / these two launches, with 0, 5, 20, 50 and 200
// pages missed in all: 8 rows, 128 attended 10.6 / 10.3, 12.9 / 13.0, 15.3 / 13.3, 20.1 / 15.6, 42.7 / 39.9; 64 rows
// 15.2 / 15.6, 17.4 / 19.6, 19.9 / 21.0, 24.7 / 24.7, 47.7 / 38.3; 128 rows 26.6 / 26.7, 29.0 / 30.4, 31.3 / 30.7, 36.0 /
// 32.9, 58.4 / 44.7.  So the few pages of a step that hardly misses cost 64 rows and more 1 to 2 us: their workgroups fill
// the chip, and those that take the place of the copying ones start behind them.  (At most 168 registers, so that they
// would fit beside these, spill: 64 rows, none missed 21.3.)
#include "spin_decode_dev.h"
#include "spin_fetch_dev.h"

#define COPY_WGS 16    // of COPY_WAVES: the 64 wavefronts that fill the link
#define COPY_WAVES 4

__global__ __launch_bounds__(512) void spin_gather_decode_kernel(
    const uint16_t *__restrict__ q, uint4 *pool, int64_t pool_slots, const int32_t *__restrict__ slots,
    const uint16_t *__restrict__ masks, const int32_t *__restrict__ npages, int page_stride, int G, int Hq, int Hkv,
    int nsplit, int pstride, int rows, const int32_t *__restrict__ page_ids, uint4 *__restrict__ host_kv,
    const int64_t *__restrict__ row_base, const int32_t *__restrict__ nmiss, const int32_t *__restrict__ miss_pages,
    const int32_t *__restrict__ miss_slots, uint16_t *__restrict__ miss_mask, host_map hm, float scale_log2e, float *part_ml,
    float *part_acc, int32_t *tickets, uint16_t *__restrict__ out, float *__restrict__ lse, int32_t *status) {
  if (blockIdx.x < COPY_WGS) {
    if (threadIdx.x >= COPY_WAVES * 64) return;          // whole wavefronts: a barrier does not wait for those that have ended
    copy_pages<false, COPY_WAVES>(blockIdx.x, COPY_WGS, host_kv, row_base, nmiss, miss_pages, miss_slots, pool, pool_slots,
                                  page_stride, rows, status, hm);
    return;
  }
  const int at = blockIdx.x - COPY_WGS, row = at / nsplit;
  int nm = nmiss[row];
  nm = nm < 0 ? 0 : (nm > page_stride ? page_stride : nm);
  const size_t list = (size_t)row * page_stride;
  const int32_t *missed = miss_pages + list;
  // both lists ascend by page
  auto hits = [&](int p, unsigned mask) {
    if (nm == 0) return mask;                            // uniform
    const int32_t page = page_ids[list + p];
    int lo = 0, hi = nm;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (missed[mid] < page) lo = mid + 1; else hi = mid;
    }
    if (lo >= nm || missed[lo] != page) return mask;
    miss_mask[list + lo] = (uint16_t)mask;
    return 0u;
  };
  decode_row<8, 2>(row, at - row * nsplit, q, pool, pool_slots, slots, masks, npages, page_stride, G, Hq, Hkv, nsplit, pstride,
                   nullptr, nm ? SPIN_DECODE_TO_PARTIAL : 0, 0, scale_log2e, part_ml, part_acc, tickets, out, lse, status, hits);
}

extern "C" int spin_gather_decode(spin_ctx *ctx, int32_t batch, const void *q, const void *host_kv, const int64_t *row_base,
                                  const int32_t *nmiss, const int32_t *miss_pages, const int32_t *miss_slots, void *kv_pool,
                                  int64_t pool_slots, const int32_t *slots, const int32_t *page_ids,
                                  const uint16_t *valid_mask, const int32_t *npages, uint16_t *miss_mask, void *out, float *lse,
                                  void *workspace, void *stream) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch || pool_slots <= 0) return SPIN_ERR_INVALID;
  if (ctx->k_token_major) return SPIN_ERR_UNSUPPORTED;
  if (batch == 0) return SPIN_OK;
  if (!q || !host_kv || !row_base || !nmiss || !miss_pages || !miss_slots || !kv_pool || !slots || !page_ids || !valid_mask ||
      !npages || !miss_mask || !out)
    return SPIN_ERR_INVALID;
  if (!workspace) return SPIN_ERR_WORKSPACE;
  const spin_config &c = ctx->cfg;
  const int rows = batch * c.num_kv_heads;
  char *ws = (char *)workspace;
  float *ml = (float *)(ws + ctx->ws_ml_off), *acc = (float *)(ws + ctx->ws_acc_off);
  int32_t *tickets = (int32_t *)(ws + ctx->ws_ticket_off), *status = (int32_t *)workspace;
  const size_t lds = (size_t)8 * ctx->group * (SPIN_HEAD_DIM + 2) * sizeof(float);
  spin_launch(ctx, SPIN_K_GATHER, spin_gather_decode_kernel, dim3((unsigned)(COPY_WGS + rows * ctx->splits)), dim3(512), lds,
              (hipStream_t)stream, (const uint16_t *)q, (uint4 *)kv_pool, pool_slots, slots, valid_mask, npages,
              ctx->page_stride, ctx->group, c.num_q_heads, c.num_kv_heads, ctx->splits, ctx->pstride, rows, page_ids,
              (uint4 *)const_cast<void *>(host_kv), row_base, nmiss, miss_pages, miss_slots, miss_mask,
              host_map{ctx->cpu_table, ctx->cpu_table_entries, ctx->cpu_pages}, ctx->scale * 1.4426950408889634f, ml, acc,
              tickets, (uint16_t *)out, lse, status);
  const int st = spin_launch_status();
  if (st != SPIN_OK) return st;
  return decode_launch(ctx, batch, q, kv_pool, pool_slots, miss_slots, miss_mask, nmiss, out, lse, ml, acc, tickets, status,
                       nullptr, SPIN_DECODE_FROM_PARTIAL | SPIN_DECODE_LISTED, 1, stream);
}
