// Stages 2, 3 and 4 in one launch (all-resident mode, uniform partitions of whole pages, rows that fit a workgroup's
// registers).
//
// A launch that depends on the one before it starts 2 to 3 us after that one's last wavefront has its result, and the
// page list goes out to memory and back in between.  Here every workgroup of a row, one per split of stage 4, selects
// and resolves the row for itself: the same device functions on the same scores, so that all of them hold the same
// list, in LDS, and no workgroup waits for another.  Split 0 stores it.  What is done more than once is a row's few KiB of
// scores and its leaf entries, on compute units that would have waited.  Whole steps, us, against the launch of stages
// 2+3 followed by that of stage 4: 128 rows of 2048 pages, 128 attended 52.6 -> 50.2; 24 rows of 512, 64 attended 23.0 ->
// 20.8; 8 rows of 8192 28.0 -> 24.7; 256 ragged rows of up to 16384 139.5 -> 137.6; 32 rows of 1024 blocks 31.5 -> 30.1;
// 512 rows of 500 and 1000 83.9 -> 72.4 and 143.5 -> 132.9 (also where the rows are more than the compute units, then).
//
// The row's always-attended pages are known before its scores are: each wavefront asks for the first of its own ahead of
// the selection and attends it when the first selected ones are under way.
#include "spin_decode_dev.h"
#include "spin_select_resolve_dev.h"

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

struct spin_step_args {
  const int32_t *leaf_pool;
  int64_t leaf_chunks;
  int32_t *sel, *nsel, *slots, *page_ids;
  uint16_t *valid_mask;
  int32_t *npages;
  const uint4 *pool;
  int64_t pool_slots;
  uint16_t *out;
  float *lse, *part_ml, *part_acc;
  int32_t *tickets, *status;
  int tp, topk, includes_forced, sink_pages, recent_pages, sel_stride, page_stride, leaf_entries;
  float scale_log2e;
};

// grid: splits x KV heads x requests
template <int KPT>
__global__ __launch_bounds__(512) void spin_select_decode_kernel(
    const float *__restrict__ scores, const int32_t *__restrict__ part_offsets, const int32_t *__restrict__ seq_lens,
    const int32_t *__restrict__ dir, const uint16_t *__restrict__ q, int Hkv, int nsplit, int G, int Hq, int dir_stride,
    spin_step_args a) {
  constexpr int WAVES = 8, BLOCK = 64 * WAVES;
  __shared__ elements_lds<BLOCK, reg_row_cap<BLOCK, KPT>()> s;
  __shared__ held_row<true> s_held;
  extern __shared__ __align__(16) float smem[];       // the merge buffers of decode_finish, then the row's page list
  spin_lds_i32 *l_slot = (spin_lds_i32 *)(smem + WAVES * G * (SPIN_HEAD_DIM + 2));
  spin_lds_u16 *l_mask = (spin_lds_u16 *)(l_slot + a.page_stride);
  const int split = blockIdx.x, h = blockIdx.y, b = blockIdx.z, row = b * Hkv + h;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, c = lane >> 4;
  const bool store = split == 0;

  // Pages are dealt round-robin, the always-attended ones (first the sink, then the recent ones) ahead of the others:
  // page v goes to split v % nsplit, wavefront (v / nsplit) % WAVES.
  const int first = wave * nsplit + split, stride = WAVES * nsplit;
  // the directory one entry per lane (larger ones: no page is asked for ahead)
  const bool ahead = dir_stride <= 64;
  const int32_t lane_dir = dir[(size_t)row * dir_stride + min(lane, dir_stride - 1)];
  spin_bf16x8 qf[4];
  load_queries(qf, q, b, h, G, Hq, n, c);

  int32_t mydir;
  page_regs rf;
  unsigned rf_mask = 0;
  forced_span fs;
  const step_sel rsel = {a.sel + (size_t)row * a.sel_stride, a.sel_stride, (spin_lds_i32 *)s_held.sel, store};
  spin_var_span span;                // (uniform partitions)
  const int take = select_reg_row<BLOCK, KPT>(
      scores, part_offsets, seq_lens, Hkv, a.tp, a.topk, a.includes_forced, a.sink_pages, a.recent_pages, rsel, a.nsel, row,
      spin_var{}, span, s, [&] {
        mydir = row_dir_entry(dir, dir_stride, row);
        const int N = seq_lens[b];
        fs = forced_pages_of(N, a.sink_pages, a.recent_pages);
        const bool mine = ahead && first < fs.nlo + fs.nhi;
        const int page = first < fs.nlo ? first : fs.recent_begin + (first - fs.nlo), ci = mine ? page / a.leaf_entries : 0;
        const int32_t chunk = __builtin_amdgcn_readlane(lane_dir, ci < dir_stride ? ci : 0);
        const bool there = mine && ci < dir_stride && chunk >= 0 && (int64_t)chunk < a.leaf_chunks;
        const int32_t slot = __builtin_amdgcn_readfirstlane(
            a.leaf_pool[there ? (size_t)chunk * a.leaf_entries + (page - ci * a.leaf_entries) : 0]);
        const bool ok = there && slot >= 0 && (int64_t)slot < a.pool_slots;
        rf_mask = ok ? page_mask(page, N) : 0u;
        load_k_tile(rf, a.pool, ok ? slot : 0, lane, rf_mask);
        load_v_tile(rf, a.pool, ok ? slot : 0, lane, rf_mask);
        __builtin_amdgcn_sched_barrier(0);
      });
  if (tid < RES_DIR_LDS) s_held.dir[tid] = mydir;
  __syncthreads();                   // the selection and the directory are whole
  if (store)
    for (int i = tid; i < take; i += BLOCK) rsel.out[i] = rsel.lds[i];
  const step_pages list = {res_row_out(a.slots, a.page_ids, a.valid_mask, a.npages, row, a.page_stride), l_slot, l_mask, store};
  const int np = resolve_row<BLOCK, true, true, true>(row, take, a.sel, seq_lens, dir, a.leaf_pool, a.leaf_chunks, Hkv, a.tp,
                                                      a.sink_pages, a.recent_pages, a.sel_stride, a.page_stride, dir_stride,
                                                      a.leaf_entries, list, a.status, spin_var{}, nullptr, &s_held);
  __syncthreads();

  // The sink pages open the list and the recent ones close it.
  softmax_state st;
  softmax_reset(st);
  const int nf = min(fs.nlo + fs.nhi, np), all = np;
  const int asked = ahead && first < nf ? 1 : 0;          // of this wavefront's pages
  const int cnt = all > first ? (all - first + stride - 1) / stride : 0;
  for (int base = asked; base == asked || base < cnt; base += 64) {
    int myslot = 0;
    unsigned mymask = 0;
    if (base + lane < cnt) {
      const int v = first + (base + lane) * stride;
      const int at = v < nf ? (v < fs.nlo ? v : max(np - fs.nhi + (v - fs.nlo), 0)) : fs.nlo + (v - nf);
      const int32_t slot = l_slot[at];
      if (slot >= 0 && (int64_t)slot < a.pool_slots) {
        myslot = slot;
        mymask = l_mask[at];
      } else if (v >= nf) {
        spin_raise(a.status, SPIN_ERR_SLOT_RANGE);        // attends to none of it
      }
    }
    attend_lane_pages<2>(st, a.pool, myslot, mymask, max(min(cnt - base, 64), 0), lane, c, qf, a.scale_log2e, [&] {
      if (base == asked && asked) tile_attend(st, tile_logits(rf, qf), rf, rf_mask, c, a.scale_log2e);
    });
  }
  decode_finish<WAVES>(st, row, split, b, h, lane, wave, n, c, G, Hq, nsplit, nsplit, a.part_ml, a.part_acc, a.tickets, a.out,
                       a.lse);
}

extern "C" int spin_select_resolve_decode(spin_ctx *ctx, int32_t batch, const float *scores, const int32_t *part_offsets,
                                          const int32_t *seq_lens, int32_t *sel, int32_t *nsel, const int32_t *dir,
                                          const int32_t *leaf_pool, int64_t leaf_chunks, int32_t *slots, int32_t *page_ids,
                                          uint16_t *valid_mask, int32_t *npages, const void *q, const void *kv_pool,
                                          int64_t pool_slots, void *out, float *lse, void *workspace, void *stream) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch || leaf_chunks <= 0 || pool_slots <= 0) return SPIN_ERR_INVALID;
  if (ctx->fused_splits == 0 || ctx->var.count) return SPIN_ERR_UNSUPPORTED;
  if (batch == 0) return SPIN_OK;
  if (!scores || !part_offsets || !seq_lens || !sel || !nsel || !dir || !leaf_pool || !slots || !page_ids ||
      !valid_mask || !npages || !q || !kv_pool || !out)
    return SPIN_ERR_INVALID;
  if (!workspace) return SPIN_ERR_WORKSPACE;
  const spin_config &c = ctx->cfg;
  char *ws = (char *)workspace;
  const spin_step_args a = {leaf_pool, leaf_chunks, sel, nsel, slots, page_ids, valid_mask, npages, (const uint4 *)kv_pool,
                            pool_slots, (uint16_t *)out, lse, (float *)(ws + ctx->ws_ml_off),
                            (float *)(ws + ctx->ws_acc_off), (int32_t *)(ws + ctx->ws_ticket_off), (int32_t *)workspace,
                            c.partition_tokens, c.topk, c.topk_includes_forced, c.sink_pages, c.recent_pages,
                            ctx->sel_stride, ctx->page_stride, c.leaf_entries, ctx->scale * 1.4426950408889634f};
#define SPIN_SD_LAUNCH(KPT)                                                                                       \
  spin_launch(ctx, SPIN_K_SELECT_DECODE, spin_select_decode_kernel<KPT>,                                          \
              dim3((unsigned)ctx->fused_splits, (unsigned)c.num_kv_heads, (unsigned)batch), dim3(512), spin_fused_lds(ctx), \
              (hipStream_t)stream, scores, part_offsets, seq_lens, dir, (const uint16_t *)q, c.num_kv_heads,      \
              ctx->fused_splits, ctx->group, c.num_q_heads, ctx->dir_stride, a)
  if (ctx->max_parts <= 2048) SPIN_SD_LAUNCH(4);
  else if (ctx->max_parts <= 4096) SPIN_SD_LAUNCH(8);
  else if (ctx->max_parts <= 8192) SPIN_SD_LAUNCH(16);
  else SPIN_SD_LAUNCH(32);
#undef SPIN_SD_LAUNCH
  return spin_launch_status();
}

extern "C" int32_t spin_fused_splits(const spin_ctx *c) { return c ? c->fused_splits : 0; }
