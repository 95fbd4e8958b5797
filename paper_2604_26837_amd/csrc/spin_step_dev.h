// What the kernels that run stages 2 to 4 in one launch share.
#pragma once
#include "spin_decode_dev.h"
#include "spin_select_resolve_dev.h"

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
  int leaf_log;                       // log2 of leaf_entries, or -1
  int lists_at;                       // floats of dynamic LDS ahead of the row's lists
  const float *maxima;                // of the scores' tiles, 2^gs_log partitions each (step_tiles)
  int max_stride, gs_log;
  spin_var var;                       // variable-length partitions (count NULL: uniform ones)
  const uint4 *summ;                  // stage 1 in the same launch: its summaries, where its scores go,
  float *scores_out;
  int reps;                           // and summary rows per partition
  float scale_log2e;
};

// Dynamic LDS ahead of the row's lists: stage 4's merge buffers, where before that a row that goes by its tiles' maxima is
// selected (no more than SPIN_TILES_LDS, which the context is sized with).
#define STEP_CAP 4096
typedef tiles_row_lds<512, STEP_CAP> step_tiles_lds;
static_assert(sizeof(step_tiles_lds) <= SPIN_TILES_LDS, "the selection by tile maxima fits");

// scores, or tile maxima, that a thread of the launch holds
static inline int spin_step_per_thread(const spin_ctx *ctx) {
  if (ctx->step_tiles) return ctx->max_stride <= 2048 ? 4 : ctx->max_stride <= 4096 ? 8 : 16;
  return ctx->max_parts <= 2048 ? 4 : ctx->max_parts <= 4096 ? 8 : ctx->max_parts <= 8192 ? 16 : 32;
}

// Which row and split a workgroup is.  Workgroups go to the chip's 8 dies in turn; the splits of a row, which all read its
// scores, are 8 workgroups apart, on the same die, whose cache then asks for them once.
struct step_place {
  int row, split;
};
__device__ __forceinline__ step_place step_place_of(int at, int rows, int nsplit) {
  const int g = at / (8 * nsplit), in = at - g * 8 * nsplit, of = min(8, rows - 8 * g);
  const int split = in / of;
  return step_place{8 * g + in - split * of, split};
}

// a selection that stays in LDS; the caller stores it
struct lds_sel {
  int stride;
  spin_lds_i32 *lds;
  __device__ __forceinline__ void put(int pos, int32_t id) const {
    if (pos < stride) lds[pos] = id;
  }
  __device__ __forceinline__ void pad(int) const {}
  __device__ __forceinline__ void count(int32_t *, int, int) const {}
};

// the launch for partitions smaller than a page
int spin_step_tokens_launch(spin_ctx *ctx, int32_t batch, const float *scores, const int32_t *part_offsets,
                            const int32_t *seq_lens, const int32_t *dir, const void *q, const spin_step_args &a, void *stream);
