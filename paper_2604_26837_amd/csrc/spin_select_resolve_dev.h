// From stage 2 to stage 3 inside one launch, shared by the launches that run both for a row.
#pragma once
#include "spin_resolve_dev.h"
#include "spin_select_dev.h"

// A row's always-attended pages: its first nlo, and nhi from recent_begin on.
struct forced_span {
  int nlo, nhi, recent_begin;
};
// the same rule as stages 2 and 3: a context no longer than the two windows is attended whole
__device__ inline forced_span forced_pages_of(int N, int sink_pages, int recent_pages) {
  const int pages = (N + 15) >> 4;
  int sink_end = min(sink_pages, pages);
  int recent_begin = max(pages - recent_pages, 0);
  if (sink_end >= recent_begin) { sink_end = pages; recent_begin = pages; }
  return forced_span{sink_end, pages - recent_begin, recent_begin};
}

// The calling thread's entry of the row's directory, asked for before stage 2, whose chain hides it.  Without a
// branch, so that nothing else waits for it.
__device__ __forceinline__ int32_t row_dir_entry(const int32_t *__restrict__ dir, int dir_stride, int row) {
  return dir[(size_t)row * dir_stride + min((int)threadIdx.x, dir_stride - 1)];
}

// Stage 3 of the row that this workgroup has just selected.  What stage 3 starts from is in LDS already: the directory,
// and (HELD) the selection, which stage 2 left nowhere else and which is stored here, so that the leaf entries are the
// one trip to memory between the last of stage 2 and the page list.  Latency bounds this: against a selection stored to
// and read back from memory and a directory fetched after stage 2, whole steps, us: 64 rows of 65536 tokens, 1024 of them
// selected 55.7 -> 54.6, 8 rows of 8192 pages 28.5 -> 27.9, 8 rows of 62500 62.1 -> 61.8, 128 rows of 2048 the same.
// HELD is a variant of the kernel: told apart at every store it cost what it gained (2 rows of 256: 13.6 -> 13.9).
template <int BLOCK, bool HELD>
__device__ __forceinline__ void resolve_selected(
    held_row<HELD> &held, const sel_row<HELD> &rsel, int32_t mydir, int row, int take, int32_t *sel,
    const int32_t *__restrict__ seq_lens, const int32_t *dir, const int32_t *__restrict__ leaf_pool, int64_t leaf_chunks,
    int Hkv, int tp, int sink_pages, int recent_pages, int page_stride, int dir_stride, int leaf_entries, int32_t *__restrict__ slots,
    int32_t *__restrict__ page_ids, uint16_t *__restrict__ valid_mask, int32_t *__restrict__ npages, int32_t *status,
    spin_var var, const spin_var_span *known) {
  static_assert(BLOCK >= RES_DIR_LDS, "an entry per thread");
  const int tid = threadIdx.x;
  if (tid < RES_DIR_LDS) held.dir[tid] = mydir;
  __syncthreads();   // the selection was written by this workgroup: visible to all its threads from here
  if (HELD)
    for (int i = tid; i < take; i += BLOCK) rsel.out[i] = rsel.lds[i];
  resolve_row<BLOCK, true, true, HELD>(row, take, sel, seq_lens, dir, leaf_pool, leaf_chunks, Hkv, tp, sink_pages,
                                       recent_pages, rsel.stride, page_stride, dir_stride, leaf_entries,
                                       res_row_out(slots, page_ids, valid_mask, npages, row, page_stride), status, var, known,
                                       &held);
}
