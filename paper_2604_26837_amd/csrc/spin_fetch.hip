// Retrieve steps 3-4 (Section 5.2): bring the missed pages from pinned host
// memory into the slots stage 3b assigned to them.
//
// Two copiers.  The host-driven one issues one 8 KiB hipMemcpyAsync per miss on
// a side stream (needs the miss list on the host).  The device-driven one is
// the paper's copy kernel (Section 5.5): one wavefront copies one page with
// 16-byte lane transactions straight out of pinned host memory; a fixed, small number of
// workgroups deals all rows' pages to its wavefronts one by one, whatever row owns them, and the
// miss list never leaves the device.  The same kernel run the other way is Offload's copy (slot ->
// host page).
#include "spin_fetch_dev.h"

extern "C" int spin_copy_misses_host(spin_ctx *ctx, int32_t batch, const void *host_kv,
                                     const int64_t *host_row_base, const int32_t *nmiss,
                                     const int32_t *miss_pages, const int32_t *miss_slots, void *kv_pool,
                                     int64_t pool_slots, void *copy_stream, int64_t *pages_copied) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch || pool_slots <= 0) return SPIN_ERR_INVALID;
  if (pages_copied) *pages_copied = 0;
  if (batch == 0) return SPIN_OK;
  if (!host_kv || !host_row_base || !nmiss || !miss_pages || !miss_slots || !kv_pool) return SPIN_ERR_INVALID;
  const int rows = batch * ctx->cfg.num_kv_heads;
  const int stride = ctx->page_stride;
  int64_t total = 0;
  for (int r = 0; r < rows; ++r) {
    const int n = nmiss[r];
    if (n < 0 || n > stride) return SPIN_ERR_INVALID;
    for (int i = 0; i < n; ++i) {
      const int32_t pg = miss_pages[(size_t)r * stride + i], slot = miss_slots[(size_t)r * stride + i];
      if (pg < 0 || slot < 0 || (int64_t)slot >= pool_slots) return SPIN_ERR_INVALID;
      int64_t hp = host_row_base[r] + pg;
      if (ctx->cpu_table) {                 // pinned host memory: readable from here as well
        if (hp < 0 || hp >= ctx->cpu_table_entries) return SPIN_ERR_INVALID;
        hp = ctx->cpu_table[hp];
      }
      // the host pool's size, when one was registered (with or without a table), bounds the page
      if (hp < 0 || (ctx->cpu_pages > 0 && hp >= ctx->cpu_pages)) return SPIN_ERR_INVALID;
      const char *src = (const char *)host_kv + (size_t)hp * SPIN_SLOT_BYTES;
      char *dst = (char *)kv_pool + (size_t)slot * SPIN_SLOT_BYTES;
      SPIN_HIP_CHECK(hipMemcpyAsync(dst, src, SPIN_SLOT_BYTES, hipMemcpyHostToDevice, (hipStream_t)copy_stream));
      ++total;
    }
  }
  if (pages_copied) *pages_copied = total;
  return SPIN_OK;
}

#define GATHER_WAVES 4
// Workgroups of a copy launch.  The host link is the limit and, for reads of host memory, 64 wavefronts with a page each
// in flight fill it; more requests at a time slow it down (64 rows that miss 1010 pages: 4 / 8 / 12 / 16 / 32 / 64 / 128 /
// 256 workgroups -> 250 / 167 / 165 / 163-165 / 166 / 166 / 180 / 199 us) and crowd the units that other launches could use
// meanwhile.  Writes to host memory want more (16 / 32 / 64 workgroups: 256 pages 45.6 / 43.1 / 41.7 us, 512 pages
// 88.3 / 83.1 / 80.5, 1024 pages 167 / 160 / 156; from 4000 pages on they are alike).
#define GATHER_MAX_WGS 16
#define OFFLOAD_MAX_WGS 64
template <bool TO_HOST>
__global__ __launch_bounds__(GATHER_WAVES * 64) void spin_gather_kernel(
    uint4 *__restrict__ host_kv, const int64_t *__restrict__ row_base, const int32_t *__restrict__ nmiss,
    const int32_t *__restrict__ miss_pages, const int32_t *__restrict__ miss_slots, uint4 *__restrict__ pool,
    int64_t pool_slots, int page_stride, int rows, int32_t *status, host_map hm) {
  copy_pages<TO_HOST, GATHER_WAVES>(blockIdx.x, gridDim.x, host_kv, row_base, nmiss, miss_pages, miss_slots, pool, pool_slots,
                                    page_stride, rows, status, hm);
}

static unsigned copy_workgroups(int64_t most_pages, int64_t most_wgs) {
  const int64_t wgs = (most_pages + GATHER_WAVES - 1) / GATHER_WAVES;
  return (unsigned)(wgs < most_wgs ? wgs : most_wgs);
}

extern "C" int spin_gather_misses(spin_ctx *ctx, int32_t batch, const void *host_kv, const int64_t *row_base,
                                  const int32_t *nmiss, const int32_t *miss_pages, const int32_t *miss_slots,
                                  void *kv_pool, int64_t pool_slots, void *workspace, void *stream) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch || pool_slots <= 0) return SPIN_ERR_INVALID;
  if (batch == 0) return SPIN_OK;
  if (!host_kv || !row_base || !nmiss || !miss_pages || !miss_slots || !kv_pool) return SPIN_ERR_INVALID;
  if (!workspace) return SPIN_ERR_WORKSPACE;
  const int rows = batch * ctx->cfg.num_kv_heads;
  spin_launch(ctx, SPIN_K_GATHER, spin_gather_kernel<false>,
              dim3(copy_workgroups((int64_t)rows * ctx->page_stride, GATHER_MAX_WGS)), dim3(GATHER_WAVES * 64), 0,
              (hipStream_t)stream, (uint4 *)const_cast<void *>(host_kv), row_base, nmiss, miss_pages, miss_slots,
              (uint4 *)kv_pool, pool_slots, ctx->page_stride, rows, (int32_t *)workspace,
              host_map{ctx->cpu_table, ctx->cpu_table_entries, ctx->cpu_pages});
  return spin_launch_status();
}

extern "C" int spin_offload_pages(spin_ctx *ctx, int32_t batch, const void *kv_pool, int64_t pool_slots, void *host_kv,
                                  const int64_t *row_base, const int32_t *count, const int32_t *pages,
                                  const int32_t *slots, void *workspace, void *stream) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch || pool_slots <= 0) return SPIN_ERR_INVALID;
  if (batch == 0) return SPIN_OK;
  if (!host_kv || !row_base || !count || !pages || !slots || !kv_pool) return SPIN_ERR_INVALID;
  if (!workspace) return SPIN_ERR_WORKSPACE;
  const int rows = batch * ctx->cfg.num_kv_heads;
  spin_launch(ctx, SPIN_K_OFFLOAD, spin_gather_kernel<true>,
              dim3(copy_workgroups((int64_t)rows * ctx->page_stride, OFFLOAD_MAX_WGS)), dim3(GATHER_WAVES * 64), 0,
              (hipStream_t)stream, (uint4 *)host_kv, row_base, count, pages, slots,
              (uint4 *)const_cast<void *>(kv_pool), pool_slots, ctx->page_stride, rows, (int32_t *)workspace,
              host_map{ctx->cpu_table, ctx->cpu_table_entries, ctx->cpu_pages});
  return spin_launch_status();
}

extern "C" int spin_set_host_page_table(spin_ctx *ctx, const int32_t *cpu_pages, int64_t entries, int64_t host_pages) {
  if (!ctx) return SPIN_ERR_INVALID;
  if (!cpu_pages) {   // identity mapping; host_pages > 0 still bounds the pages the copiers touch
    if (host_pages < 0) return SPIN_ERR_INVALID;
    ctx->cpu_table = nullptr; ctx->cpu_table_entries = 0; ctx->cpu_pages = host_pages;
    return SPIN_OK;
  }
  if (entries <= 0 || host_pages <= 0) return SPIN_ERR_INVALID;
  ctx->cpu_table = cpu_pages; ctx->cpu_table_entries = entries; ctx->cpu_pages = host_pages;
  return SPIN_OK;
}

// Splits a row's token masks by whether the page had to be fetched: while the copy of the missed pages is under
// way, attention can already run over the pages that hit (Section 5.2, Retrieve: only the misses travel).  Both
// lists ascend by page id, so a page is a miss iff a binary search finds it in the row's miss list.
__global__ __launch_bounds__(256) void spin_split_kernel(const int32_t *__restrict__ page_ids,
                                                         const uint16_t *__restrict__ mask,
                                                         const int32_t *__restrict__ npages,
                                                         const int32_t *__restrict__ miss_pages,
                                                         const int32_t *__restrict__ nmiss, int page_stride,
                                                         uint16_t *__restrict__ mask_hits,
                                                         uint16_t *__restrict__ mask_misses) {
  const int row = blockIdx.x;
  int np = npages[row], nm = nmiss[row];
  np = np < 0 ? 0 : (np > page_stride ? page_stride : np);
  nm = nm < 0 ? 0 : (nm > page_stride ? page_stride : nm);
  const int32_t *mp = miss_pages + (size_t)row * page_stride;
  for (int i = threadIdx.x; i < page_stride; i += blockDim.x) {
    uint16_t hit = 0, miss = 0;
    if (i < np) {
      const int32_t pg = page_ids[(size_t)row * page_stride + i];
      int lo = 0, hi = nm;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (mp[mid] < pg) lo = mid + 1; else hi = mid;
      }
      const bool is_miss = lo < nm && mp[lo] == pg;
      const uint16_t m = mask[(size_t)row * page_stride + i];
      hit = is_miss ? 0 : m;
      miss = is_miss ? m : 0;
    }
    mask_hits[(size_t)row * page_stride + i] = hit;
    mask_misses[(size_t)row * page_stride + i] = miss;
  }
}

extern "C" int spin_split_hits_misses(spin_ctx *ctx, int32_t batch, const int32_t *page_ids, const uint16_t *valid_mask,
                                      const int32_t *npages, const int32_t *miss_pages, const int32_t *nmiss,
                                      uint16_t *mask_hits, uint16_t *mask_misses, void *stream) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch) return SPIN_ERR_INVALID;
  if (batch == 0) return SPIN_OK;
  if (!page_ids || !valid_mask || !npages || !miss_pages || !nmiss || !mask_hits || !mask_misses) return SPIN_ERR_INVALID;
  const int rows = batch * ctx->cfg.num_kv_heads;
  spin_launch(ctx, SPIN_K_META, spin_split_kernel, dim3((unsigned)rows), dim3(256), 0, (hipStream_t)stream, page_ids,
              valid_mask, npages, miss_pages, nmiss, ctx->page_stride, mask_hits, mask_misses);
  return spin_launch_status();
}
