// The copy between pinned host memory and slots, shared by the copy kernels and by the launch that attends beside it.
#pragma once
#include "spin_common.h"

#define GATHER_ROWS 1024   // rows whose miss counts a workgroup holds as prefix sums at a time

struct host_map {
  const int32_t *table;     // NULL: identity
  int64_t entries, pages;
};

// TO_HOST = false: host page -> slot (Retrieve).  TO_HOST = true: slot -> host page (Offload's copy,
// Table 1: copy(gpu_kv, cpu_kv, map)); the lists have the same shape in both directions.
//
// The host link bounds it, provided that the pages are spread over the wavefronts whatever the rows' counts are: a
// wavefront takes every (number of wavefronts)-th page of all rows' lists, found by the prefix sums of the counts.
// (Dealt in chunks of 16 pages of one row, rows that miss 16 pages or fewer each had an eighth of 64 workgroups at
// work.  1010 pages of 64 rows: 167.6 -> 163-165 us; 6490 of 256 rows: 1016 -> 1003 us, 53 GB/s.)
// Workgroup `wg` of `wgs`.
template <bool TO_HOST, int WAVES>
__device__ __forceinline__ void copy_pages(
    int wg, int wgs, uint4 *__restrict__ host_kv, const int64_t *__restrict__ row_base, const int32_t *__restrict__ nmiss,
    const int32_t *__restrict__ miss_pages, const int32_t *__restrict__ miss_slots, uint4 *__restrict__ pool,
    int64_t pool_slots, int page_stride, int rows, int32_t *status, host_map hm) {
  __shared__ int s_end[GATHER_ROWS];     // pages of the rows up to and including this one
  __shared__ int s_wtot[WAVES];
  constexpr int RPT = GATHER_ROWS / (WAVES * 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nwaves = wgs * WAVES;
  int item = wave * wgs + wg;            // neighbouring pages go to different compute units
  for (int row0 = 0; row0 < rows; row0 += GATHER_ROWS) {
    int cnt[RPT], mine = 0;
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      const int row = row0 + threadIdx.x * RPT + j;
      const int n = row < rows ? nmiss[row] : 0;
      cnt[j] = n < 0 ? 0 : (n > page_stride ? page_stride : n);
      mine += cnt[j];
    }
    const int inc = spin_wave_inclusive_scan(mine);
    if (row0) __syncthreads();                         // the sums of the rows before have been read
    if (lane == 63) s_wtot[wave] = inc;
    __syncthreads();
    int run = inc - mine, total = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      if (w < wave) run += s_wtot[w];
      total += s_wtot[w];
    }
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      run += cnt[j];
      s_end[threadIdx.x * RPT + j] = run;
    }
    __syncthreads();
    for (; item < total; item += nwaves) {
      int lo = 0, hi = min(rows - row0, GATHER_ROWS) - 1;   // the first row whose pages end behind `item`
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (s_end[mid] > item) hi = mid; else lo = mid + 1;
      }
      const int row = row0 + lo, i = item - (lo ? s_end[lo - 1] : 0);
      const int32_t pg = miss_pages[(size_t)row * page_stride + i];
      const int32_t slot = miss_slots[(size_t)row * page_stride + i];
      if (pg < 0 || slot < 0 || (int64_t)slot >= pool_slots) {
        if (lane == 0) spin_raise(status, SPIN_ERR_SLOT_RANGE);
        continue;
      }
      int64_t hpage = row_base[row] + pg;
      if (hm.table) {                       // CPU page table: offset of the page in the row's list -> physical host page
        const bool in_table = hpage >= 0 && hpage < hm.entries;
        hpage = in_table ? hm.table[hpage] : -1;
      }
      // the host pool's size, when one was registered (with or without a table), bounds the page
      if (hpage < 0 || (hm.pages > 0 && hpage >= hm.pages)) {
        if (lane == 0) spin_raise(status, SPIN_ERR_SLOT_RANGE);
        continue;
      }
      uint4 *hp = host_kv + (size_t)hpage * SPIN_SLOT_U4 + lane;
      uint4 *dp = pool + (size_t)slot * SPIN_SLOT_U4 + lane;
      const uint4 *src = TO_HOST ? dp : hp;
      uint4 *dst = TO_HOST ? hp : dp;
      uint4 v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = src[k * 64];
#pragma unroll
      for (int k = 0; k < 8; ++k) dst[k * 64] = v[k];
    }
    item -= total;
  }
}
