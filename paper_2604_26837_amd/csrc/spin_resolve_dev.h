// Device code of stage 3 (all-resident mode) shared by the stand-alone kernel
// and the fused launch.
#pragma once
#include "spin_common.h"

template <int RES_BLOCK>
__device__ inline int res_block_exclusive_scan(int v, int *s_wave, int &total) {
  constexpr int RES_WAVES = RES_BLOCK / 64;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int inc = spin_wave_inclusive_scan(v);
  __syncthreads();
  if (lane == 63) s_wave[wave] = inc;
  __syncthreads();
  return spin_waves_before<RES_WAVES>(s_wave[lane % RES_WAVES], wave, total) + inc - v;
}

__device__ inline uint32_t page_mask(int page, int N) {
  const int n = min(max(N - page * 16, 0), 16);
  return (1u << n) - 1u;
}

// where a row's page list goes
struct res_out {
  int32_t *slots, *page_ids;
  uint16_t *mask;
  int32_t *npages;
  __device__ __forceinline__ void put(int pos, int32_t slot, int32_t page, uint32_t m) const {
    slots[pos] = slot;
    page_ids[pos] = page;
    mask[pos] = (uint16_t)m;
  }
  __device__ __forceinline__ void count(int total) const { *npages = total; }
};
__device__ __forceinline__ res_out res_row_out(int32_t *__restrict__ slots, int32_t *__restrict__ page_ids,
                                               uint16_t *__restrict__ valid_mask, int32_t *__restrict__ npages, int row,
                                               int page_stride) {
  const size_t at = (size_t)row * page_stride;
  return res_out{slots + at, page_ids + at, valid_mask + at, npages + row};
}

#define RES_DIR_LDS 256
#define SEL_HELD SPIN_SEL_HELD

// What the launch that selects a row has of it in LDS when it goes on to stage 3: the selection (HELD: no longer than
// SEL_HELD) and the directory entries (where at most RES_DIR_LDS).
template <bool HELD>
struct held_row {
  int32_t sel[HELD ? SEL_HELD : 1];
  int32_t dir[RES_DIR_LDS];
};

// a row's directory, in LDS when it fits.  (Told apart by a branch: through a pointer to either, every lookup would be
// a generic load that waits for all memory and LDS operations under way.)
struct row_dir {
  const int32_t *global;
  spin_lds_i32 *lds;
  bool in_lds;
  __device__ __forceinline__ int32_t at(int i) const {
    if (in_lds) return lds[i];
    return global[i];
  }
};

// LOOKUP = false: only the page list and the masks are wanted (budget mode decides the slots)
template <bool LOOKUP, typename OUT>
__device__ __forceinline__ void emit_page(const OUT &o, int pos, int page_stride, int page, uint32_t mask,
                                          const row_dir &dir, const int32_t *__restrict__ leaf_pool, int64_t leaf_chunks,
                                          int dir_stride, int leaf_entries, int32_t *status) {
  if (pos < 0 || pos >= page_stride) return;
  int32_t slot = -1;
  if (LOOKUP) {
    const int ci = page < 0 ? dir_stride : page / leaf_entries;
    if (ci < dir_stride) {
      const int32_t chunk = dir.at(ci);
      if (chunk >= 0 && (int64_t)chunk < leaf_chunks)
        slot = leaf_pool[(size_t)chunk * leaf_entries + (page - ci * leaf_entries)];
    }
    if (slot < 0) {
      spin_raise(status, SPIN_ERR_NOT_RESIDENT);
      slot = -1;
      mask = 0;
    }
  }
  o.put(pos, slot, page, mask);
}

// A selection entry outside the row: its output position holds no page (nothing of a previous
// step stays there for stage 4 to attend) and the fault is reported.
template <typename OUT>
__device__ inline void emit_invalid(const OUT &o, int pos, int page_stride, int32_t *status) {
  spin_raise(status, SPIN_ERR_INVALID);
  if (pos < 0 || pos >= page_stride) return;
  o.put(pos, -1, -1, 0);
}

// Resolves one row with the calling workgroup of RES_BLOCK threads; `ns` = the
// row's selection count.  `known`: the row's windows, where the caller has them
// (variable-length partitions).  HELD_DIR, HELD_SEL: the calling launch has staged the row's directory, or its selection,
// in `held`.  TABLES > 0: so are the row's partition tables in `tables`, first pages [TABLES] and then tokens.  Returns the
// length of the page list.
template <int RES_BLOCK, bool LOOKUP = true, bool HELD_DIR = false, bool HELD_SEL = false, int TABLES = 0, typename OUT>
__device__ __forceinline__ int resolve_row(
    int row, int ns, const int32_t *__restrict__ sel, const int32_t *__restrict__ seq_lens,
    const int32_t *dir, const int32_t *__restrict__ leaf_pool, int64_t leaf_chunks, int Hkv, int tp,
    int sink_pages, int recent_pages, int sel_stride, int page_stride, int dir_stride, int leaf_entries, const OUT &o,
    int32_t *status, spin_var var, const spin_var_span *known = nullptr,
    held_row<HELD_SEL> *held = nullptr, const int32_t *tables = nullptr) {
  constexpr int RES_WAVES = RES_BLOCK / 64;
  __shared__ int s_wave[RES_WAVES];
  __shared__ int s_flagA, s_flagB, s_cntB;
  __shared__ int32_t s_dir[HELD_DIR ? 1 : RES_DIR_LDS];
  const int tid = threadIdx.x;
  const int b = row / Hkv;
  // the row's directory entries are fetched together with its selection, so the
  // leaf lookups below are the only dependent round trip
  const int32_t *gdir = dir + (size_t)row * dir_stride;
  const bool dir_in_lds = dir_stride <= RES_DIR_LDS;
  if (!HELD_DIR && dir_in_lds)
    for (int i = tid; i < dir_stride; i += RES_BLOCK) s_dir[i] = gdir[i];
  const row_dir rdir = {gdir, (spin_lds_i32 *)(HELD_DIR ? held->dir : s_dir), dir_in_lds};
  const int N = seq_lens[b];
  const int pages = (N + 15) >> 4;
  ns = ns < 0 ? 0 : (ns > sel_stride ? sel_stride : ns);
  const int32_t *rsel = sel + (size_t)row * sel_stride;
  spin_lds_i32 *lsel = (spin_lds_i32 *)(HELD_SEL ? held->sel : s_dir);
  auto sel_at = [&](int i) -> int32_t {
    if (HELD_SEL) return lsel[i];
    return rsel[i];
  };
  if (!HELD_DIR && dir_in_lds) __syncthreads();

  if (var.count) {
    // Variable-length partitions: the page list of partition p starts at
    // first_page[p] and holds ceil(tokens[p]/16) pages (Partition Offset and
    // Meta-partition tables).  Output positions come from a prefix sum of the
    // selected partitions' page counts; then every thread takes output pages
    // (found back through the sums in LDS), so that all leaf lookups are under
    // way at once.  One thread per partition, with its lookups one after the
    // other: stages 2+3 of 32 rows of up to 2400 clusters, 32 clusters selected,
    // 18.3 us together with the binary searches for the windows; now 10.9.
    __shared__ int s_sumA, s_sumB;
    const size_t vb = spin_var_base(var, row, Hkv);
    const int PP = var.part_offsets[b + 1] - var.part_offsets[b];
    const spin_var_span w = known ? *known : spin_var_span_of(var, vb, row, PP, sink_pages, recent_pages);
    const int P = w.P;
    // selection entry i: partition (-1: names none of the row), first page, tokens
    struct part { int s, first, tokens; };
    auto first_of = [&](int p) { return TABLES ? tables[p] : var.first_page[vb + p]; };
    auto tokens_of = [&](int p) { return TABLES ? tables[TABLES + p] : var.tokens[vb + p]; };
    auto entry = [&](int i) {
      part e = {sel_at(i), 0, 0};
      if (e.s < 0 || e.s >= P) e.s = -1;
      else { e.first = first_of(e.s); e.tokens = tokens_of(e.s); }
      return e;
    };
    part mine = {-1, 0, 0};
    if (tid < ns) mine = entry(tid);
    // partition A straddles the end of the sink pages, B the beginning of the recent ones
    part pa = {w.sink_end > 0 ? w.at_sink : -1, 0, 0}, pb = {w.recent_begin < w.pages ? w.at_recent : -1, 0, 0};
    if (pa.s >= 0) { pa.first = first_of(pa.s); pa.tokens = tokens_of(pa.s); }
    if (pb.s >= 0) { pb.first = first_of(pb.s); pb.tokens = tokens_of(pb.s); }
    const int endA = pa.first + ((pa.tokens + 15) >> 4), endB = pb.first + ((pb.tokens + 15) >> 4);
    const int A = pa.s >= 0 && endA > w.sink_end ? pa.s : -1, B = pb.s >= 0 && pb.first < w.recent_begin ? pb.s : -1;
    if (tid == 0) { s_flagA = 0; s_flagB = 0; s_sumA = 0; s_sumB = 0; }
    __syncthreads();
    for (int i = tid; i < ns; i += RES_BLOCK) {
      const part e = i == tid ? mine : entry(i);
      if (e.s < 0) { spin_raise(status, SPIN_ERR_INVALID); continue; }   // takes no output position
      const int n = (e.tokens + 15) >> 4;
      if (e.s == A) s_flagA = 1;
      if (e.s == B) s_flagB = 1;
      if (A >= 0 && e.s < A) atomicAdd(&s_sumA, n);
      if (B >= 0 && e.s < B) atomicAdd(&s_sumB, n);
    }
    __syncthreads();
    const int extraA = (A >= 0 && !s_flagA) ? (w.sink_end - pa.first) : 0;
    const int extraB = (B >= 0 && !s_flagB) ? (endB - w.recent_begin) : 0;
    auto put = [&](int pos, const part &e, int k) {      // page k of partition e
      const int nv = min(max(e.tokens - 16 * k, 0), 16);
      emit_page<LOOKUP>(o, pos, page_stride, e.first + k, (1u << nv) - 1u, rdir, leaf_pool, leaf_chunks, dir_stride,
                        leaf_entries, status);
    };
    auto shift = [&](int s) { return ((extraA && s > A) ? extraA : 0) + ((extraB && s > B) ? extraB : 0); };
    int carry = 0;
    for (int i0 = 0; i0 < ns; i0 += RES_BLOCK) {
      const int i = i0 + tid;
      const part e = i0 == 0 ? mine : (i < ns ? entry(i) : part{-1, 0, 0});
      const int n = e.s >= 0 ? (e.tokens + 15) >> 4 : 0;
      int tot;
      const int before = res_block_exclusive_scan<RES_BLOCK>(n, s_wave, tot);
      if constexpr (LOOKUP) {
        __shared__ int s_before[RES_BLOCK], s_at[RES_BLOCK];
        __shared__ part s_part[RES_BLOCK];
        s_before[tid] = before;
        s_at[tid] = carry + before + shift(e.s);
        s_part[tid] = e;
        __syncthreads();
        for (int x = tid; x < tot; x += RES_BLOCK) {
          int lo = 0, hi = min(ns - i0, RES_BLOCK) - 1;   // the last entry that begins at or before x: it has page x
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_before[mid] <= x) lo = mid; else hi = mid - 1;
          }
          const int k = x - s_before[lo];
          put(s_at[lo] + k, s_part[lo], k);
        }                                                // (the next round's scan has a barrier before it writes)
      } else if (e.s >= 0) {
        // no lookups to wait for: a thread lists its partition's pages
        for (int k = 0; k < n; ++k) put(carry + before + shift(e.s) + k, e, k);
      }
      carry += tot;
    }
    for (int k = tid; k < extraA; k += RES_BLOCK) put(s_sumA + k, pa, k);
    for (int k = tid; k < extraB; k += RES_BLOCK)
      put(s_sumB + ((A >= 0 && A <= B) ? extraA : 0) + k, pb, w.recent_begin - pb.first + k);
    const int total = min(carry + extraA + extraB, page_stride);
    for (int i = total + tid; i < page_stride; i += RES_BLOCK) o.put(i, -1, -1, 0);
    if (tid == 0) o.count(total);
    return total;
  } else if (tp == 16) {
    // partition == page: the selection is the page list.  The entry is loaded
    // before the row's counts are known (the buffer is sel_stride wide), so the
    // leaf lookup is the only dependent round trip.
    for (int i0 = 0; i0 < sel_stride; i0 += RES_BLOCK) {
      const int i = i0 + tid;
      const int s = i < sel_stride ? sel_at(i) : -1;
      if (i < ns) {
        if (s >= 0 && s < pages)
          emit_page<LOOKUP>(o, i, page_stride, s, page_mask(s, N), rdir, leaf_pool, leaf_chunks, dir_stride,
                        leaf_entries, status);
        else
          emit_invalid(o, i, page_stride, status);   // an entry that names no page of the row
      }
      if (i0 + RES_BLOCK >= ns) break;
    }
    const int total = min(ns, page_stride);
    for (int i = total + tid; i < page_stride; i += RES_BLOCK) o.put(i, -1, -1, 0);
    if (tid == 0) o.count(total);
    return total;
  } else if (tp > 16) {
    const int m = tp >> 4;
    int sink_end = min(sink_pages, pages);
    int recent_begin = max(pages - recent_pages, 0);
    if (sink_end >= recent_begin) { sink_end = pages; recent_begin = pages; }
    // partition partly covered by the sink pages / by the recent pages (or -1)
    int A = -1, B = -1, a0 = 0, a1 = 0, b0 = 0, b1 = 0;
    if (m > 1 && sink_end > 0) {
      const int pa = (sink_end - 1) / m;
      if (min((pa + 1) * m, pages) > sink_end) { A = pa; a0 = pa * m; a1 = sink_end; }
    }
    if (m > 1 && recent_begin < pages) {
      const int pb = recent_begin / m;
      if (pb * m < recent_begin) { B = pb; b0 = recent_begin; b1 = min((pb + 1) * m, pages); }
    }
    if (tid == 0) { s_flagA = 0; s_flagB = 0; s_cntB = 0; }
    __syncthreads();
    int below_b = 0;
    for (int i = tid; i < ns; i += RES_BLOCK) {
      const int s = sel_at(i);
      if (s == A) s_flagA = 1;
      if (s == B) s_flagB = 1;
      below_b += (B >= 0 && s < B);
    }
    if (B >= 0 && below_b) atomicAdd(&s_cntB, below_b);
    __syncthreads();
    const int extraA = (A >= 0 && !s_flagA) ? (a1 - a0) : 0;   // standalone sink pages
    const int extraB = (B >= 0 && !s_flagB) ? (b1 - b0) : 0;   // standalone recent pages
    const int sel_below_b = s_cntB;
    // pages of the selected partitions
    for (int idx = tid; idx < ns * m; idx += RES_BLOCK) {
      const int i = idx / m, k = idx - i * m;
      const int s = sel_at(i);
      const int pg = s * m + k;
      int pos = i * m + k;
      if (extraA && s > A) pos += extraA;
      if (extraB && s > B) pos += extraB;
      if (s < 0 || (int64_t)s * m >= pages) {        // an entry that names no partition of the row
        emit_invalid(o, pos, page_stride, status);
        continue;
      }
      if (pg >= pages) continue;                     // the ragged end of the context's last partition
      emit_page<LOOKUP>(o, pos, page_stride, pg, page_mask(pg, N), rdir, leaf_pool, leaf_chunks, dir_stride,
                        leaf_entries, status);
    }
    // standalone forced pages: partitions 0..A-1 are wholly forced, hence selected
    for (int k = tid; k < extraA; k += RES_BLOCK)
      emit_page<LOOKUP>(o, A * m + k, page_stride, a0 + k, page_mask(a0 + k, N), rdir, leaf_pool, leaf_chunks, dir_stride,
                        leaf_entries, status);
    for (int k = tid; k < extraB; k += RES_BLOCK)
      emit_page<LOOKUP>(o, sel_below_b * m + ((A >= 0 && A <= B) ? extraA : 0) + k, page_stride, b0 + k,
                        page_mask(b0 + k, N), rdir, leaf_pool, leaf_chunks, dir_stride, leaf_entries, status);
    // total: only the context's last partition can be short
    int total = ns * m + extraA + extraB;
    if (ns > 0) {
      const int last = sel_at(ns - 1);
      total -= max((last + 1) * m - pages, 0);
    }
    total = min(total, page_stride);
    for (int i = total + tid; i < page_stride; i += RES_BLOCK) o.put(i, -1, -1, 0);
    if (tid == 0) o.count(total);
    return total;
  } else {
    const int ppp = 16 / tp;   // partitions per page: a power of two
    const int ppp_log = 31 - __clz(ppp);
    auto page_of = [&](int s) { return (s + ((s >> 31) & (ppp - 1))) >> ppp_log; };   // s / ppp
    int carry = 0;
    for (int i0 = 0; i0 < ns; i0 += RES_BLOCK) {
      const int i = i0 + tid;
      int first = 0, pg = -1;
      if (i < ns) {
        pg = page_of(sel_at(i));
        first = (i == 0) || (page_of(sel_at(i - 1)) != pg);
      }
      int tot;
      const int before = res_block_exclusive_scan<RES_BLOCK>(first, s_wave, tot);
      if (first) {
        uint32_t mk = 0;
        for (int j = i; j < ns && j < i + ppp; ++j) {
          const int s = sel_at(j);
          if (page_of(s) != pg) break;
          const int t0 = s * tp, cnt = min(tp, N - t0);
          if (s < 0 || cnt <= 0) { spin_raise(status, SPIN_ERR_INVALID); continue; }   // names no token of the row
          mk |= ((1u << cnt) - 1u) << (t0 & 15);
        }
        emit_page<LOOKUP>(o, carry + before, page_stride, pg, mk, rdir, leaf_pool, leaf_chunks, dir_stride,
                        leaf_entries, status);
      }
      carry += tot;
    }
    const int total = min(carry, page_stride);
    for (int i = total + tid; i < page_stride; i += RES_BLOCK) o.put(i, -1, -1, 0);
    if (tid == 0) o.count(total);
    return total;
  }
}

