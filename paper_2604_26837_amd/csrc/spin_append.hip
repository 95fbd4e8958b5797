// Index at decode time (Section 4.1: Index is invoked during decode to
// incorporate newly generated tokens): append one token's K/V per row into its
// page slot and bring the summaries of the partition it lands in up to date.
//
// One workgroup of 128 threads per row, thread d = channel d.  The summary
// update reproduces what a full rebuild would store: min/max fold in the new key
// (or restart on the first token of a partition), the sketch row is written,
// and a block representative is recomputed from the keys in the pool with the
// same exact fp64 sum and single rounding as the bulk builder.
//
// Latency bounds it.  A representative's keys were read token by token, each behind its own walk through the page
// table; now lanes walk its pages side by side, the new token's among them, and the keys of four pages are asked for
// at once and added up in the same order; pages without tokens before the new one are passed over, so that the first
// token of a sub-range costs no more than it did.  A partition with one representative, 128 rows, a launch after the
// other: token 0 / 3 / 15 / 64 / 127 of it 2.9 / 3.7 / 6.8 / 19.9 / 36.5 -> 2.9 / 3.8 / 3.8 / 4.9 / 5.9 us.
#include "spin_common.h"

__device__ inline size_t k_elem(int token_major, int t, int d) {
  return ((size_t)spin_k_unit(token_major, t, d >> 3) << 3) + (d & 7);
}
__device__ inline size_t v_elem(int token_major, int t, int d) {
  if (token_major) return (size_t)t * SPIN_HEAD_DIM + d;
  return (((size_t)((d >> 5) * 64 + (t >> 2) * 16 + (d & 15)) * 2 + ((d >> 4) & 1)) << 2) + (t & 3);
}
__device__ inline size_t summ_elem(size_t R, int e, int kd, int kc) {
  return (R >> 4) * (size_t)(16 * kd) + ((size_t)(e / kc) * 16 + (R & 15)) * kc + (e % kc);
}
__device__ inline uint16_t f64_to_bf16(double x) {
  float f = __double2float_rz(x);
  uint32_t u = __float_as_uint(f);
  if ((double)f != x) u |= 1u;   // sticky bit: round to odd, then one rounding to bf16
  return spin_f32_to_bf16(__uint_as_float(u));
}

__global__ __launch_bounds__(128) void spin_append_kernel(
    const uint16_t *__restrict__ k_new, const uint16_t *__restrict__ v_new, const int32_t *__restrict__ seq_lens,
    uint16_t *pool, int64_t pool_slots, const int32_t *__restrict__ dir, const int32_t *__restrict__ leaf_pool,
    int64_t leaf_chunks, const int32_t *__restrict__ part_offsets, const int32_t *__restrict__ chan,
    uint16_t *summ, int Hkv, int tp, int kind, int reps, int sub, int dir_stride, int leaf_entries, int k_token_major,
    int32_t *status) {
  const int row = blockIdx.x, d = threadIdx.x;
  const int b = row / Hkv, h = row - b * Hkv;
  const int t = seq_lens[b];                 // position of the new token
  const int PP = part_offsets[b + 1] - part_offsets[b];
  const int p = t / tp;
  if (t < 0 || p >= PP) {                     // no room reserved for this partition
    if (d == 0) spin_raise(status, SPIN_ERR_INVALID);
    return;
  }
  // representative: the sub-range of `sub` tokens that the new one lands in starts at t0; lane i of either wavefront
  // holds the slot of its i-th page (the token's own is page `last`; in the first page one walk on scalars serves)
  const int at = kind == SPIN_SCORE_REPMAX ? t / sub : t;
  const int r = at - p * reps, t0 = kind == SPIN_SCORE_REPMAX ? at * sub : t;
  const int first = t0 >> 4, last = (t >> 4) - first, lane = d & 63;
  int32_t mine = -1, slot;
  if (last > 0 && lane <= last)
    mine = spin_walk(dir, leaf_pool, leaf_chunks, row, dir_stride, leaf_entries, first + lane);
  if (last > 0 && last < 64) slot = __builtin_amdgcn_readlane(mine, last);
  else slot = spin_walk(dir, leaf_pool, leaf_chunks, row, dir_stride, leaf_entries, t >> 4);
  if (last == 0) mine = slot;
  if (slot < 0 || (int64_t)slot >= pool_slots) {
    if (d == 0) spin_raise(status, SPIN_ERR_NOT_RESIDENT);
    return;
  }
  uint16_t *page = pool + (size_t)slot * (SPIN_SLOT_U4 * 8);
  const uint16_t kb = k_new[(size_t)row * SPIN_HEAD_DIM + d];
  const uint16_t vb = v_new[(size_t)row * SPIN_HEAD_DIM + d];
  page[k_elem(k_token_major, t & 15, d)] = kb;
  page[SPIN_KTILE_U4 * 8 + v_elem(k_token_major, t & 15, d)] = vb;

  const size_t base = (size_t)Hkv * part_offsets[b] + (size_t)h * PP;
  const bool first_in_part = (t == p * tp);
  if (kind == SPIN_SCORE_MINMAX) {
    const size_t R = base + p;
    uint16_t *mx = summ + summ_elem(R, d, 256, 8), *mn = summ + summ_elem(R, 128 + d, 256, 8);
    const float k = spin_bf16_to_f32(kb);
    if (first_in_part) { *mx = kb; *mn = kb; }
    else {
      if (k > spin_bf16_to_f32(*mx)) *mx = kb;
      if (k < spin_bf16_to_f32(*mn)) *mn = kb;
    }
  } else if (kind == SPIN_SCORE_SKETCH) {
    if (d < 16) summ[summ_elem(base + t, d, 16, 4)] = k_new[(size_t)row * SPIN_HEAD_DIM + chan[h * 16 + d]];
  } else {
    // representative of the sub-range the token lands in: mean of its keys so far
    double acc = (double)spin_bf16_to_f32(kb);
    for (int j = 0; t0 < t && j <= last; j += 4) {
      if (j && (j & 63) == 0)
        mine = j + lane <= last
                   ? spin_walk(dir, leaf_pool, leaf_chunks, row, dir_stride, leaf_entries, first + j + lane) : -1;
      uint16_t key[4][SPIN_PAGE_TOKENS];
      bool there[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // pages that hold tokens before the new one
        const bool wanted = j + i <= last && (first + j + i) * SPIN_PAGE_TOKENS < t;
        const int32_t s2 = __builtin_amdgcn_readlane(mine, (j + i) & 63);
        there[i] = wanted && s2 >= 0 && (int64_t)s2 < pool_slots;
        if (there[i]) {
          const uint16_t *tile = pool + (size_t)s2 * (SPIN_SLOT_U4 * 8);
#pragma unroll
          for (int x = 0; x < SPIN_PAGE_TOKENS; ++x) key[i][x] = tile[k_elem(k_token_major, x, d)];
        } else if (wanted && d == 0) {
          spin_raise(status, SPIN_ERR_NOT_RESIDENT);
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (!there[i]) continue;                           // uniform, as are the page's bounds
        const int u0 = (first + j + i) * SPIN_PAGE_TOKENS, lo = t0 - u0, hi = t - u0;
        if (lo <= 0 && hi >= SPIN_PAGE_TOKENS) {
#pragma unroll
          for (int x = 0; x < SPIN_PAGE_TOKENS; ++x) acc += (double)spin_bf16_to_f32(key[i][x]);
        } else {
#pragma unroll
          for (int x = 0; x < SPIN_PAGE_TOKENS; ++x)
            if (x >= lo && x < hi) acc += (double)spin_bf16_to_f32(key[i][x]);
        }
      }
    }
    const uint16_t m = f64_to_bf16(acc / (double)(t - t0 + 1));
    const size_t R = (base + p) * reps;
    summ[summ_elem(R + r, d, 128, 8)] = m;
    // sub-ranges that hold no token yet repeat representative 0
    if (r == 0)
      for (int r2 = 1; r2 < reps; ++r2) summ[summ_elem(R + r2, d, 128, 8)] = m;
  }
}

extern "C" int spin_append_kv(spin_ctx *ctx, int32_t batch, const void *k_new, const void *v_new,
                              const int32_t *seq_lens, void *kv_pool, int64_t pool_slots, const int32_t *dir,
                              const int32_t *leaf_pool, int64_t leaf_chunks, const int32_t *part_offsets,
                              const int32_t *chan_idx, void *summaries, void *workspace, void *stream) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch || pool_slots <= 0 || leaf_chunks <= 0) return SPIN_ERR_INVALID;
  if (batch == 0) return SPIN_OK;
  if (!k_new || !v_new || !seq_lens || !kv_pool || !dir || !leaf_pool || !part_offsets || !summaries)
    return SPIN_ERR_INVALID;
  if (!workspace) return SPIN_ERR_WORKSPACE;
  // the kernel finds the token's partition by division: not with registered partition tables
  if (ctx->var.count) return SPIN_ERR_UNSUPPORTED;
  const spin_config &c = ctx->cfg;
  if (c.score_kind == SPIN_SCORE_SKETCH && (!chan_idx || c.partition_tokens != 1)) return SPIN_ERR_INVALID;
  const int rows = batch * c.num_kv_heads;
  spin_launch(ctx, SPIN_K_APPEND, spin_append_kernel, dim3((unsigned)rows), dim3(128), 0, (hipStream_t)stream,
              (const uint16_t *)k_new, (const uint16_t *)v_new, seq_lens, (uint16_t *)kv_pool, pool_slots, dir,
              leaf_pool, leaf_chunks, part_offsets, chan_idx, (uint16_t *)summaries, c.num_kv_heads,
              c.partition_tokens, c.score_kind, c.reps_per_partition,
              c.score_kind == SPIN_SCORE_REPMAX ? c.partition_tokens / c.reps_per_partition : 1, ctx->dir_stride, c.leaf_entries,
              ctx->k_token_major, (int32_t *)workspace);
  return spin_launch_status();
}
