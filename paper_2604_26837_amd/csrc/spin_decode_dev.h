// Device code of stage 4 shared by the attention kernels and by the launch that attends a row's
// always-attended pages beside stages 2+3: page loads, the logit / softmax / P V step of one
// 16-token tile on the matrix cores, and the merge of wavefront and workgroup partials.
#pragma once
#include "spin_common.h"

#define NEG_INF (-__builtin_inff())

struct page_regs {
  uint4 k[4], v[4];
};

// The tiles of a page.  Only what its attended tokens need is fetched: in the K tile a lane holds 16 bytes of ONE token,
// in the V tile 16 bytes of ONE token quad, so lanes of unattended tokens / quads (all of them for an empty mask) are
// sent beyond the slot and hold zeros (their logits are masked and their probabilities are exactly zero, so the
// result has the same bits as with the whole page loaded).  `slot` and `mask` are uniform.
__device__ __forceinline__ void load_k_tile(page_regs &r, const uint4 *__restrict__ pool, int slot, int lane, unsigned mask) {
  const __amdgpu_buffer_rsrc_t buf = spin_buffer(pool + (size_t)slot * SPIN_SLOT_U4, SPIN_SLOT_U4 * 16);
  const uint32_t at = ((mask >> (lane & 15)) & 1u) ? (uint32_t)lane * 16 : SPIN_SLOT_U4 * 16;
#pragma unroll
  for (int j = 0; j < 4; ++j) r.k[j] = spin_buffer_load(buf, at, j * 1024);
}
__device__ __forceinline__ void load_v_tile(page_regs &r, const uint4 *__restrict__ pool, int slot, int lane, unsigned mask) {
  const __amdgpu_buffer_rsrc_t buf = spin_buffer(pool + (size_t)slot * SPIN_SLOT_U4, SPIN_SLOT_U4 * 16);
  const uint32_t at = ((mask >> (4 * (lane >> 4))) & 0xfu) ? (uint32_t)lane * 16 : SPIN_SLOT_U4 * 16;
#pragma unroll
  for (int j = 0; j < 4; ++j) r.v[j] = spin_buffer_load(buf, at, SPIN_KTILE_U4 * 16 + j * 1024);
}

struct softmax_state {
  float m, l;
  spin_f32x4 acc[8];
};

// S[token 4c+i][head n] of a tile of 16 tokens
__device__ __forceinline__ spin_f32x4 tile_logits(const page_regs &r, const spin_bf16x8 (&qf)[4]) {
  spin_f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < 4; ++j)
    s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(spin_bf16x8, r.k[j]), qf[j], s, 0, 0, 0);
  return s;
}

// the online softmax over a tile's logits, and its share of P V
__device__ __forceinline__ void tile_attend(softmax_state &st, const spin_f32x4 &s, const page_regs &r, unsigned mask, int c,
                                            float scale_log2e) {
  const unsigned mbits = (mask >> (4 * c)) & 0xFu;
  float sv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) sv[i] = ((mbits >> i) & 1u) ? s[i] * scale_log2e : NEG_INF;
  float pm = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
  pm = fmaxf(pm, __shfl_xor(pm, 16));
  pm = fmaxf(pm, __shfl_xor(pm, 32));
  const float m_new = fmaxf(st.m, pm);
  const float m_safe = (m_new == NEG_INF) ? 0.f : m_new;
  const float alpha = __builtin_amdgcn_exp2f(st.m - m_safe);
  float pr[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) pr[i] = __builtin_amdgcn_exp2f(sv[i] - m_safe);
  st.l = st.l * alpha + ((pr[0] + pr[1]) + (pr[2] + pr[3]));
  st.m = m_new;

  // rescale the accumulator rows (head 4c+i) by that head's alpha, only when some maximum moved
  if (__any(alpha != 1.0f)) {
    float ar[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) ar[i] = __shfl(alpha, 4 * c + i);
#pragma unroll
    for (int jn = 0; jn < 8; ++jn)
#pragma unroll
      for (int i = 0; i < 4; ++i) st.acc[jn][i] *= ar[i];
  }

  // P as the A operand: row n = head, k = tokens 4c..4c+3
  spin_bf16x2 p01 = {(__bf16)pr[0], (__bf16)pr[1]};
  spin_bf16x2 p23 = {(__bf16)pr[2], (__bf16)pr[3]};
  uint2 pk = {__builtin_bit_cast(uint32_t, p01), __builtin_bit_cast(uint32_t, p23)};
  const spin_s16x4 pa = __builtin_bit_cast(spin_s16x4, pk);
#pragma unroll
  for (int jv = 0; jv < 4; ++jv) {
    uint2 lo = {r.v[jv].x, r.v[jv].y}, hi = {r.v[jv].z, r.v[jv].w};
    st.acc[2 * jv] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pa, __builtin_bit_cast(spin_s16x4, lo),
                                                               st.acc[2 * jv], 0, 0, 0);
    st.acc[2 * jv + 1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pa, __builtin_bit_cast(spin_s16x4, hi),
                                                                   st.acc[2 * jv + 1], 0, 0, 0);
  }
}

// Attends `cnt` (<= 64) pages whose slot and mask are held one per lane (lane i: the i-th page; a slot inside the pool
// in every lane), in lane order from page `from` on, through a ring of DEPTH register buffers.  A tile's registers are
// loaded again as soon as it has been consumed, and what lies past the end is loaded as an empty page, so that the loop
// is straight-line code that waits for exactly the tile it is about to read (see spin_buffer).  `asked` runs once the
// first DEPTH pages have been asked for.
template <int DEPTH, typename ASKED>
__device__ __forceinline__ void attend_lane_pages(softmax_state &st, const uint4 *__restrict__ pool, int myslot,
                                                  unsigned mymask, int from, int cnt, int lane, int c,
                                                  const spin_bf16x8 (&qf)[4], float scale_log2e, ASKED asked) {
  page_regs r[DEPTH];
  auto slot_of = [&](int i) { return __builtin_amdgcn_readlane(myslot, i < cnt ? i : 0); };
  auto mask_of = [&](int i) { return (unsigned)__builtin_amdgcn_readlane((int)mymask, i & 63) & (i < cnt ? 0xffffu : 0u); };
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) {
    load_k_tile(r[d], pool, slot_of(from + d), lane, mask_of(from + d));
    __builtin_amdgcn_sched_barrier(0);   // asked for in the order in which the loop asks again
    load_v_tile(r[d], pool, slot_of(from + d), lane, mask_of(from + d));
    __builtin_amdgcn_sched_barrier(0);
  }
  asked();
  int i = from;
  for (; i + DEPTH <= cnt; i += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      const int ahead = i + d + DEPTH;
      const spin_f32x4 s = tile_logits(r[d], qf);
      load_k_tile(r[d], pool, slot_of(ahead), lane, mask_of(ahead));
      tile_attend(st, s, r[d], mask_of(i + d), c, scale_log2e);
      load_v_tile(r[d], pool, slot_of(ahead), lane, mask_of(ahead));
    }
  }
#pragma unroll
  for (int d = 0; d < DEPTH - 1; ++d)
    if (i + d < cnt) tile_attend(st, tile_logits(r[d], qf), r[d], mask_of(i + d), c, scale_log2e);
}

template <int DEPTH>
__device__ __forceinline__ void attend_lane_pages(softmax_state &st, const uint4 *__restrict__ pool, int myslot,
                                                  unsigned mymask, int cnt, int lane, int c,
                                                  const spin_bf16x8 (&qf)[4], float scale_log2e) {
  attend_lane_pages<DEPTH>(st, pool, myslot, mymask, 0, cnt, lane, c, qf, scale_log2e, [] {});
}

// the group's queries as the second matrix operand of the logit tile: column n = head, k = channels 32j+8c..+8
__device__ __forceinline__ void load_queries(spin_bf16x8 (&qf)[4], const uint16_t *__restrict__ q, int b, int h, int G,
                                             int Hq, int n, int c) {
  const uint4 *qrow = (const uint4 *)(q + ((size_t)(b * Hq + h * G + (n < G ? n : 0))) * SPIN_HEAD_DIM);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint4 v = qrow[j * 4 + c];
    if (n >= G) v = make_uint4(0, 0, 0, 0);
    qf[j] = __builtin_bit_cast(spin_bf16x8, v);
  }
}

__device__ inline void softmax_reset(softmax_state &st) {
  st.m = NEG_INF;
  st.l = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) st.acc[i] = (spin_f32x4){0.f, 0.f, 0.f, 0.f};
}

// channels d and d + 1 (d even) of a query head
__device__ inline void write_out(uint16_t *__restrict__ out, float *__restrict__ lse, int qhead, int d, float M,
                                 float L, float2 O) {
  const spin_bf16x2 r = {(__bf16)(L > 0.f ? O.x / L : 0.f), (__bf16)(L > 0.f ? O.y / L : 0.f)};
  uint16_t *o = out + (size_t)qhead * SPIN_HEAD_DIM + d;
  const uint32_t w = __builtin_bit_cast(uint32_t, r);
  o[0] = (uint16_t)w;                         // (the output need not be aligned to more than its elements)
  o[1] = (uint16_t)(w >> 16);
  if (lse && d == 0) lse[qhead] = L > 0.f ? (M + __builtin_amdgcn_logf(L)) * 0.6931471805599453f : NEG_INF;
}

// After a workgroup's wavefronts have consumed their tiles: merge the wavefront partials through
// LDS and, with several splits, the workgroup partials through the workspace (see the header).
// Partial `s` of a row lives at index row * pstride + s (pstride = splits + the partials earlier launches may leave); the
// row's output is the merge, in index order, of the partials 0 .. nsplit-1 of the calling launch.
// ONLY_PARTIAL (then `split` is the index j of the calling workgroup among those that attend a row's
// always-attended pages): the workgroup only stores its partial, at index nsplit + j, for a later
// launch on the same stream to start from.
// to_partial: the merged result of the row is stored there as well, unnormalised, instead of being
// written to `out` (the first of two attention passes over one page list).
// LANE_ROWS: a lane's accumulators of channel block jn are of channel 8n + jn, not 16 jn + n.
// Returns true in the workgroup that wrote the row's output.
template <int WAVES, bool ONLY_PARTIAL = false, bool LANE_ROWS = false>
__device__ __forceinline__ bool decode_finish(softmax_state &st, int row, int split, int b, int h, int lane, int wave,
                                              int n, int c, int G, int Hq, int nsplit, int pstride,
                                              float *part_ml, float *part_acc, int32_t *tickets,
                                              uint16_t *__restrict__ out, float *__restrict__ lse,
                                              bool to_partial = false) {
  extern __shared__ __align__(16) float smem[];
  float *s_acc = smem;                                  // [WAVES][G][128]
  float *s_m = smem + WAVES * G * SPIN_HEAD_DIM;        // [WAVES][G]
  float *s_l = s_m + WAVES * G;                         // [WAVES][G]
  __shared__ int s_last;
  // denominators: sum the four token-quad lanes of each head
  float l = st.l;
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);

  // wavefront partials -> LDS
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int head = 4 * c + i;
    if (head < G) {
#pragma unroll
      for (int jn = 0; jn < 8; ++jn)
        s_acc[(wave * G + head) * SPIN_HEAD_DIM + (LANE_ROWS ? 8 * n + jn : 16 * jn + n)] = st.acc[jn][i];
    }
  }
  if (c == 0 && n < G) {
    s_m[wave * G + n] = st.m;
    s_l[wave * G + n] = l;
  }
  __syncthreads();

  // the wavefronts' partials merged: a wavefront has one head g at a time, a lane two channels d, d + 1
  for (int idx = threadIdx.x; idx < G * (SPIN_HEAD_DIM / 2); idx += WAVES * 64) {
    const int g = __builtin_amdgcn_readfirstlane(idx >> 6), d = (idx & 63) * 2;
    float M = NEG_INF, m[WAVES], l_of[WAVES];
    float2 a[WAVES];
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      m[w] = s_m[w * G + g];
      l_of[w] = s_l[w * G + g];
      a[w] = *(const float2 *)(s_acc + (w * G + g) * SPIN_HEAD_DIM + d);
    }
#pragma unroll
    for (int w = 0; w < WAVES; ++w) M = fmaxf(M, m[w]);
    const float Ms = (M == NEG_INF) ? 0.f : M;
    float L = 0.f;
    float2 O = make_float2(0.f, 0.f);
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const float wgt = __builtin_amdgcn_exp2f(m[w] - Ms);
      L += l_of[w] * wgt;
      O.x += a[w].x * wgt;
      O.y += a[w].y * wgt;
    }
    if (ONLY_PARTIAL || (nsplit == 1 && to_partial)) {
      // read by a later launch on the same stream: plain stores
      const size_t pi = ((size_t)row * pstride + nsplit + (ONLY_PARTIAL ? split : 0)) * G + g;
      *(float2 *)(part_acc + pi * SPIN_HEAD_DIM + d) = O;
      if (d == 0) *(float2 *)(part_ml + pi * 2) = make_float2(M, L);
    } else if (nsplit == 1) {
      write_out(out, lse, b * Hq + h * G + g, d, M, L, O);
    } else {
      // device-scope stores: written through to where every compute die sees them
      const size_t pi = ((size_t)row * pstride + split) * G + g;
      spin_dev_store2(part_acc + pi * SPIN_HEAD_DIM + d, O);
      if (d == 0) spin_dev_store2(part_ml + pi * 2, make_float2(M, L));
    }
  }
  if (ONLY_PARTIAL) return false;
  if (nsplit == 1) return true;

  // Ticket: the last workgroup of the row to arrive merges all splits in split
  // order.  Partials travel through device-scope atomic stores and loads (no
  // cache-wide write-back or invalidate); each thread waits for its own stores
  // to be acknowledged, the barrier orders them before thread 0's ticket.
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __syncthreads();
  if (threadIdx.x == 0)
    s_last = (__hip_atomic_fetch_add(&tickets[row], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nsplit - 1);
  __syncthreads();
  if (!s_last) return false;
  // A chain of dependent steps on one compute unit ends every row, so this is written for latency: nothing passes
  // through LDS, and no load waits for another.  With up to CH splits a lane asks for all its accumulators and all
  // (m, l) pairs (the same ones in a whole wavefront) at once.  From the ticket to the output: 2 splits 1.8 -> 1.3 us,
  // 8 splits 2.6 -> 1.8, against one channel per lane, four rounds of predicated loads and the pairs staged in LDS
  // behind a barrier.  With more, lane s asks for the pair of split s (there are at most 64) beside the first 2 * CH
  // accumulators, and the next ones are under way while the ones before are summed.  Stage 4, against a loop over the
  // pairs ahead of rounds of eight and against the pairs staged in LDS: 2 rows of 580 pages, 18 splits 15.3 / 14.1 ->
  // 11.9 us; 8 rows of 1036 pages, 32 splits 23.7 / 20.9 -> 18.3; 24 rows of 64 pages, 16 splits 16.5 / 15.9 -> 13.6;
  // 8 rows of 384 pages, groups of 16, 12 splits 20.2 / 21.0 -> 13.8; 2 rows of 65536 tokens, 64 splits 22.6 / 15.7 -> 13.2.
  const size_t pbase = (size_t)row * pstride * G;
  constexpr int CH = 8;
  for (int idx = threadIdx.x; idx < G * (SPIN_HEAD_DIM / 2); idx += WAVES * 64) {
    const int g = __builtin_amdgcn_readfirstlane(idx >> 6), d = (idx & 63) * 2;
    const float *acc_at = part_acc + (pbase + g) * SPIN_HEAD_DIM + d, *ml_at = part_ml + (pbase + g) * 2;
    float M = NEG_INF, L = 0.f;
    float2 O = make_float2(0.f, 0.f);
    auto load = [&](float2 (&a)[CH], int s0) {
#pragma unroll
      for (int s = 0; s < CH; ++s) {
        if (s0 + s >= nsplit) break;                     // uniform
        a[s] = spin_dev_load2(acc_at + (unsigned)((s0 + s) * G * SPIN_HEAD_DIM));
      }
    };
    auto add = [&](float wgt, float l_of, const float2 &a) {
      L += l_of * wgt;
      O.x += a.x * wgt;
      O.y += a.y * wgt;
    };
    if (nsplit <= CH) {
      float2 a[CH], ml[CH];
#pragma unroll
      for (int s = 0; s < CH; ++s) {
        if (s >= nsplit) break;
        ml[s] = spin_dev_load2(ml_at + (unsigned)(s * G * 2));
        a[s] = spin_dev_load2(acc_at + (unsigned)(s * G * SPIN_HEAD_DIM));
      }
#pragma unroll
      for (int s = 0; s < CH; ++s)
        if (s < nsplit) M = fmaxf(M, ml[s].x);
      const float Ms = (M == NEG_INF) ? 0.f : M;
#pragma unroll
      for (int s = 0; s < CH; ++s) {                     // the splits in split order
        if (s >= nsplit) break;
        add(__builtin_amdgcn_exp2f(ml[s].x - Ms), ml[s].y, a[s]);
      }
    } else {
      float2 ml = make_float2(NEG_INF, 0.f), a[2][CH];
      if (lane < nsplit) ml = spin_dev_load2(ml_at + (unsigned)(lane * G * 2));
      load(a[0], 0);
      load(a[1], CH);
      M = fmaxf(spin_wave_max(ml.x), NEG_INF);
      const float wgt = __builtin_amdgcn_exp2f(ml.x - (M == NEG_INF ? 0.f : M));
      auto add_all = [&](float2 (&a_of)[CH], int s0) {
#pragma unroll
        for (int s = 0; s < CH; ++s) {
          if (s0 + s >= nsplit) break;
          add(spin_readlane(wgt, s0 + s), spin_readlane(ml.y, s0 + s), a_of[s]);
        }
      };
      for (int s0 = 0; s0 < nsplit; s0 += 2 * CH) {
        add_all(a[0], s0);
        load(a[0], s0 + 2 * CH);
        add_all(a[1], s0 + CH);
        load(a[1], s0 + 3 * CH);
      }
    }
    if (to_partial) {
      const size_t pi = ((size_t)row * pstride + nsplit) * G + g;
      *(float2 *)(part_acc + pi * SPIN_HEAD_DIM + d) = O;
      if (d == 0) *(float2 *)(part_ml + pi * 2) = make_float2(M, L);
    } else {
      write_out(out, lse, b * Hq + h * G + g, d, M, L, O);
    }
  }
  if (threadIdx.x == 0)   // ready for the next launch
    __hip_atomic_store(&tickets[row], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

#define SPIN_DECODE_FROM_PARTIAL 1   // the row's first wavefront starts from the partial at index nsplit
#define SPIN_DECODE_TO_PARTIAL 2     // the row's merged result goes there instead of to `out`
#define SPIN_DECODE_LISTED 4         // rows without a page in the list are left alone

// The part of a row's pages that workgroup `split` of it attends (the kernel's arguments, see the header of stage 4).
// only(position, mask): what of the page at that position of the list is attended.
template <int WAVES, int DEPTH, typename ONLY>
__device__ __forceinline__ void decode_row(
    int row, int split, const uint16_t *__restrict__ q, const uint4 *__restrict__ pool, int64_t pool_slots,
    const int32_t *__restrict__ slots, const uint16_t *__restrict__ masks,
    const int32_t *__restrict__ npages, int page_stride, int G, int Hq, int Hkv, int nsplit, int pstride,
    const int32_t *__restrict__ skip, int mode, int nside, float scale_log2e, float *part_ml, float *part_acc, int32_t *tickets,
    uint16_t *__restrict__ out, float *__restrict__ lse, int32_t *status, ONLY only) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform, and so are its page count and its loops
  const int n = lane & 15;   // column: query head of the group (logits), channel-in-block (output)
  const int c = lane >> 4;   // token quad (logits) / head quad (output)
  const int b = row / Hkv;
  const int h = row - b * Hkv;

  // Pages are dealt round-robin: page p belongs to split p % nsplit and, inside
  // it, to wavefront (p / nsplit) % WAVES.  The addresses of this wavefront's
  // slot entries therefore do not depend on the row's page count, and their
  // load is issued together with it.
  const int32_t *rslots = slots + (size_t)row * page_stride;
  const uint16_t *rmask = masks + (size_t)row * page_stride;
  // A list of missed pages is short more often than not: it is dealt to a split's wavefronts before the next split's, and
  // the splits without a page end, so that one of at most WAVES pages is attended by one workgroup, which has nothing to
  // merge.  (Dealt as a whole row is, 5 missed pages of 8 rows: both launches 15.0 -> 12.9 us, of
  // 64 rows 21.6 -> 19.7, 50 of 24 rows 17.5 -> 15.6.)
  const bool listed = (mode & SPIN_DECODE_LISTED) != 0;
  const int first = listed ? split * WAVES + wave : wave * nsplit + split, stride = WAVES * nsplit;
  int np = npages[row];
  np = np < 0 ? 0 : (np > page_stride ? page_stride : np);
  if (listed && np <= split * WAVES) return;
  const int parts = listed ? min((np + WAVES - 1) / WAVES, nsplit) : nsplit;
  // list positions [0, skip_lo) and [np - skip_hi, np) were attended by an earlier launch (the row's
  // always-attended pages): they keep their place in the dealing but are not fetched or attended here
  const int32_t *skip_at = skip ? skip + 2 * row : npages + row;   // read either way, in one round trip with the count
  const int skip_0 = skip_at[0], skip_1 = skip_at[skip ? 1 : 0];
  const int skip_lo = skip ? skip_0 : 0, skip_hi = skip ? skip_1 : 0;
  const int keep_end = np - (skip_hi > 0 ? skip_hi : 0);

  // this wavefront's pages: first + i * stride, i < nw; the entries of the first 64 are asked for ahead of all else
  int p = first + lane * stride;
  int next_slot = rslots[min(p, page_stride - 1)];
  unsigned next_mask = rmask[min(p, page_stride - 1)];

  spin_bf16x8 qf[4];
  load_queries(qf, q, b, h, G, Hq, n, c);
  softmax_state st;
  softmax_reset(st);

  // The first wavefront of split s < nside starts from the s-th partial (m, l, O) an earlier launch left for
  // the row (its always-attended pages, or the first of two passes over the page list) instead of from the
  // empty state: that partial then is part of the ordinary merge.
  if ((mode & SPIN_DECODE_FROM_PARTIAL) && split < nside && wave == 0) {
    const size_t pf = ((size_t)row * pstride + nsplit + split) * G;
    if (n < G) {
      st.m = part_ml[(pf + n) * 2];
      if (c == 0) st.l = part_ml[(pf + n) * 2 + 1];   // the lanes' denominators are summed over c at the end
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * c + i < G) {
#pragma unroll
        for (int jn = 0; jn < 8; ++jn) st.acc[jn][i] = part_acc[(pf + 4 * c + i) * SPIN_HEAD_DIM + 16 * jn + n];
      }
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): waited for here, or every page's turn would wait as if they were under way
  }

  const int nw = np > first ? (np - first + stride - 1) / stride : 0;
  for (int base = 0; base == 0 || base < nw; base += 64) {
    const int cnt = min(nw - base, 64);
    int myslot = 0;
    unsigned mymask = 0;
    if (lane < cnt && p >= skip_lo && p < keep_end) {   // the others are attended elsewhere, or past the end of the list
      if (next_slot < 0 || (int64_t)next_slot >= pool_slots) {
        spin_raise(status, SPIN_ERR_SLOT_RANGE);        // attends to none of it
      } else {
        myslot = next_slot;
        mymask = only(p, next_mask);
      }
    }
    p += 64 * stride;
    if (base + 64 < nw) {
      next_slot = rslots[min(p, page_stride - 1)];
      next_mask = rmask[min(p, page_stride - 1)];
    }
    attend_lane_pages<DEPTH>(st, pool, myslot, mymask, cnt, lane, c, qf, scale_log2e);
  }

  decode_finish<WAVES>(st, row, split, b, h, lane, wave, n, c, G, Hq, parts, pstride, part_ml, part_acc, tickets, out,
                       lse, (mode & SPIN_DECODE_TO_PARTIAL) != 0);
}

int decode_launch(spin_ctx *ctx, int32_t batch, const void *q, const void *kv_pool, int64_t pool_slots,
                  const int32_t *slots, const uint16_t *valid_mask, const int32_t *npages, void *out, float *lse,
                  float *part_ml, float *part_acc, int32_t *tickets, int32_t *status, const int32_t *skip, int mode,
                  int nside, void *stream);
