// Device code of stage 2 (register-resident variant) shared by the stand-alone
// kernel and the fused launch.
#pragma once
#include <type_traits>

#include "spin_common.h"

struct sel_plan {
  int P, nf_lo, first_hi, kprime, take;
};

// k' and the selection's length of a row of P partitions whose forced ones are [0, nf_lo) and [first_hi, P)
__device__ inline sel_plan plan_of(int P, int nf_lo, int first_hi, int topk, int includes_forced, int sel_stride) {
  sel_plan pl;
  if (first_hi <= nf_lo) { nf_lo = P; first_hi = P; }
  const int nforced = nf_lo + (P - first_hi);
  int kprime = includes_forced ? max(topk - nforced, 0) : topk;
  kprime = min(kprime, P - nforced);
  int take = nforced + kprime;
  if (take > sel_stride) {   // cannot happen for strides from spin_sel_stride(); keep stores in range
    kprime = max(sel_stride - nforced, 0);
    take = min(nforced + kprime, sel_stride);
  }
  pl.P = P; pl.nf_lo = nf_lo; pl.first_hi = first_hi; pl.kprime = kprime; pl.take = take;
  return pl;
}

// the same of a row of uniform partitions
__device__ inline sel_plan select_plan(int N, int PP, int tp, int topk, int includes_forced, int sink_pages,
                                       int recent_pages, int sel_stride) {
  int P = N > 0 ? (N + tp - 1) / tp : 0;
  if (P > PP) P = PP;
  const int pages = (N + 15) >> 4;
  int sink_end = min(sink_pages, pages);
  int recent_begin = max(pages - recent_pages, 0);
  if (sink_end >= recent_begin) { sink_end = pages; recent_begin = pages; }
  const int nf_lo = (N <= sink_end * 16) ? P : min((sink_end * 16) / tp, P);
  const int first_hi = min((recent_begin * 16 + tp - 1) / tp, P);
  return plan_of(P, nf_lo, first_hi, topk, includes_forced, sel_stride);
}

// ---------------------------------------------------------------------------
// Keys held in registers: KPT consecutive ones per thread, a bit mask says which of them count.
template <int KPT>
struct key_bits {
  typedef typename std::conditional<(KPT > 32), uint64_t, uint32_t>::type type;
};
__device__ inline int popc_bits(uint32_t m) { return __popc(m); }
__device__ inline int popc_bits(uint64_t m) { return __popcll(m); }
__device__ inline int ffs_bits(uint32_t m) { return __ffs(m); }
__device__ inline int ffs_bits(uint64_t m) { return __ffsll((unsigned long long)m); }
// bits k of 0 .. KPT-1 with c0 + k in [a, b)
template <int KPT>
__device__ inline typename key_bits<KPT>::type range_bits(int c0, int a, int b) {
  typedef typename key_bits<KPT>::type M;
  constexpr M all = KPT == (int)(8 * sizeof(M)) ? ~(M)0 : (((M)1 << (KPT & (int)(8 * sizeof(M) - 1))) - 1);
  const int lo = min(max(a - c0, 0), KPT), hi = min(max(b - c0, 0), KPT);
  const M from = lo >= KPT ? (M)0 : (all << lo) & all;
  const M upto = hi >= KPT ? all : ((M)1 << hi) - 1;
  return from & upto;
}

template <int BLOCK>
struct kth_lds {
  int hist[4][256];   // one histogram per digit: no buffer is cleared while others read it
  uint32_t wmax[BLOCK / 64], wmin[BLOCK / 64];
};

// Radix select over the workgroup's valid keys, most significant digit first: finds the threshold T and the
// number `need_eq` of keys equal to T such that the keys above T and the first need_eq keys equal to T are the
// k largest (lowest position first among equals), 1 <= k <= number of valid keys.  With slack > 0 the search
// stops as soon as the keys at or above the digits settled so far number at most k + slack, and those are all
// taken.  The digits start at the highest bit in which the keys differ at all (one min/max reduction): scores
// of one row usually share sign, exponent and leading mantissa bits, so this saves a pass or two and, above
// all, spreads the first histogram over many bins instead of piling every key onto one LDS counter.  Every
// wavefront scans the 256 bins for itself: one barrier per digit.  A workgroup barrier must lie between two
// uses of the same kth_lds.
template <int BLOCK, int KPT>
__device__ inline void block_kth(const uint32_t (&key)[KPT], typename key_bits<KPT>::type valid, int k, int slack,
                                 kth_lds<BLOCK> &s, uint32_t &T, unsigned &need_eq) {
  constexpr int NW = BLOCK / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = tid; i < 4 * 256; i += BLOCK) (&s.hist[0][0])[i] = 0;
  uint32_t kmx = 0u, kmn = 0xffffffffu;
#pragma unroll
  for (int j = 0; j < KPT; ++j)
    if ((valid >> j) & 1u) { kmx = max(kmx, key[j]); kmn = min(kmn, key[j]); }
  kmx = spin_wave_max_u32(kmx);
  kmn = spin_wave_min_u32(kmn);
  if (lane == 0) { s.wmax[wave] = kmx; s.wmin[wave] = kmn; }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) { kmx = max(kmx, s.wmax[w]); kmn = min(kmn, s.wmin[w]); }
  int hi = kmx == kmn ? 0 : 32 - __clz((int)(kmx ^ kmn));   // the low `hi` bits are the ones that vary
  uint32_t prefix = hi < 32 ? kmx >> hi : 0u;
  int remaining = k;
#pragma unroll
  for (int pass = 0; pass < 4; ++pass) {
    if (hi <= 0) break;                                  // block-uniform
    const int lo = max(hi - 8, 0), width = hi - lo;
    const uint32_t dmask = (1u << width) - 1u;
#pragma unroll
    for (int j = 0; j < KPT; ++j)
      if (((valid >> j) & 1u) && (pass == 0 || (key[j] >> hi) == prefix))
        atomicAdd(&s.hist[pass][(key[j] >> lo) & dmask], 1);
    __syncthreads();
    // suffix scan: lane handles digits 255-4*lane .. 252-4*lane, in descending order
    int hv[4], local = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) { hv[j] = s.hist[pass][255 - 4 * lane - j]; local += hv[j]; }
    int running = spin_wave_inclusive_scan(local) - local;
    int my_digit = -1, my_rem = 0, my_cnt = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (running < remaining && running + hv[j] >= remaining) {
        my_digit = 255 - 4 * lane - j;
        my_rem = remaining - running;
        my_cnt = hv[j];
      }
      running += hv[j];
    }
    const unsigned long long found = __ballot(my_digit >= 0);
    if (!found) break;                                   // fewer than k valid keys: not a call this function takes
    const int src = __ffsll((long long)found) - 1;
    const int digit = __builtin_amdgcn_readlane(my_digit, src), in_digit = __builtin_amdgcn_readlane(my_cnt, src);
    remaining = __builtin_amdgcn_readlane(my_rem, src);
    prefix = (prefix << width) | (uint32_t)digit;
    hi = lo;
    // every key that shares this prefix is wanted (or may be taken as well): the digits below cannot change
    // the outcome.  The threshold becomes the smallest key with the prefix, of which there may be several or
    // none: all are wanted, and the count of the prefix covers them.
    if (in_digit - remaining <= slack && hi > 0) {       // block-uniform
      prefix <<= hi;
      remaining = in_digit;
      break;
    }
  }
  T = prefix;
  need_eq = (unsigned)remaining;
}

// of `eq`, the bits that fall within the first `quota` in order
template <typename M>
__device__ inline M first_bits(M eq, unsigned quota) {
  M out = 0;
  while (eq && quota) {
    const M b = eq & (M)(~eq + 1);
    out |= b;
    eq ^= b;
    --quota;
  }
  return out;
}

// Turns every thread's `sure` bits (taken) and `eq` bits (taken while fewer than need_eq of them precede) into
// its final pick mask and the output position of its first pick (positions follow thread, then bit order).
template <int BLOCK, typename M>
__device__ inline M ordered_picks(M sure, M eq, unsigned need_eq, unsigned long long *s_wtot, int &pos) {
  constexpr int NW = BLOCK / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n_sure = popc_bits(sure), n_eq = popc_bits(eq);
  // the two counts never carry into one another: scanned separately, passed on in one word
  const uint32_t i_sure = (uint32_t)spin_wave_inclusive_scan(n_sure), i_eq = (uint32_t)spin_wave_inclusive_scan(n_eq);
  if (lane == 63) s_wtot[wave] = (unsigned long long)i_sure | ((unsigned long long)i_eq << 32);
  __syncthreads();
  unsigned sure_before = i_sure - n_sure, eq_before = i_eq - n_eq;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const unsigned long long t = s_wtot[w];
    if (w < wave) { sure_before += (uint32_t)t; eq_before += (uint32_t)(t >> 32); }
  }
  pos = (int)(sure_before + min(eq_before, need_eq));
  return sure | first_bits(eq, need_eq > eq_before ? need_eq - eq_before : 0u);
}

// The smallest score whose key is at least K (keys as in score_key).  Bit patterns that are no
// ordered number: below -inf every real key of the bin is at least key(-inf), so `low_end` asks
// for -inf there; above +inf no key exists and the NaN returned fails every comparison.
__device__ inline float key_floor_score(uint32_t K, bool low_end) {
  const uint32_t u = (K & 0x80000000u) ? (K ^ 0x80000000u) : ~K;
  if ((u & 0x7fffffffu) > 0x7f800000u) return (low_end && (u & 0x80000000u)) ? -__builtin_inff() : __builtin_nanf("");
  return __uint_as_float(u);
}
#define SPIN_KEY_MINUS_INF 0x007fffffu

// LDS of select_elements: the candidates that are left, in partition order
template <int BLOCK, int CAP>
struct elements_lds {
  kth_lds<BLOCK> kth;
  unsigned long long wtot[BLOCK / 64];
  uint32_t key[CAP > 0 ? CAP : 1];
  int32_t id[CAP > 0 ? CAP : 1];
};

// Picks the kprime best of the candidates a workgroup holds in registers (KPT scores per thread, bit k of `cand`:
// f[k] is a candidate; thread, then k is ascending partition order; id(k) names its partition) and stores their
// ids at rsel[first ..], ascending.  `bound`: a key that at least kprime of the candidates reach (0: none known).
// What the one compute unit of a row spends its time on is instructions per score (at 1024 threads one
// instruction on every thread's score takes the unit 6.7 ns), so a score is only compared as a float with the
// bound (key order is float order) and the few that pass form a list in LDS, on which the exact search runs with
// one to CAP / BLOCK keys per thread.  A row with more than CAP of them (every row where CAP is 0: few scores per
// thread, for which the list does not pay) searches its registers.
template <int BLOCK, int KPT, int CAP, typename ID>
__device__ inline void select_elements(const float (&f)[KPT], typename key_bits<KPT>::type cand, uint32_t bound,
                                       int kprime, int first, int sel_stride, int32_t *__restrict__ rsel,
                                       elements_lds<BLOCK, CAP> &s, ID id) {
  typedef typename key_bits<KPT>::type M;
  [[maybe_unused]] constexpr int NW = BLOCK / 64;
  [[maybe_unused]] const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  M valid = cand;
  if (bound > SPIN_KEY_MINUS_INF) {            // (at -inf NaN scores, which rank there, would fail the comparison)
    const float bf = key_floor_score(bound, true);
    M above = 0;
#pragma unroll
    for (int k = 0; k < KPT; ++k) above |= f[k] >= bf ? (M)1 << k : (M)0;
    valid &= above;
  }
  uint32_t T;
  unsigned need_eq;
  if constexpr (CAP > 0) {
    // ordered list of the candidates left
    const int mine = popc_bits(valid);
    const int inc = spin_wave_inclusive_scan(mine);
    if (lane == 63) s.wtot[wave] = (unsigned)inc;
    __syncthreads();
    int before = inc - mine, total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int t = (int)s.wtot[w];
      if (w < wave) before += t;
      total += t;
    }
    if (total <= CAP) {                          // block-uniform
      if (valid) {
        int pos = before;
#pragma unroll
        for (int k = 0; k < KPT; ++k)
          if ((valid >> k) & 1u) {
            s.key[pos] = score_key(f[k]);
            s.id[pos] = id(k);
            ++pos;
          }
      }
      __syncthreads();
      constexpr int LPT = CAP / BLOCK;           // list entries per thread
      auto pick_list = [&](auto entries) {
        constexpr int E = decltype(entries)::value;
        uint32_t key[E];
#pragma unroll
        for (int j = 0; j < E; ++j) key[j] = tid * E + j < total ? s.key[tid * E + j] : 0u;
        const uint32_t have = range_bits<E>(tid * E, 0, total);
        block_kth<BLOCK, E>(key, have, kprime, 0, s.kth, T, need_eq);
        uint32_t gt = 0, eq = 0;
#pragma unroll
        for (int j = 0; j < E; ++j) {
          gt |= key[j] > T ? 1u << j : 0u;
          eq |= key[j] == T ? 1u << j : 0u;
        }
        int pos;
        uint32_t pick = ordered_picks<BLOCK>(gt & have, eq & have, need_eq, s.wtot, pos);
        pos += first;
#pragma unroll
        for (int j = 0; j < E; ++j)
          if ((pick >> j) & 1u) {
            if (pos < sel_stride) rsel[pos] = s.id[tid * E + j];
            ++pos;
          }
      };
      if (total <= BLOCK) pick_list(std::integral_constant<int, 1>());
      else pick_list(std::integral_constant<int, LPT>());
      return;
    }
  }
  uint32_t key[KPT];
#pragma unroll
  for (int k = 0; k < KPT; ++k) key[k] = score_key(f[k]);
  block_kth<BLOCK, KPT>(key, valid, kprime, 0, s.kth, T, need_eq);
  M gt = 0, eq = 0;
#pragma unroll
  for (int k = 0; k < KPT; ++k) {
    gt |= key[k] > T ? (M)1 << k : (M)0;
    eq |= key[k] == T ? (M)1 << k : (M)0;
  }
  int pos;
  const M pick = ordered_picks<BLOCK>((M)(gt & valid), (M)(eq & valid), need_eq, s.wtot, pos);
  pos += first;
#pragma unroll
  for (int k = 0; k < KPT; ++k)
    if ((pick >> k) & 1u) {
      if (pos < sel_stride) rsel[pos] = id(k);
      ++pos;
    }
}

// forced partitions (a prefix and a suffix of the row) around the kprime candidates, and the padding
template <int BLOCK>
__device__ inline void emit_forced(const sel_plan &pl, int sel_stride, int32_t *__restrict__ rsel,
                                   int32_t *__restrict__ nsel, int row) {
  const int tid = threadIdx.x;
  for (int i = tid; i < min(pl.nf_lo, sel_stride); i += BLOCK) rsel[i] = i;
  const int at = pl.nf_lo + pl.kprime;
  for (int i = tid; i < pl.P - pl.first_hi && at + i < sel_stride; i += BLOCK) rsel[at + i] = pl.first_hi + i;
  for (int i = pl.take + tid; i < sel_stride; i += BLOCK) rsel[i] = -1;
  if (tid == 0) nsel[row] = pl.take;
}

// Register-resident variant for rows of at most BLOCK * KPT partitions: every
// thread keeps KPT consecutive scores in registers, so they are read once.
// With 16 or more of them per thread most are ruled out first: the k'-th largest of the threads' largest keys
// is a lower bound of the threshold (k' threads hold a key at least that large).
// Latency bounds this kernel: dependent loads, a barrier per digit, and the instructions per score on the row's
// one compute unit.  Stages 2+3, top 128, before (every score in every histogram) and after: 8 rows of 8192
// 14.7 -> 9.4 us, 8 rows of 16384 16.2 -> 11.5, 256 ragged rows of up to 16384 17.4 -> 13.4; rows of 62500 in the
// long-row kernel's multi-pass fall-back 69 -> 29.
// Returns the number of selected partitions.
template <int BLOCK, int KPT>
__device__ inline int select_reg_row(
    const float *__restrict__ scores, const int32_t *__restrict__ part_offsets,
    const int32_t *__restrict__ seq_lens, int Hkv, int tp, int topk, int includes_forced, int sink_pages,
    int recent_pages, int sel_stride, int32_t *__restrict__ sel, int32_t *__restrict__ nsel, int row,
    spin_var var) {
  typedef typename key_bits<KPT>::type M;
  constexpr int CAP = KPT >= 16 ? 2 * BLOCK : 0;
  __shared__ elements_lds<BLOCK, CAP> s;

  const int b = row / Hkv, h = row - b * Hkv;
  const int N = seq_lens[b];
  const int off_b = part_offsets[b];
  const int PP = part_offsets[b + 1] - off_b;
  const size_t vbase = (size_t)Hkv * off_b + (size_t)h * PP;
  const float *rs = scores + vbase;
  int32_t *rsel = sel + (size_t)row * sel_stride;
  const int c0 = threadIdx.x * KPT;   // this thread's partitions: c0 .. c0 + KPT - 1
  float f[KPT];
#pragma unroll
  for (int k4 = 0; k4 < KPT; k4 += 4) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (c0 + k4 < PP) v = *(const float4 *)(rs + c0 + k4);
    f[k4] = v.x; f[k4 + 1] = v.y; f[k4 + 2] = v.z; f[k4 + 3] = v.w;
  }

  // forced partitions: a prefix [0, nf_lo) and a suffix [first_hi, P)
  sel_plan pl;
  if (var.count) {
    int P = var.count[row];
    P = P < 0 ? 0 : (P > PP ? PP : P);
    const int pages = spin_var_row_pages(var, vbase, P);
    int sink_end = min(sink_pages, pages);
    int recent_begin = max(pages - recent_pages, 0);
    if (sink_end >= recent_begin) { sink_end = pages; recent_begin = pages; }
    pl = plan_of(P, spin_var_count_end_le(var, vbase, P, sink_end), spin_var_lower_bound_start(var, vbase, P, recent_begin),
                 topk, includes_forced, sel_stride);
  } else {
    pl = select_plan(N, PP, tp, topk, includes_forced, sink_pages, recent_pages, sel_stride);
  }
  if (pl.P > BLOCK * KPT) {           // the host picks a variant that fits; keep indexing in range
    pl.P = BLOCK * KPT;
    pl.nf_lo = min(pl.nf_lo, pl.P);
    pl.first_hi = max(min(pl.first_hi, pl.P), pl.nf_lo);
    pl.kprime = min(pl.kprime, pl.first_hi - pl.nf_lo);
    pl.take = min(pl.nf_lo + pl.kprime + pl.P - pl.first_hi, sel_stride);
  }
  emit_forced<BLOCK>(pl, sel_stride, rsel, nsel, row);   // under way while the scores are still coming
  if (pl.kprime > 0) {
    const M cand = range_bits<KPT>(c0, pl.nf_lo, pl.first_hi);
    uint32_t bound = 0;
    if (KPT >= 16) {
      const int holders = (pl.first_hi - 1) / KPT - pl.nf_lo / KPT + 1;   // threads that hold a candidate
      if (holders >= pl.kprime + (pl.kprime >> 1)) {                      // block-uniform
        float mx = -__builtin_inff();                                     // NaN scores rank as -inf: dropped
#pragma unroll
        for (int k = 0; k < KPT; ++k) mx = fmaxf(mx, ((cand >> k) & 1u) ? f[k] : mx);
        const uint32_t top[1] = {score_key(mx)};
        unsigned at_bound;
        block_kth<BLOCK, 1>(top, cand ? 1u : 0u, pl.kprime, pl.kprime >> 2, s.kth, bound, at_bound);
      }
    }
    select_elements<BLOCK, KPT, CAP>(f, cand, bound, pl.kprime, pl.nf_lo, sel_stride, rsel, s,
                                     [&](int k) { return c0 + k; });
  }
  return pl.take;
}
