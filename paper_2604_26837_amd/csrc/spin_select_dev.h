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

// Where a row's selection goes: to global memory, or (HELD: the same launch resolves the row) to LDS only, from where
// the caller stores it.
template <bool HELD>
struct sel_row {
  int32_t *__restrict__ out;
  int stride;
  spin_lds_i32 *lds;
  __device__ __forceinline__ void put(int pos, int32_t id) const {
    if (pos < stride) {
      if (HELD) lds[pos] = id;
      else out[pos] = id;
    }
  }
  __device__ __forceinline__ void pad(int pos) const { out[pos] = -1; }
  __device__ __forceinline__ void count(int32_t *__restrict__ nsel, int row, int take) const { nsel[row] = take; }
};

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

// The digit in whose bin the element of rank `rank` (1: the largest) falls, from the 256 bins of a histogram, with
// the rank inside that bin and its count; -1 where the bins hold fewer.  Every wavefront computes it for itself.
// Lane handles digits 255-4*lane .. 252-4*lane, in descending order.
__device__ inline int digit_of_rank(const int *hist, int &rank, int &in_digit) {
  const int lane = threadIdx.x & 63;
  const int4 bins = *(const int4 *)(hist + 252 - 4 * lane);
  const int hv[4] = {bins.w, bins.z, bins.y, bins.x};
  const int local = (hv[0] + hv[1]) + (hv[2] + hv[3]);
  int running = spin_wave_inclusive_scan(local) - local;
  int my_digit = -1, my_rem = 0, my_cnt = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (running < rank && running + hv[j] >= rank) {
      my_digit = 255 - 4 * lane - j;
      my_rem = rank - running;
      my_cnt = hv[j];
    }
    running += hv[j];
  }
  const unsigned long long found = __ballot(my_digit >= 0);
  if (!found) return -1;
  const int src = __ffsll((long long)found) - 1;
  rank = __builtin_amdgcn_readlane(my_rem, src);
  in_digit = __builtin_amdgcn_readlane(my_cnt, src);
  return __builtin_amdgcn_readlane(my_digit, src);
}

template <int BLOCK>
struct kth_lds {
  alignas(16) int hist[4][256];   // one histogram per digit: no buffer is cleared while others read it
  uint32_t wmax[BLOCK / 64], wmin[BLOCK / 64];
  alignas(16) int4 found[4];
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
// MANY and `many` (a row's scores, 16 per thread): those of a bell-shaped row still share a dozen first digits, so a
// thread counts its keys of the eight largest in a register, and the others only where the k-th is among them.  Stage 2
// of 8 rows of 16384 normal scores, k 2048 / 8192: 14.3 / 16.0 us, with one LDS addition per score 22.7 / 24.1; of scores
// spread over many digits the detour costs up to 2.5 us (almost all close together, k 8192: 37.8 -> 40.2), and with few
// keys the additions are the shorter way (256 ragged rows, below 4096 of them: step 142.6 us against 144.9).
template <int BLOCK, int KPT, bool MANY = false>
__device__ __forceinline__ void block_kth(const uint32_t (&key)[KPT], typename key_bits<KPT>::type valid, int k, int slack,
                                 kth_lds<BLOCK> &s, uint32_t &T, unsigned &need_eq, bool many = false) {
  constexpr int NW = BLOCK / 64;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  for (int i = tid; i < 4 * 256; i += BLOCK) (&s.hist[0][0])[i] = 0;
  uint32_t kmx = 0u, kmn = 0xffffffffu;
#pragma unroll
  for (int j = 0; j < KPT; ++j)
    if ((valid >> j) & 1u) { kmx = max(kmx, key[j]); kmn = min(kmn, key[j]); }
  kmx = spin_wave_max_u32(kmx);
  kmn = spin_wave_min_u32(kmn);
  if (lane == 0) { s.wmax[wave] = kmx; s.wmin[wave] = kmn; }
  __syncthreads();
  kmx = spin_wave_max_u32(s.wmax[lane % NW]);
  kmn = spin_wave_min_u32(s.wmin[lane % NW]);
  int hi = kmx == kmn ? 0 : 32 - __clz((int)(kmx ^ kmn));   // the low `hi` bits are the ones that vary
  uint32_t prefix = hi < 32 ? kmx >> hi : 0u;
  int remaining = k;
#pragma unroll
  for (int pass = 0; pass < 4; ++pass) {
    if (hi <= 0) break;                                  // block-uniform
    const int lo = max(hi - 8, 0), width = hi - lo;
    const uint32_t dmask = (1u << width) - 1u;
    [[maybe_unused]] const bool ahead = MANY && pass == 0 && many;   // block-uniform
    [[maybe_unused]] const uint32_t top = (kmx >> lo) & dmask;       // in the first pass the largest digit there is
    if (MANY && ahead) {
      unsigned long long acc = 0;                          // byte o: keys whose digit is top - o
#pragma unroll
      for (int j = 0; j < KPT; ++j) {
        const uint32_t o = top - ((key[j] >> lo) & dmask);
        if (((valid >> j) & 1u) && o < 8u) acc += 1ull << (8u * o);
      }
      // 16 bits each, of which a wavefront's sum needs 12
      static_assert(!MANY || KPT <= 255, "a thread's count fits a byte, a wavefront's 16 bits");
      uint32_t part[4] = {(uint32_t)acc & 0x00ff00ffu, (uint32_t)(acc >> 8) & 0x00ff00ffu,
                          (uint32_t)(acc >> 32) & 0x00ff00ffu, (uint32_t)(acc >> 40) & 0x00ff00ffu};
#pragma unroll
      for (int i = 0; i < 4; ++i) part[i] = (uint32_t)spin_wave_inclusive_scan((int)part[i]);   // lane 63: the sums
      if (lane == 63) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {                      // part i: digits 4 (i / 2) + i % 2 and two further below
          const uint32_t o = 4u * (i >> 1) + (i & 1);
          if (part[i] & 0xffffu) atomicAdd(&s.hist[0][top - o], (int)(part[i] & 0xffffu));
          if (part[i] >> 16) atomicAdd(&s.hist[0][top - o - 2], (int)(part[i] >> 16));
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < KPT; ++j)
        if (((valid >> j) & 1u) && (pass == 0 || (key[j] >> hi) == prefix))
          atomicAdd(&s.hist[pass][(key[j] >> lo) & dmask], 1);
    }
    __syncthreads();
    int in_digit = 0, digit;
    if (BLOCK >= 1024) {
      if (wave == 0) {
        digit = digit_of_rank(s.hist[pass], remaining, in_digit);
        if (lane == 0) s.found[pass] = make_int4(digit, remaining, in_digit, 0);
      }
      __syncthreads();
      const int4 f = s.found[pass];
      digit = __builtin_amdgcn_readfirstlane(f.x);
      remaining = __builtin_amdgcn_readfirstlane(f.y);
      in_digit = __builtin_amdgcn_readfirstlane(f.z);
    } else {
      digit = digit_of_rank(s.hist[pass], remaining, in_digit);
    }
    if constexpr (MANY) {
      if (ahead && digit < 0) {                            // below the eight
        __syncthreads();                                   // (every wavefront has read the bins)
#pragma unroll
        for (int j = 0; j < KPT; ++j) {
          const uint32_t dg = (key[j] >> lo) & dmask;
          if (((valid >> j) & 1u) && top - dg >= 8u) atomicAdd(&s.hist[0][dg], 1);
        }
        __syncthreads();
        digit = digit_of_rank(s.hist[0], remaining, in_digit);
      }
    }
    if (digit < 0) break;                                // fewer than k valid keys: not a call this function takes
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
// its final pick mask and the output position of its first pick (positions follow thread, then bit order); `picked`:
// all threads' picks, `eq_picked`: those of equal keys.
template <int BLOCK, typename M>
__device__ inline M ordered_picks(M sure, M eq, unsigned need_eq, uint2 *s_wtot, int &pos, int &picked, int &eq_picked) {
  constexpr int NW = BLOCK / 64;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_sure = popc_bits(sure), n_eq = popc_bits(eq);
  const int i_sure = spin_wave_inclusive_scan(n_sure), i_eq = spin_wave_inclusive_scan(n_eq);
  if (lane == 63) s_wtot[wave] = make_uint2((uint32_t)i_sure, (uint32_t)i_eq);
  __syncthreads();
  const uint2 t = s_wtot[lane % NW];
  int all_sure, all_eq;
  const unsigned sure_before = (unsigned)(spin_waves_before<NW>((int)t.x, wave, all_sure) + i_sure - n_sure);
  const unsigned eq_before = (unsigned)(spin_waves_before<NW>((int)t.y, wave, all_eq) + i_eq - n_eq);
  eq_picked = (int)min((unsigned)all_eq, need_eq);
  picked = all_sure + eq_picked;
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

// the candidates that are left, in partition order
template <int BLOCK, int CAP>
struct elements_lds {
  kth_lds<BLOCK> kth;
  uint2 wtot[BLOCK / 64];
  uint32_t key[CAP];
  int32_t id[CAP];
};

// The kprime best of the `total` entries of an ordered list in LDS, stored ascending at rsel[first ..].
template <int BLOCK, int CAP, typename ROW>
__device__ __forceinline__ void pick_from_list(int total, int kprime, int first, const ROW &rsel,
                                      elements_lds<BLOCK, CAP> &s) {
  const int tid = threadIdx.x;
  auto pick_list = [&](auto entries) {
    constexpr int E = decltype(entries)::value;  // list entries per thread
    uint32_t T;
    unsigned need_eq;
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
    int pos, picked, eq_picked;
    uint32_t pick = ordered_picks<BLOCK>(gt & have, eq & have, need_eq, s.wtot, pos, picked, eq_picked);
    pos += first;
#pragma unroll
    for (int j = 0; j < E; ++j)
      if ((pick >> j) & 1u) {
        rsel.put(pos, s.id[tid * E + j]);
        ++pos;
      }
  };
  constexpr int LPT = CAP / BLOCK;
  if (total <= BLOCK) pick_list(std::integral_constant<int, 1>());
  else if (LPT > 2 && total <= 2 * BLOCK) pick_list(std::integral_constant<int, 2>());
  else if (LPT > 4 && total <= 4 * BLOCK) pick_list(std::integral_constant<int, 4>());
  else pick_list(std::integral_constant<int, LPT>());
}

// ---------------------------------------------------------------------------
// Rows whose scores a workgroup holds in registers.
#define TAIL_BINS 512
#define TAIL_MEMBERS 64
template <int BLOCK>
struct reg_row_lds {
  kth_lds<BLOCK> kth;
  alignas(16) int bins[TAIL_BINS + TAIL_BINS / 2];
  alignas(16) float lo[BLOCK / 64];
  float top[BLOCK];
  uint2 wtot[BLOCK / 64];
  int listed;
  alignas(16) uint64_t member[TAIL_MEMBERS];     // key, then the complement of the partition: the better, the greater
};

// Where bin `b` of the tail's histogram lies: four words of padding after every eight, so that tail_bin_of_rank's lanes,
// which read eight each, meet in no bank.
__device__ __forceinline__ int tail_word(int b) { return b + ((b >> 3) << 2); }

// As digit_of_rank, of TAIL_BINS bins: lane l has the eight from TAIL_BINS - 1 - 8 l down.
__device__ __forceinline__ int tail_bin_of_rank(const int *bins, int &rank, int &in_bin) {
  const int block = 63 - (threadIdx.x & 63);
  const int4 u = *(const int4 *)(bins + block * 12), v = *(const int4 *)(bins + block * 12 + 4);
  const int upper = (v.x + v.y) + (v.z + v.w), local = ((u.x + u.y) + (u.z + u.w)) + upper;
  const int inc = spin_wave_inclusive_scan(local);
  const unsigned long long found = __ballot(inc >= rank);   // the first of them has it
  if (!found) return -1;
  int r = rank - (inc - local);
  const bool below = r > upper;                             // in the lower four of the lane's
  r -= below ? upper : 0;
  const int4 q = below ? u : v;
  int e = below ? 3 : 7, n = q.w;
  if (r > n) {
    r -= n; n = q.z; --e;
    if (r > n) {
      r -= n; n = q.y; --e;
      if (r > n) { r -= n; n = q.x; --e; }
    }
  }
  const int src = __ffsll((long long)found) - 1;
  rank = __builtin_amdgcn_readlane(r, src);
  in_bin = __builtin_amdgcn_readlane(n, src);
  return __builtin_amdgcn_readlane(block * 8 + e, src);
}

// Picks the kprime best of the candidates a workgroup holds in registers: thread t has the scores f[k] of partitions
// c0 + k, c0 = t * KPT, and the candidates are [nf_lo, first_hi).  put(pos, k) is called for those and the `forced` ones
// (bit k: of the calling thread's), pos = 0, 1 .. in ascending partition order.
// Latency bounds this (the row's one compute unit waits for memory, LDS and barriers in turn, and an instruction of all
// eight wavefronts takes it 8 cycles), so the chain is short: one histogram of the row's upper tail in equal steps of
// score, an exact ranking of the few scores in the step that holds the threshold, one prefix sum; three barriers.
// Both ends of the tail are places in the row's order, so that the steps lie where the scores do, however these are
// spread.  The lower one is the least of the maxima of groups of scores (of four threads down to a quarter of a
// thread's): with at least kprime groups that hold candidates, at least kprime scores reach it.  The upper one is the
// least of the maxima of 2, 8 or 64 interleaved parts of the row, which some 3, 20 or 300 scores exceed; those share the
// last step.
// A step is a monotone function of the score (subtraction, product with a positive scale and truncation are), so the
// order is the scores' own.
// Rows for which that does not work (more than 64 scores in the threshold's step: ties) take block_kth, over all of the
// row or over that step.
// Against one radix digit of 8 bits per barrier (and, with 16 scores per thread and more, a bound from a search among the
// threads' maxima and a list in LDS first), stages 2+3 of normal scores, us: 128 rows of 2048, k 128 5.9 -> 5.8; 32 of 4096
// 7.0 -> 6.4; 64 of 8192 8.0 -> 6.6, 8 of them with k 1024 9.6 -> 7.9; 256 ragged ones of up to 16384 10.7 -> 8.5, 32 of 16384
// with k 1500 13.3 -> 10.2.  Slower where many scores tie at the threshold (128 rows of 2048 with steps of a quarter of their
// deviation 6.7 -> 8.4, 64 of 8192 9.3 -> 10.8) or more outliers than there are parts are a million times the others
// (256 of 16384 10.8 -> 16.2).
// Pinned partitions (scores of +inf) may leave no part of the row without one.  Then the upper end is the greatest finite
// score, and with more of them than are wanted they are the only candidates.  Stage 2 alone, us, with 10 / 64 / 200 of them
// in each row, against a search over the whole row: 128 rows of 2048, k' 116 5.2 / 5.6 / 6.3 -> 4.0 / 4.4 / 4.1; 256 of 16384
// 16.7 / 17.2 / 13.1 -> 8.2 / 8.6 / 8.5 (none: 7.6).  Few of few, where that search is short as well: 8 rows of 256, k' 20,
// 2 / 10 4.4 / 4.6 -> 3.8 / 3.8.
template <int BLOCK, int KPT, typename PUT>
__device__ __forceinline__ void select_elements(float (&f)[KPT], typename key_bits<KPT>::type cand,
                                                typename key_bits<KPT>::type forced, int c0, int nf_lo, int first_hi,
                                                int kprime, reg_row_lds<BLOCK> &s, PUT put) {
  typedef typename key_bits<KPT>::type M;
  constexpr int NW = BLOCK / 64, KLOG = KPT == 4 ? 2 : KPT == 8 ? 3 : KPT == 16 ? 4 : KPT == 32 ? 5 : 6;
  static_assert(KPT == 1 << KLOG, "a power of two");
  constexpr M full = KPT == (int)(8 * sizeof(M)) ? ~(M)0 : ((M)1 << (KPT & (int)(8 * sizeof(M) - 1))) - 1;
  const float inf = __builtin_inff();
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int i = tid; i < TAIL_BINS + TAIL_BINS / 2; i += BLOCK) s.bins[i] = 0;
  if (tid < TAIL_MEMBERS) s.member[tid] = 0;
  if (tid == 0) s.listed = 0;
  // groups of KPT * 2^g partitions that hold a candidate: at least kprime of them (g < -2: there are not)
  int g = 2;
  while (g >= -2 && ((first_hi - 1) >> (KLOG + g)) - (nf_lo >> (KLOG + g)) + 1 < kprime) --g;
#pragma unroll
  for (int k = 0; k < KPT; ++k) f[k] = fmaxf(f[k], -inf);        // NaN ranks as -inf
  if (!__all(cand == full)) {
#pragma unroll
    for (int k = 0; k < KPT; ++k) f[k] = (cand >> k) & 1u ? f[k] : -inf;
  }
  float part[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    part[i] = f[i * (KPT / 4)];
#pragma unroll
    for (int k = 1; k < KPT / 4; ++k) part[i] = fmaxf(part[i], f[i * (KPT / 4) + k]);
  }
  float lo, top = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
  // (groups of -inf do not count: either they hold no candidate, or the tail may be too short, which the search tells)
  auto counts = [&](float v) { return v == -inf ? inf : v; };
  if (g >= 0) {
    lo = top;
    if (g >= 1) lo = fmaxf(lo, spin_dpp<SPIN_DPP_XOR1>(lo));
    if (g == 2) lo = fmaxf(lo, spin_dpp<SPIN_DPP_XOR2>(lo));
    lo = counts(lo);
  } else if (g == -1) {
    lo = fminf(counts(fmaxf(part[0], part[1])), counts(fmaxf(part[2], part[3])));
  } else if (g == -2 || KPT == 4) {
    lo = fminf(fminf(counts(part[0]), counts(part[1])), fminf(counts(part[2]), counts(part[3])));
  } else {
    lo = inf;
#pragma unroll
    for (int k = 0; k < KPT; ++k) lo = fminf(lo, counts(f[k]));
  }
  lo = -spin_wave_max(-lo);
  s.top[tid] = top;
  if (lane == 0) s.lo[wave] = lo;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NW; i += 4) {
    const float4 l = *(const float4 *)(s.lo + i);
    lo = i ? fminf(lo, l.x) : l.x;
    lo = fminf(fminf(lo, l.y), fminf(l.z, l.w));
  }
#pragma unroll
  for (int i = 0; i < NW; ++i) top = fmaxf(top, s.top[i * 64 + lane]);
  if (kprime < 512) {                            // 64 interleaved parts of the row, or these merged to 8 or 2
    top = spin_max_xor32(spin_max_xor16(fmaxf(top, spin_dpp<SPIN_DPP_ROR8>(top))));
    if (kprime < 64) {
      top = fmaxf(top, spin_dpp<SPIN_DPP_XOR1>(top));
      top = fmaxf(top, spin_dpp<SPIN_DPP_XOR2>(top));
    }
    top = counts(top);
    top = fminf(top, spin_dpp<SPIN_DPP_XOR1>(top));
    top = fminf(top, spin_dpp<SPIN_DPP_XOR2>(top));
    top = fminf(top, spin_dpp<SPIN_DPP_HALF_MIRROR>(top));
  } else {
    top = -spin_wave_max(-counts(top));
  }
  lo = spin_readlane(lo, 0);
  top = spin_readlane(top, 0);
  M member = kprime > 0 ? cand : 0;
  if (__builtin_expect(kprime > 0 && top == inf && lo < inf, 0)) {   // uniform: pinned partitions in every part
    float finite = -inf;
    M pinned = 0;
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
      pinned |= f[k] == inf ? (M)1 << k : (M)0;
      finite = fmaxf(finite, f[k] == inf ? -inf : f[k]);
    }
    finite = spin_wave_max(finite);
    int pins = spin_wave_inclusive_scan(popc_bits(pinned));
    __syncthreads();                             // the maxima have been read
    if (lane == 63) {
      s.top[wave] = finite;
      s.wtot[wave].x = (uint32_t)pins;
    }
    __syncthreads();
    (void)spin_waves_before<NW>((int)s.wtot[lane % NW].x, wave, pins);
    if (pins < kprime) top = spin_wave_max(s.top[lane % NW]);    // the greatest finite one: the last step holds little else
    else member &= pinned;                       // more of them than are wanted: the first ones
  }
  const float spread = top - lo;
  // (no group that counts: lo = inf; below 2^-100 the scale might overflow)
  const bool usable = kprime > 0 && spread > 0x1p-100f && spread < inf;
  const float scale = (float)(TAIL_BINS - 1) * __builtin_amdgcn_rcpf(spread);
  int bin = -1, need = kprime, in_bin = 0;
  // (64 scores leave no registers for their steps, which are taken twice then: 32 rows of 40000 20.6 -> 18.1 us)
  constexpr bool KEPT = KPT <= 32;
  auto step_of = [&](float v, float by) { return (int)fminf((v - lo) * by, (float)(TAIL_BINS - 1)); };
  int b[KEPT ? KPT : 1];
  M sure = forced;
  if (usable) {
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
      int at = -1;
      if (f[k] >= lo) {
        at = step_of(f[k], scale);
        atomicAdd(&s.bins[tail_word(at)], 1);
      }
      if (KEPT) b[KEPT ? k : 0] = at;
    }
    __syncthreads();
    bin = tail_bin_of_rank(s.bins, need, in_bin);
    if (bin >= 0) {
      float again = scale;
      if (!KEPT) asm volatile("" : "+v"(again));   // (or the compiler would keep them all the same)
      member = 0;
#pragma unroll
      for (int k = 0; k < KPT; ++k) {
        const int at = KEPT ? b[KEPT ? k : 0] : f[k] >= lo ? step_of(f[k], again) : -1;
        sure |= at > bin ? (M)1 << k : (M)0;
        member |= at == bin ? (M)1 << k : (M)0;
      }
    }
  }
  int pos;
  if (kprime > 0 && (bin < 0 || (in_bin > TAIL_MEMBERS && in_bin != need))) {   // uniform
    uint32_t key[KPT], T;
    unsigned need_eq;
#pragma unroll
    for (int k = 0; k < KPT; ++k) key[k] = score_key(f[k]);
    block_kth<BLOCK, KPT, KPT == 16 || KPT == 32>(key, member, need, 0, s.kth, T, need_eq, first_hi - nf_lo >= 4096);
    M gt = 0, eq = 0;
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
      gt |= key[k] > T ? (M)1 << k : (M)0;
      eq |= key[k] == T ? (M)1 << k : (M)0;
    }
    int picked, eq_picked;
    sure = ordered_picks<BLOCK>((M)(sure | (gt & member)), (M)(eq & member), need_eq, s.wtot, pos, picked, eq_picked);
  } else {
    const bool all = in_bin == need;
    if (all) {
      sure |= member;
    } else if (member) {
#pragma unroll
      for (int k = 0; k < KPT; ++k)
        if ((member >> k) & 1u) s.member[atomicAdd(&s.listed, 1)] = ((uint64_t)score_key(f[k]) << 32) | (uint32_t)~(c0 + k);
    }
    const int mine = popc_bits(sure), inc = spin_wave_inclusive_scan(mine);
    if (lane == 63) s.wtot[wave].x = (uint32_t)inc;
    __syncthreads();
    int total;
    pos = spin_waves_before<NW>((int)s.wtot[lane % NW].x, wave, total) + inc - mine;
    if (!all) {                                  // the `need` best of the bin's scores, lower partitions first among equals
      const uint64_t me = s.member[lane];
      int better = 0;
      for (int j = 0; j < in_bin; j += 8) {      // (zeros past the last: no score's key is)
        uint64_t other[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) other[i] = s.member[j + i];
#pragma unroll
        for (int i = 0; i < 8; ++i) better += other[i] > me;
      }
      for (unsigned long long m = __ballot(lane < in_bin && better < need); m; m &= m - 1) {
        const int d = ~__builtin_amdgcn_readlane((int)(uint32_t)me, __ffsll((long long)m) - 1) - c0;
        pos += d < 0;
        sure |= d >= 0 && d < KPT ? (M)1 << (d & (KPT - 1)) : (M)0;
      }
    }
  }
  if constexpr (KPT <= 8) {
#pragma unroll
    for (int k = 0; k < KPT; ++k)
      if ((sure >> k) & 1u) {
        put(pos, k);
        ++pos;
      }
  } else {                                       // few of a thread's many
    for (; sure; sure &= sure - 1, ++pos) put(pos, ffs_bits(sure) - 1);
  }
}

// forced partitions (a prefix and a suffix of the row) around the kprime candidates, and the padding
template <int BLOCK, typename ROW>
__device__ __forceinline__ void emit_forced(const sel_plan &pl, const ROW &rsel, int32_t *__restrict__ nsel, int row) {
  const int tid = threadIdx.x;
  for (int i = tid; i < min(pl.nf_lo, rsel.stride); i += BLOCK) rsel.put(i, i);
  const int at = pl.nf_lo + pl.kprime;
  for (int i = tid; i < pl.P - pl.first_hi && at + i < rsel.stride; i += BLOCK) rsel.put(at + i, pl.first_hi + i);
  for (int i = pl.take + tid; i < rsel.stride; i += BLOCK) rsel.pad(i);
  if (tid == 0) rsel.count(nsel, row, pl.take);
}

// The windows of a row of at most BLOCK * KPT variable-length partitions, and its forced prefix and suffix
// [0, nf_lo) and [first_hi, P).  Every thread holds the table entries of its KPT partitions, so one round of loads and
// two barriers stand for four binary searches of a dozen dependent loads each.  (With more than 16 per thread, which
// the registers would not hold beside the scores, the entries are read where they are used.)  TABLES: they also go to
// `tables`, first pages [BLOCK * KPT] and then tokens, for the stage that looks the selection up.
template <int BLOCK, int KPT, bool TABLES>
__device__ __forceinline__ spin_var_span block_var_span(const spin_var &var, size_t vbase, int row, int PP, int sink_pages,
                                               int recent_pages, int &nf_lo, int &first_hi, int32_t *tables) {
  constexpr int NW = BLOCK / 64, HELD = KPT <= 16 ? KPT : 1;
  __shared__ int s_pages;
  __shared__ int4 s_cnt[NW];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c0 = threadIdx.x * KPT;
  spin_var_span w;
  struct entry { int start, end; };
  auto load = [&](int k) {                             // the tables are as long as the score array
    entry e = {0, 0};
    if (c0 + k < PP) {
      e.start = var.first_page[vbase + c0 + k];
      e.end = e.start + spin_var_npages(var, vbase, c0 + k);
    }
    return e;
  };
  entry held[HELD];
  if constexpr (HELD == KPT) {                         // four at a time, and without a branch (see spin_buffer)
    const __amdgpu_buffer_rsrc_t first = spin_buffer(var.first_page + vbase, (uint32_t)max(PP, 0) * sizeof(int32_t));
    const __amdgpu_buffer_rsrc_t tokens = spin_buffer(var.tokens + vbase, (uint32_t)max(PP, 0) * sizeof(int32_t));
    int4 f[KPT / 4], t[KPT / 4];
#pragma unroll
    for (int k = 0; k < KPT / 4; ++k) {
      f[k] = __builtin_bit_cast(int4, spin_buffer_load_kept(first, (uint32_t)(c0 + 4 * k) * sizeof(int32_t)));
      t[k] = __builtin_bit_cast(int4, spin_buffer_load_kept(tokens, (uint32_t)(c0 + 4 * k) * sizeof(int32_t)));
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < KPT / 4; ++k) {
      if (TABLES) {
        *(int4 *)(tables + c0 + 4 * k) = f[k];
        *(int4 *)(tables + BLOCK * KPT + c0 + 4 * k) = t[k];
      }
      const int fs[4] = {f[k].x, f[k].y, f[k].z, f[k].w}, ts[4] = {t[k].x, t[k].y, t[k].z, t[k].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) held[4 * k + i] = entry{fs[i], fs[i] + ((ts[i] + 15) >> 4)};
    }
  }
  w.P = min(min(max(var.count[row], 0), PP), BLOCK * KPT);
  if (w.P == 0 && threadIdx.x == 0) s_pages = 0;
  if (HELD == KPT) {
#pragma unroll
    for (int k = 0; k < HELD; ++k)
      if (c0 + k == w.P - 1) s_pages = held[k].end;
  } else if (w.P > 0 && (w.P - 1) / KPT == (int)threadIdx.x) {
    s_pages = load((w.P - 1) % KPT).end;
  }
  __syncthreads();
  w.pages = s_pages;
  spin_var_windows(w, sink_pages, recent_pages);
  // partitions that end by sink_end, start before it, start before recent_begin, start at or before it
  int4 n = make_int4(0, 0, 0, 0);
#pragma unroll
  for (int k = 0; k < KPT; ++k)
    if (c0 + k < w.P) {
      const entry e = HELD == KPT ? held[k < HELD ? k : 0] : load(k);
      n.x += e.end <= w.sink_end;
      n.y += e.start < w.sink_end;
      n.z += e.start < w.recent_begin;
      n.w += e.start <= w.recent_begin;
    }
  n.x = spin_wave_inclusive_scan(n.x);
  n.y = spin_wave_inclusive_scan(n.y);
  n.z = spin_wave_inclusive_scan(n.z);
  n.w = spin_wave_inclusive_scan(n.w);
  if (lane == 63) s_cnt[wave] = n;
  __syncthreads();
  n = make_int4(0, 0, 0, 0);
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    n.x += s_cnt[i].x;
    n.y += s_cnt[i].y;
    n.z += s_cnt[i].z;
    n.w += s_cnt[i].w;
  }
  nf_lo = n.x;
  w.at_sink = n.y - 1;
  first_hi = n.z;
  w.at_recent = n.w - 1;
  return w;
}

// Register-resident variant for rows of at most BLOCK * KPT partitions: every
// thread keeps KPT consecutive scores in registers, so they are read once.
// Returns the number of selected partitions (and, with variable-length partitions, the row's windows in `span`).
// `meanwhile` issues what the caller wants under way beside the scores.
template <int BLOCK, int KPT, bool TABLES = false, typename ROW, typename MEANWHILE>
__device__ __forceinline__ int select_reg_row(
    const float *__restrict__ scores, const int32_t *__restrict__ part_offsets,
    const int32_t *__restrict__ seq_lens, int Hkv, int tp, int topk, int includes_forced, int sink_pages,
    int recent_pages, const ROW &rsel, int32_t *__restrict__ nsel, int row, spin_var var,
    spin_var_span &span, reg_row_lds<BLOCK> &s,
    MEANWHILE meanwhile, int32_t *tables = nullptr) {
  typedef typename key_bits<KPT>::type M;
  const int b = row / Hkv, h = row - b * Hkv;
  const int N = seq_lens[b];
  const int off_b = part_offsets[b];
  const int PP = part_offsets[b + 1] - off_b;
  const size_t vbase = (size_t)Hkv * off_b + (size_t)h * PP;
  const float *rs = scores + vbase;
  const int sel_stride = rsel.stride;
  const int c0 = threadIdx.x * KPT;   // this thread's partitions: c0 .. c0 + KPT - 1
  float f[KPT];
  const __amdgpu_buffer_rsrc_t buf = spin_buffer(rs, (uint32_t)max(PP, 0) * sizeof(float));   // zeros past the row's end
#pragma unroll
  for (int k4 = 0; k4 < KPT; k4 += 4) {
    const float4 v = __builtin_bit_cast(float4, spin_buffer_load_kept(buf, (uint32_t)(c0 + k4) * sizeof(float)));
    f[k4] = v.x; f[k4 + 1] = v.y; f[k4 + 2] = v.z; f[k4 + 3] = v.w;
  }
  __builtin_amdgcn_sched_barrier(0);
  meanwhile();

  // forced partitions: a prefix [0, nf_lo) and a suffix [first_hi, P)
  sel_plan pl;
  if (var.count) {
    int nf_lo, first_hi;
    span = block_var_span<BLOCK, KPT, TABLES>(var, vbase, row, PP, sink_pages, recent_pages, nf_lo, first_hi, tables);
    pl = plan_of(span.P, nf_lo, first_hi, topk, includes_forced, sel_stride);
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
  for (int i = pl.take + (int)threadIdx.x; i < sel_stride; i += BLOCK) rsel.pad(i);
  if (threadIdx.x == 0) rsel.count(nsel, row, pl.take);
  const M cand = range_bits<KPT>(c0, pl.nf_lo, pl.first_hi);
  const M forced = range_bits<KPT>(c0, 0, pl.P) & ~cand;
  select_elements<BLOCK, KPT>(f, cand, forced, c0, pl.nf_lo, pl.first_hi, pl.kprime, s,
                              [&](int pos, int k) { rsel.put(pos, c0 + k); });
  return pl.take;
}

// ---------------------------------------------------------------------------
// Rows whose scores come with the maximum of every tile (2^gs_log consecutive partitions; 16, 8 or 4): stage 1
// writes it as it holds the scores, or a launch of its own takes it from the score array.
//
// The k'-th largest maximum T0 bounds the threshold from below (k' tiles hold a score at least that large), so
// candidates above T0 lie in the fewer than k' tiles whose maximum is above it, and of the tiles whose maximum
// equals T0 only the first that make up k' can matter: each holds a candidate with exactly that key, and among
// equals the lowest partitions win.  The row's one workgroup therefore reads one value per tile and then the scores
// of k' tiles, whatever the row's length and however many scores tie; tiles that hold forced partitions are no
// bound for anything and are read as well.  T0 then rules most of those scores out and the rest form the list.
#define TILE_LIST 4098     // tiles a row may read (16-bit ids: rows of up to 131072 partitions, 4 or more to a tile)
#define ROW_PARTS 131072   // partitions of the longest row
#define ROW_BINS 4096
#define ROW_LIST 2048
template <int BLOCK, int CAP>
struct tiles_lds : elements_lds<BLOCK, CAP> {
  uint16_t tile[TILE_LIST];
};
// LDS of select_whole_row
template <int BLOCK>
struct row_lds {
  kth_lds<BLOCK> kth;
  uint2 wtot[BLOCK / 64];
  alignas(16) int4 found;
  int listed;
  uint32_t above[ROW_PARTS / 32], equal[ROW_PARTS / 32];   // one bit per partition
  union {
    alignas(16) int bins[ROW_BINS];
    struct { uint32_t key[ROW_LIST]; int32_t id[ROW_LIST]; } list;
  };
};
template <int BLOCK, int CAP>
union tiles_row_lds {
  tiles_lds<BLOCK, CAP> tiles;
  row_lds<BLOCK> row;
};

// The kprime best candidates of a row of at most ROW_PARTS partitions, stored ascending at rsel[nf_lo ..], from walks
// over all its scores (a quad per lane and load): a histogram of the keys from `lo` to `hi`, which
// is repeated inside the bin of the k'-th candidate while that holds too many scores (ties, or a row whose scores lie
// close together), then one walk that marks the scores above the bin in a bitmap and lists those inside it.
// No candidate's key reaches `hi`; fewer than kprime may reach `lo`, and then the keys below it are searched.
// This is the path of rows whose k' tiles hold more scores than a list takes.  The one compute unit is bound by
// instructions per score: about ten for the histogram, four for the bitmap.  Against a radix search that read the tiles'
// scores five times and, for k' beyond the tile list, one contiguous stretch of scores per thread: stages 2+3, 2 rows of
// 65536 token partitions, k' 2560 / 3600 / 4096 / 8192: 67 / 82 / 202 / 217 -> 34 / 37 / 38 / 53 us; 2 rows of 20000,
// k' 2048 / 8192: 44 / 90 -> 22 / 64.  (Being in the kernel it costs rows that do not come here 0.2 to 0.3 us, out of
// line as well; four quads under way as good as eight, which take 30 more registers.)
template <int BLOCK, typename ROW>
__device__ __forceinline__ void select_whole_row(const float *__restrict__ rs, uint32_t lo, uint32_t hi, const sel_plan &pl,
                                        const ROW &rsel, row_lds<BLOCK> &s) {
  constexpr int NW = BLOCK / 64, V = 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int words = (pl.first_hi + 31) >> 5;
  for (int i = tid; i < words; i += BLOCK) s.above[i] = s.equal[i] = 0u;
  if (tid == 0) s.listed = 0;
  // `use` gets V quads of scores, the partition of the first (load i: i * BLOCK * 4 further on) and a bit per candidate
  auto walk = [&](auto use) {
    for (int base = pl.nf_lo & ~3; base < pl.first_hi; base += BLOCK * 4 * V) {
      const int p0 = base + tid * 4;
      float4 v[V];
      uint32_t have = 0;
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const int p = p0 + i * BLOCK * 4;                // the row's scores are padded to a multiple of 16
        v[i] = p < pl.first_hi ? *(const float4 *)(rs + p) : make_float4(0.f, 0.f, 0.f, 0.f);
        have |= range_bits<4>(p, pl.nf_lo, pl.first_hi) << (4 * i);
      }
      use(v, p0, have);
    }
  };
  int rank = pl.kprime;                                  // of the threshold among the keys of [lo, hi)
  // settles 12 bits a time, after one walk in vain at most
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = max(20 - __clz((int)(hi - lo - 1)), 0);
    const uint32_t span = hi - lo;
    int same = 0;                                        // of one key: counted by the thread, not one by one in LDS
    for (int i = tid; i < ROW_BINS; i += BLOCK) s.bins[i] = 0;
    __syncthreads();
    walk([&](const float4 (&v)[V], int, uint32_t have) {
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const float f[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t d = score_key(f[e]) - lo;       // (below lo: wraps to more than any span)
          const bool in = ((have >> (4 * i + e)) & 1u) && d < span;
          if (span == 1) same += in;
          else if (in) atomicAdd(&s.bins[d >> shift], 1);
        }
      }
    });
    if (span == 1) atomicAdd(&s.bins[0], same);
    __syncthreads();
    // thread t has the bins from ROW_BINS - 1 - t * BPT down
    constexpr int BPT = ROW_BINS / BLOCK;
    int c[BPT], local = 0, total;
#pragma unroll
    for (int j = 0; j < BPT; ++j) { c[j] = s.bins[ROW_BINS - 1 - tid * BPT - j]; local += c[j]; }
    const int inc = spin_wave_inclusive_scan(local);
    if (lane == 63) s.wtot[wave].x = (unsigned)inc;
    __syncthreads();
    int running = spin_waves_before<NW>((int)s.wtot[lane % NW].x, wave, total) + inc - local;
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
      if (running < rank && running + c[j] >= rank) s.found = make_int4(ROW_BINS - 1 - tid * BPT - j, rank - running, c[j], 0);
      running += c[j];
    }
    __syncthreads();
    if (total < rank) {                                  // uniform
      if (lo == 0) break;                                // (cannot be: every candidate was counted)
      rank -= total;
      hi = lo;
      lo = 0;
      continue;
    }
    const int4 f = s.found;
    const uint32_t bin = (uint32_t)__builtin_amdgcn_readfirstlane(f.x);
    rank = __builtin_amdgcn_readfirstlane(f.y);
    lo += bin << shift;
    hi = lo + min(1u << shift, hi - lo);
    if (__builtin_amdgcn_readfirstlane(f.z) <= ROW_LIST || hi - lo == 1) break;
  }
  // key order is float order, but NaN scores, which rank as -inf, fail every comparison
  const bool all = lo <= SPIN_KEY_MINUS_INF, one = hi - lo == 1;
  const float f_lo = key_floor_score(lo, true), f_hi = key_floor_score(hi, false);
  walk([&](const float4 (&v)[V], int p0, uint32_t have) {
    uint32_t above = 0, within = 0;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const float f[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        within |= (all || f[e] >= f_lo) ? 1u << (4 * i + e) : 0u;
        above |= f[e] >= f_hi ? 1u << (4 * i + e) : 0u;
      }
    }
    above &= have;
    within &= have & ~above;
#pragma unroll
    for (int i = 0; i < V; ++i) {                        // (p is a multiple of 4: a quad's bits lie in one word)
      const int p = p0 + i * BLOCK * 4;
      const uint32_t bits = (above >> (4 * i)) & 15u, eq = (within >> (4 * i)) & 15u;
      if (bits) atomicOr(&s.above[p >> 5], bits << (p & 31));
      if (one && eq) atomicOr(&s.equal[p >> 5], eq << (p & 31));
    }
    if (!one && __ballot(within != 0u)) {
      const int inc = spin_wave_inclusive_scan(__popc(within));
      int to = 0;
      if (lane == 63) to = atomicAdd(&s.listed, inc);
      to = __builtin_amdgcn_readlane(to, 63) + inc - __popc(within);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const float f[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((within >> (4 * i + e)) & 1u) {
            if (to < ROW_LIST) {
              s.list.key[to] = score_key(f[e]);
              s.list.id[to] = p0 + i * BLOCK * 4 + e;
            }
            ++to;
          }
      }
    }
  });
  __syncthreads();
  unsigned quota = (unsigned)rank;                       // scores equal to the threshold that are wanted
  if (!one) {
    constexpr int E = ROW_LIST / BLOCK;
    const int n = min(s.listed, ROW_LIST);
    uint32_t key[E], T;
#pragma unroll
    for (int j = 0; j < E; ++j) key[j] = tid * E + j < n ? s.list.key[tid * E + j] : 0u;
    block_kth<BLOCK, E>(key, range_bits<E>(tid * E, 0, n), rank, 0, s.kth, T, quota);
#pragma unroll
    for (int j = 0; j < E; ++j) {
      if (tid * E + j >= n || key[j] < T) continue;
      const int p = s.list.id[tid * E + j];
      atomicOr(key[j] > T ? &s.above[p >> 5] : &s.equal[p >> 5], 1u << (p & 31));
    }
  }
  int first = pl.nf_lo;
  for (int w0 = 0; w0 < words; w0 += BLOCK) {
    __syncthreads();
    const int w = w0 + tid;
    int at, picked, eq_picked;
    uint32_t taken = ordered_picks<BLOCK>(w < words ? s.above[w] : 0u, w < words ? s.equal[w] : 0u, quota, s.wtot, at,
                                          picked, eq_picked);
    for (at += first; taken; taken &= taken - 1, ++at)
      rsel.put(at, w * 32 + __ffs((int)taken) - 1);
    first += picked;
    quota -= (unsigned)eq_picked;
  }
}

// False (for the whole workgroup, nothing stored): more scores than the list holds.
template <int BLOCK, int MPT, int CAP, typename ROW>
__device__ __forceinline__ bool list_by_tile_maxima(const float *__restrict__ rs, const uint32_t (&top)[MPT],
                                           typename key_bits<MPT>::type cand, int t_lo, int t_hi, int gs_log,
                                           int slack, const sel_plan &pl, const ROW &rsel, tiles_lds<BLOCK, CAP> &s) {
  constexpr int NW = BLOCK / 64;
  typedef typename key_bits<MPT>::type M;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int gs = 1 << gs_log, kprime = pl.kprime, m0 = tid * MPT;
  uint32_t T0 = 0;
  unsigned need_eq = 0;
  if (t_hi - t_lo >= kprime) block_kth<BLOCK, MPT>(top, cand, kprime, slack, s.kth, T0, need_eq);
  // ascending list of the tiles to read, the one that straddles either end of the candidates among them (both
  // ends in one tile: that one)
  const int has_lo = (pl.nf_lo & (gs - 1)) ? 1 : 0, has_hi = (pl.first_hi & (gs - 1)) && t_hi >= t_lo ? 1 : 0;
  M gt = 0, eq = 0;
#pragma unroll
  for (int j = 0; j < MPT; ++j) {
    gt |= top[j] > T0 ? (M)1 << j : (M)0;
    eq |= top[j] == T0 ? (M)1 << j : (M)0;
  }
  int pos, ntiles, eq_tiles;
  M pick = ordered_picks<BLOCK>((M)(gt & cand), (M)(eq & cand), need_eq, s.wtot, pos, ntiles, eq_tiles);
  ntiles += has_lo;
  pos += has_lo;
  while (pick) {
    const int j = ffs_bits(pick) - 1;
    pick &= pick - 1;
    if (pos < TILE_LIST) s.tile[pos] = (uint16_t)(m0 + j);
    ++pos;
  }
  if (tid == 0) {
    if (has_lo) s.tile[0] = (uint16_t)(t_lo - 1);
    if (has_hi && ntiles < TILE_LIST) s.tile[ntiles] = (uint16_t)t_hi;
  }
  ntiles = min(ntiles + has_hi, TILE_LIST);
  __syncthreads();
  const bool all = T0 <= SPIN_KEY_MINUS_INF;           // (NaN scores rank at -inf and would fail the comparison)
  const float bf = key_floor_score(T0, true);
  const int q_log = gs_log - 2, nquads = ntiles << q_log;
  // Four scores (a quad) per lane and load, neighbouring lanes neighbouring quads: a wavefront's load touches as few
  // lines as there are, which matters because the one compute unit that fetches k' scattered lines is bound by them
  // (1024 tiles: 6.5 us; 7.0 with four quads in a row per lane).  A round is V loads per lane; wavefront w has the
  // quads [64 V w, 64 V (w + 1)) of it, so order is wavefront, load, lane, score.
  auto load_quad = [&](int qd, int &p, float4 &v) {
    p = -4;                                            // no candidates
    v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (qd < nquads) {
      p = ((int)s.tile[qd >> q_log] << gs_log) + ((qd & ((1 << q_log) - 1)) << 2);
      v = *(const float4 *)(rs + p);
    }
  };
  // which of a quad's scores are candidates above the bound
  auto quad_bits = [&](int p, const float4 &v) {
    const float f[4] = {v.x, v.y, v.z, v.w};
    uint32_t bits = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) bits |= (all || f[e] >= bf) ? 1u << e : 0u;
    return bits & range_bits<4>(p, pl.nf_lo, pl.first_hi);
  };
  int total = 0;
  auto gather = [&](auto loads) {
    constexpr int V = decltype(loads)::value;
    for (int q0 = 0; q0 < nquads; q0 += BLOCK * V) {
      float4 v[V];
      int p[V];
#pragma unroll
      for (int j = 0; j < V; ++j) load_quad(q0 + (wave * V + j) * 64 + lane, p[j], v[j]);
      // the loads' counts (at most 256 each over the wavefront) share words for the prefix sums, two to a word
      uint32_t keep[V], inc[(V + 1) / 2];
#pragma unroll
      for (int j = 0; j < V; j += 2) {
        keep[j] = quad_bits(p[j], v[j]);
        uint32_t cnt = (uint32_t)__popc(keep[j]);
        if (j + 1 < V) {
          keep[j + 1] = quad_bits(p[j + 1], v[j + 1]);
          cnt |= (uint32_t)__popc(keep[j + 1]) << 16;
        }
        inc[j / 2] = (uint32_t)spin_wave_inclusive_scan((int)cnt);
      }
      int at[V], wave_total = 0;
#pragma unroll
      for (int j = 0; j < V; ++j) {
        const int sh = (j & 1) * 16;
        at[j] = wave_total + (int)((inc[j / 2] >> sh) & 0xffffu) - __popc(keep[j]);
        wave_total += (int)(((uint32_t)__builtin_amdgcn_readlane((int)inc[j / 2], 63) >> sh) & 0xffffu);
      }
      if (lane == 0) s.wtot[wave].x = (unsigned)wave_total;
      __syncthreads();
      int round_total;
      const int before = total + spin_waves_before<NW>((int)s.wtot[lane % NW].x, wave, round_total);
      total += round_total;
      if (total > CAP) return;                         // block-uniform
#pragma unroll
      for (int j = 0; j < V; ++j) {
        if (!keep[j]) continue;
        const float f[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
        int to = before + at[j];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((keep[j] >> e) & 1u) {
            s.key[to] = score_key(f[e]);
            s.id[to] = p[j] + e;
            ++to;
          }
      }
      __syncthreads();                                 // the list is whole, and s.wtot may be written again
    }
  };
  // loads per lane: a quad that is not there costs as many instructions as one that is
  if (nquads <= BLOCK * 3) gather(std::integral_constant<int, 3>());
  else if (nquads <= BLOCK * 5) gather(std::integral_constant<int, 5>());
  else gather(std::integral_constant<int, 9>());
  if (total > CAP) return false;
  pick_from_list<BLOCK, CAP>(total, kprime, pl.nf_lo, rsel, s);
  return true;
}

// Stores the kprime best candidates ascending at rsel[nf_lo ..].  A row with fewer than k' tiles reads them all; one
// with more scores above the bound than the list holds is walked whole.
// `maxima`: the calling thread's MPT of the row (load_tile_maxima, whose loads need not wait for the row's plan).
template <int MPT>
__device__ inline void load_tile_maxima(float4 (&v)[MPT / 4], const float *__restrict__ maxima, int maxima_stride) {
  const int m0 = threadIdx.x * MPT;
#pragma unroll
  for (int j = 0; j < MPT / 4; ++j)                    // the stride is a multiple of 4
    v[j] = m0 + 4 * j < maxima_stride ? *(const float4 *)(maxima + m0 + 4 * j) : make_float4(0.f, 0.f, 0.f, 0.f);
}
template <int BLOCK, int MPT, int CAP, typename ROW>
__device__ __forceinline__ void select_by_tile_maxima(const float *__restrict__ rs, const float4 (&maxima)[MPT / 4], int gs_log,
                                             const sel_plan &pl, const ROW &rsel, tiles_row_lds<BLOCK, CAP> &lds) {
  constexpr int NW = BLOCK / 64;
  typedef typename key_bits<MPT>::type M;
  tiles_lds<BLOCK, CAP> &s = lds.tiles;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int gs = 1 << gs_log, kprime = pl.kprime;
  const int t_lo = (pl.nf_lo + gs - 1) >> gs_log, t_hi = pl.first_hi >> gs_log;   // tiles of candidates only
  const int m0 = tid * MPT;
  uint32_t top[MPT];
#pragma unroll
  for (int j = 0; j < MPT / 4; ++j) {
    top[4 * j] = score_key(maxima[j].x);
    top[4 * j + 1] = score_key(maxima[j].y);
    top[4 * j + 2] = score_key(maxima[j].z);
    top[4 * j + 3] = score_key(maxima[j].w);
  }
  const M cand = range_bits<MPT>(m0, t_lo, t_hi);
  // Scores above the bound: all candidates where there is none, else a share of 1 - k'/T of the T tiles holds none, so
  // that there are about T ln(T / (T - k')) where scores come in no order.  The search for the bound is shorter with a
  // slack of an eighth (1152 tiles instead of 1024: one round of loads either way), which is left out where the list
  // would not hold the scores of so many (64 rows of 9000, k' 512: step 26.3 -> 23.9 us; stage 2 of 2 rows of 65536, k'
  // 2560: 26.2 -> 22.0).
  const int T = t_hi - t_lo;
  auto fits = [&](int tiles) {                                                     // block-uniform
    return tiles < T && tiles + 2 <= TILE_LIST &&
           (float)T * (__builtin_amdgcn_logf((float)T) - __builtin_amdgcn_logf((float)(T - tiles))) <= CAP * 1.4427f;
  };
  const int slack = fits(kprime + (kprime >> 3)) ? kprime >> 3 : 0;
  const bool whole = pl.first_hi - pl.nf_lo > CAP && !fits(kprime);
  if (whole) {
    uint32_t kmx = 0u, kmn = 0xffffffffu;
#pragma unroll
    for (int j = 0; j < MPT; ++j)
      if ((cand >> j) & 1u) { kmx = max(kmx, top[j]); kmn = min(kmn, top[j]); }
    kmx = spin_wave_max_u32(kmx);
    kmn = spin_wave_min_u32(kmn);
    if (lane == 0) { s.kth.wmax[wave] = kmx; s.kth.wmin[wave] = kmn; }
  } else if (list_by_tile_maxima<BLOCK, MPT, CAP>(rs, top, cand, t_lo, t_hi, gs_log, slack, pl, rsel, s)) {
    return;
  }
  __syncthreads();
  // from the least to the greatest of the tiles' maxima, which block_kth leaves in LDS as well; the candidates of the
  // tiles that straddle either end may be greater
  uint32_t kmx = spin_wave_max_u32(s.kth.wmax[lane % NW]);
  const uint32_t kmn = spin_wave_min_u32(s.kth.wmin[lane % NW]);
  const int p = ((lane & 16 ? t_hi : t_lo - 1) << gs_log) + (lane & (gs - 1));
  kmx = max(kmx, spin_wave_max_u32(p >= pl.nf_lo && p < pl.first_hi ? score_key(rs[p]) : 0u));
  __syncthreads();
  select_whole_row<BLOCK>(rs, min(kmn, kmx), kmx + 1, pl, rsel, lds.row);
}

// exclusive prefix sum of one int per thread over the workgroup, plus the total
template <int BLOCK>
__device__ inline int block_exclusive_scan(int v, int *s_wave, int &total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int inc = spin_wave_inclusive_scan(v);
  __syncthreads();  // s_wave may still be read from a previous scan
  if (lane == 63) s_wave[wave] = inc;
  __syncthreads();
  int off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < BLOCK / 64; ++w) {
    const int x = s_wave[w];
    if (w < wave) off += x;
    tot += x;
  }
  total = tot;
  return off + inc - v;
}

// Rows of any length: every pass re-reads the row's scores.
template <int BLOCK>
__device__ inline void select_generic_row(
    const float *__restrict__ scores, const int32_t *__restrict__ part_offsets,
    const int32_t *__restrict__ seq_lens, int Hkv, int tp, int topk, int includes_forced, int sink_pages,
    int recent_pages, int sel_stride, int32_t *__restrict__ sel, int32_t *__restrict__ nsel, int row) {
  __shared__ int s_hist[256];
  __shared__ int s_wave[BLOCK / 64];
  __shared__ int s_digit, s_remaining;

  const int b = row / Hkv, h = row - b * Hkv;
  const int N = seq_lens[b];
  const int PP = part_offsets[b + 1] - part_offsets[b];
  const float *rs = scores + (size_t)Hkv * part_offsets[b] + (size_t)h * PP;
  int32_t *rsel = sel + (size_t)row * sel_stride;
  const int tid = threadIdx.x;
  int P = N > 0 ? (N + tp - 1) / tp : 0;
  if (P > PP) P = PP;

  // forced partitions: a prefix [0, nf_lo) and a suffix [first_hi, P)
  const int pages = (N + 15) >> 4;
  int sink_end = min(sink_pages, pages);
  int recent_begin = max(pages - recent_pages, 0);
  if (sink_end >= recent_begin) { sink_end = pages; recent_begin = pages; }
  int nf_lo = (N <= sink_end * 16) ? P : (sink_end * 16) / tp;
  int first_hi = min((recent_begin * 16 + tp - 1) / tp, P);
  if (first_hi <= nf_lo) { nf_lo = P; first_hi = P; }
  const int nforced = nf_lo + (P - first_hi);
  const int ncand = P - nforced;
  int kprime = includes_forced ? max(topk - nforced, 0) : topk;
  kprime = min(kprime, ncand);
  int take = nforced + kprime;
  if (take > sel_stride) {   // cannot happen for strides from spin_sel_stride(); keep stores in range
    kprime = max(sel_stride - nforced, 0);
    take = min(nforced + kprime, sel_stride);
  }

  // contiguous chunk of partitions per thread
  int chunk = (P + BLOCK - 1) / BLOCK;
  chunk = (chunk + 3) & ~3;
  const int c0 = min(tid * chunk, P), c1 = min(c0 + chunk, P);

  // ---- radix select of the kprime-th largest candidate key ----
  uint32_t prefix = 0;
  int remaining = kprime;   // rank (1-based) of the wanted key among keys matching the prefix
  if (kprime > 0) {
    for (int shift = 24; shift >= 0; shift -= 8) {
      if (tid < 256) s_hist[tid] = 0;
      __syncthreads();
      for (int p = c0; p < c1; ++p) {
        if (p < nf_lo || p >= first_hi) continue;
        const uint32_t k = score_key(rs[p]);
        if (shift == 24 || (k >> (shift + 8)) == prefix) atomicAdd(&s_hist[(k >> shift) & 255u], 1);
      }
      __syncthreads();
      // suffix sums over digits: thread t looks at digit 255 - t
      int cnt = tid < 256 ? s_hist[255 - tid] : 0, total;
      const int excl = block_exclusive_scan<BLOCK>(cnt, s_wave, total);
      if (tid < 256 && excl < remaining && excl + cnt >= remaining) {
        s_digit = 255 - tid;
        s_remaining = remaining - excl;
      }
      __syncthreads();
      prefix = (prefix << 8) | (uint32_t)s_digit;
      remaining = s_remaining;
      __syncthreads();
    }
  }
  const uint32_t T = prefix;
  const int need_eq = kprime > 0 ? remaining : 0;   // how many candidates with key == T to take

  // ---- index-ordered compaction ----
  int my_gt = 0, my_eq = 0;
  for (int p = c0; p < c1; ++p) {
    if (p < nf_lo || p >= first_hi) { ++my_gt; continue; }
    if (kprime == 0) continue;
    const uint32_t k = score_key(rs[p]);
    my_gt += k > T;
    my_eq += k == T;
  }
  int total_eq, total_sel;
  const int eq_before = block_exclusive_scan<BLOCK>(my_eq, s_wave, total_eq);
  int eq_quota = min(max(need_eq - eq_before, 0), my_eq);
  const int pos0 = block_exclusive_scan<BLOCK>(my_gt + eq_quota, s_wave, total_sel);
  int pos = pos0;
  for (int p = c0; p < c1; ++p) {
    bool pick;
    if (p < nf_lo || p >= first_hi) pick = true;
    else if (kprime == 0) pick = false;
    else {
      const uint32_t k = score_key(rs[p]);
      pick = k > T;
      if (k == T && eq_quota > 0) { pick = true; --eq_quota; }
    }
    if (pick && pos < sel_stride) rsel[pos++] = p;
  }
  for (int i = take + tid; i < sel_stride; i += BLOCK) rsel[i] = -1;
  if (tid == 0) nsel[row] = min(total_sel, sel_stride);
}

// Selects a row of at most ROW_PARTS partitions from its scores and their tiles' maxima; returns the selection's length.
// HELD: `rsel` keeps the selection in LDS and the caller stores it.  (A row that is longer than the context's longest one
// has no maxima for all its tiles: its selection goes through `sel` in memory.)
template <int BLOCK, int MPT, int CAP, bool HELD, typename ROW>
__device__ __forceinline__ int select_tiles_row(
    const float *__restrict__ scores, const float *__restrict__ maxima, int max_stride, int gs_log,
    const int32_t *__restrict__ part_offsets, const int32_t *__restrict__ seq_lens, int Hkv, int tp, int topk,
    int includes_forced, int sink_pages, int recent_pages, int32_t *sel, const ROW &rsel, int32_t *__restrict__ nsel,
    int row, tiles_row_lds<BLOCK, CAP> &s) {
  float4 mine[MPT / 4];
  load_tile_maxima<MPT>(mine, maxima + (size_t)row * max_stride, max_stride);
  const int b = row / Hkv, h = row - b * Hkv;
  const int PP = part_offsets[b + 1] - part_offsets[b];
  const float *rs = scores + (size_t)Hkv * part_offsets[b] + (size_t)h * PP;
  const sel_plan pl = select_plan(seq_lens[b], PP, tp, topk, includes_forced, sink_pages, recent_pages, rsel.stride);
  const bool no_maxima = pl.kprime > 0 && ((pl.P >> gs_log) > min(max_stride, BLOCK * MPT) || pl.P > ROW_PARTS);
  if (!no_maxima) {
    emit_forced<BLOCK>(pl, rsel, nsel, row);
    if (pl.kprime > 0) select_by_tile_maxima<BLOCK, MPT, CAP>(rs, mine, gs_log, pl, rsel, s);
  } else {
    select_generic_row<BLOCK>(scores, part_offsets, seq_lens, Hkv, tp, topk, includes_forced, sink_pages, recent_pages,
                              rsel.stride, sel, nsel, row);
    __syncthreads();
    if (HELD)
      for (int i = threadIdx.x; i < pl.take; i += BLOCK) rsel.put(i, sel[(size_t)row * rsel.stride + i]);
  }
  return pl.take;
}
