// Stages 2, 3 and 4 in one launch for partitions smaller than a page (all-resident mode): as spin_select_decode_kernel,
// every workgroup of a row selects for itself.  What it attends is dealt by tiles of 16 selected tokens, straight from the
// selection: a lane looks the slot of its token up, so that no wavefront waits for the page list to be drawn up and all
// have the same number of tiles (dealt by pages, whose selected tokens are few and uneven, a wavefront's last tile is
// nearly empty).  The page list is made meanwhile, each workgroup storing the part that begins in its share of the
// selection, while its first tiles are under way.
// Latency bounds it: of 24 us from its start to the last output (64 rows of 65536 tokens, 1024 attended), maxima 1.1,
// tiles chosen 3.8, their scores fetched and listed 4.2, tokens chosen 2.7, slots 1.5, attended 5.9, merged 2.8.  Whole
// steps, us, against the launch of stages 2+3 followed by that of stage 4: those rows 53.9 -> 50.4; 8 of them 31.0 -> 24.4;
// 96 of 20001, 1500 attended 58.9 -> 51.7; 32 of 9001, 400 attended 25.9 -> 19.5.  With a row's splits on different dies,
// each of which then fetched the row's tiles from memory, the first took 2.5 more.
#include "spin_token_tiles_dev.h"
#include "spin_step_dev.h"

#define STEP_TOK_ROUNDS 4                        // lookups per lane and batch
#define STEP_TOK_LIST (64 * STEP_TOK_ROUNDS)     // list entries per wavefront
static_assert(8 * STEP_TOK_LIST * sizeof(uint32_t) == SPIN_STEP_TOKENS_LDS, "the context sizes the launch");

template <int KPT, bool TILES>
__global__ __launch_bounds__(512) void spin_select_decode_tokens_kernel(
    const float *__restrict__ scores, const int32_t *__restrict__ part_offsets, const int32_t *__restrict__ seq_lens,
    const int32_t *__restrict__ dir, const uint16_t *__restrict__ q, int Hkv, int rows, int nsplit, int G, int Hq,
    int dir_stride, spin_step_args a) {
  constexpr int WAVES = 8, BLOCK = 64 * WAVES;
  __shared__ typename std::conditional<TILES, int, reg_row_lds<BLOCK>>::type s;
  __shared__ int32_t s_dir[RES_DIR_LDS];
  __shared__ int s_wave[WAVES];
  __shared__ int s_before[WAVES];
  extern __shared__ __align__(16) float smem[];       // the merge buffers of decode_finish, the token lists, the selection
  const step_place at = step_place_of(blockIdx.x, rows, nsplit);
  const int split = at.split, row = at.row, b = row / Hkv, h = row - b * Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, c = lane >> 4;
  uint32_t *tok = (uint32_t *)(smem + a.lists_at) + wave * STEP_TOK_LIST;
  spin_lds_i32 *l_sel = (spin_lds_i32 *)(smem + a.lists_at) + WAVES * STEP_TOK_LIST;

  const int32_t mydir = row_dir_entry(dir, dir_stride, row);
  const int N = max(seq_lens[b], 0);
  spin_bf16x8 qf[4];
  load_queries(qf, q, b, h, G, Hq, n, c);
  const lds_sel rsel = {a.sel_stride, l_sel};
  int take;
  if constexpr (TILES) {
    take = select_tiles_row<BLOCK, KPT, STEP_CAP, true>(scores, a.maxima, a.max_stride, a.gs_log, part_offsets, seq_lens, Hkv,
                                                        a.tp, a.topk, a.includes_forced, a.sink_pages, a.recent_pages, a.sel,
                                                        rsel, a.nsel, row, *(step_tiles_lds *)smem);
  } else {
    spin_var_span span;                               // (uniform partitions)
    take = select_reg_row<BLOCK, KPT>(scores, part_offsets, seq_lens, Hkv, a.tp, a.topk, a.includes_forced, a.sink_pages,
                                      a.recent_pages, rsel, a.nsel, row, spin_var{}, span, s, [] {});
  }
  if (tid < RES_DIR_LDS) s_dir[tid] = mydir;
  __syncthreads();                                    // the selection and the directory are whole

  const int tp_log = 31 - __clz(a.tp);                // 1, 2, 4 or 8 tokens
  const int32_t *rdir = dir + (size_t)row * dir_stride;
  auto page_of = [&](int i) { return l_sel[i] >> (4 - tp_log); };
  // the page's slot, -1 where it has none
  auto lookup = [&](int page) {
    const int ci = a.leaf_log >= 0 ? page >> a.leaf_log : page / a.leaf_entries;
    int32_t chunk = -1;
    if (ci < dir_stride) chunk = dir_stride <= RES_DIR_LDS ? ((spin_lds_i32 *)s_dir)[ci] : rdir[ci];
    const bool there = chunk >= 0 && (int64_t)chunk < a.leaf_chunks;
    const int32_t slot = a.leaf_pool[there ? (size_t)chunk * a.leaf_entries + (page - ci * a.leaf_entries) : 0];
    return there && slot >= 0 ? slot : -1;
  };

  // the selected tokens (the context's last partition may be short) in tiles; tile t goes to split t % nsplit, wavefront
  // (t / nsplit) % WAVES
  int T = take << tp_log;
  if (take > 0) T -= max((l_sel[take - 1] + 1) * a.tp - N, 0);
  const int ntiles = (T + 15) >> 4, first = wave * nsplit + split, stride = WAVES * nsplit;
  const int nt = ntiles > first ? (ntiles - first + stride - 1) / stride : 0;
  int32_t slot[STEP_TOK_ROUNDS];
  int token[STEP_TOK_ROUNDS];                         // -1: none
  auto ask = [&](int base) {
#pragma unroll
    for (int r = 0; r < STEP_TOK_ROUNDS; ++r) {
      slot[r] = -1;
      token[r] = -1;
      const int i = base + 4 * r + c, j = (first + i * stride) * 16 + n;
      if (base + 4 * r < nt) {                        // uniform
        const bool have = i < nt && j < T;
        const int t = (l_sel[have ? j >> tp_log : 0] << tp_log) + (j & (a.tp - 1));
        slot[r] = lookup(t >> 4);
        token[r] = have ? t : -1;
      }
    }
  };
  ask(0);

  // this workgroup's share of the selection: where its pages begin in the row's list
  const int per = (take + nsplit - 1) / nsplit, e0 = min(split * per, take), e1 = min(e0 + per, take);
  const int E = (e1 - e0 + BLOCK - 1) / BLOCK;        // entries per thread, in a row
  auto opens = [&](int i) { return i == 0 || page_of(i - 1) != page_of(i); };
  const int mine0 = e0 + tid * E, mine1 = min(mine0 + E, e1);
  int32_t page_slot = -1;
  if (E == 1 && mine0 < mine1) page_slot = lookup(page_of(mine0));
  int before = 0, opened = 0;
  for (int i = tid; i < e0; i += BLOCK) before += opens(i);
  for (int i = mine0; i < mine1; ++i) opened += opens(i);
  const int inc = spin_wave_inclusive_scan(opened), inc_before = spin_wave_inclusive_scan(before);
  if (lane == 63) {
    s_wave[wave] = inc;
    s_before[wave] = inc_before;
  }
  __syncthreads();
  int own, ahead;
  int pos = spin_waves_before<WAVES>(s_wave[lane % WAVES], wave, own) + inc - opened;
  (void)spin_waves_before<WAVES>(s_before[lane % WAVES], wave, ahead);
  pos += ahead;

  softmax_state st;
  softmax_reset(st);
  const res_out out = res_row_out(a.slots, a.page_ids, a.valid_mask, a.npages, row, a.page_stride);
  for (int base = 0; base == 0 || base < nt; base += 4 * STEP_TOK_ROUNDS) {
    if (base) ask(base);
    int total = 0;
    if (base == 0 && lane == 0) tok[0] = 0;           // without any token: a place inside the pool
#pragma unroll
    for (int r = 0; r < STEP_TOK_ROUNDS; ++r) {
      if (base + 4 * r >= nt) break;                  // uniform
      const bool inside = slot[r] >= 0 && (int64_t)slot[r] < a.pool_slots;
      if (token[r] >= 0 && !inside) spin_raise(a.status, slot[r] < 0 ? SPIN_ERR_NOT_RESIDENT : SPIN_ERR_SLOT_RANGE);
      const bool have = token[r] >= 0 && inside;      // the others are not attended
      const unsigned long long m = __ballot(have);
      const int at = total + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
      if (have) tok[at] = ((uint32_t)slot[r] << 4) | (uint32_t)(token[r] & 15);
      total += __popcll(m);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the wavefront reads its own list: program order
    attend_token_tiles<2>(st, a.pool, tok, total, lane, c, qf, a.scale_log2e, [&] {
      if (base) return;
      for (int i = mine0, at = pos; i < mine1; ++i) {
        if (!opens(i)) continue;
        const int page = page_of(i);
        uint32_t mask = 0;
        for (int j = i; j < take && page_of(j) == page; ++j) {
          const int t0 = l_sel[j] << tp_log;
          mask |= ((1u << min(a.tp, N - t0)) - 1u) << (t0 & 15);
        }
        const int32_t found = E == 1 ? page_slot : lookup(page);
        if (at < a.page_stride) out.put(at, found, page, found >= 0 ? mask : 0);
        ++at;
      }
      int32_t *rsel_out = a.sel + (size_t)row * a.sel_stride;
      for (int i = e0 + tid; i < e1; i += BLOCK) rsel_out[i] = l_sel[i];
      if (split == nsplit - 1) {                      // its share ends the selection
        const int np = min(ahead + own, a.page_stride);
        for (int i = take + tid; i < a.sel_stride; i += BLOCK) rsel_out[i] = -1;
        for (int i = np + tid; i < a.page_stride; i += BLOCK) out.put(i, -1, -1, 0);
        if (tid == 0) {
          a.nsel[row] = take;
          out.count(np);
        }
      }
    });
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // before the next batch overwrites the list
  }
  decode_finish<WAVES, false, true>(st, row, split, b, h, lane, wave, n, c, G, Hq, nsplit, nsplit, a.part_ml, a.part_acc,
                                    a.tickets, a.out, a.lse);
}

int spin_step_tokens_launch(spin_ctx *ctx, int32_t batch, const float *scores, const int32_t *part_offsets,
                            const int32_t *seq_lens, const int32_t *dir, const void *q, const spin_step_args &a, void *stream) {
  const spin_config &c = ctx->cfg;
  const int rows = batch * c.num_kv_heads;
#define SPIN_SDT_LAUNCH(KPT, TILES)                                                                               \
  spin_launch(ctx, SPIN_K_SELECT_DECODE, spin_select_decode_tokens_kernel<KPT, TILES>,                            \
              dim3((unsigned)(rows * ctx->fused_splits)), dim3(512), spin_fused_lds(ctx), (hipStream_t)stream,    \
              scores, part_offsets, seq_lens, dir, (const uint16_t *)q, c.num_kv_heads, rows,                     \
              ctx->fused_splits, ctx->group, c.num_q_heads, ctx->dir_stride, a)
  const int per_thread = spin_step_per_thread(ctx);
  if (ctx->step_tiles) {
    if (per_thread == 4) SPIN_SDT_LAUNCH(4, true);
    else if (per_thread == 8) SPIN_SDT_LAUNCH(8, true);
    else SPIN_SDT_LAUNCH(16, true);
  } else if (per_thread == 4) SPIN_SDT_LAUNCH(4, false);
  else if (per_thread == 8) SPIN_SDT_LAUNCH(8, false);
  else if (per_thread == 16) SPIN_SDT_LAUNCH(16, false);
  else SPIN_SDT_LAUNCH(32, false);
#undef SPIN_SDT_LAUNCH
  return spin_launch_status();
}
