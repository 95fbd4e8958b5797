// Stage 4: paged GQA decode attention over the resolved pages of each row
// (Section 4.1, Attention: standard attention restricted to the selected KV).
//
// One workgroup = one (row, split) pair; its wavefronts are dealt the split's
// pages round-robin.  Per page a wavefront issues eight contiguous 1 KiB loads
// (K tile then V tile of the slot), forms the 16 x 16 logit tile
// S[token][head] = K Q^T with four 16x16x32 bf16 matrix instructions (the
// group's G <= 16 query heads padded to 16 columns), runs the online softmax
// on its four logits per lane, and accumulates O[head][dim] += P V with eight
// 16x16x16 instructions; the logit tile's register layout is exactly the
// operand layout of P, so nothing moves between lanes except two max
// exchanges.  Two pages are under way while one is consumed (two register
// buffers, each asked for again as soon as it has been read, in a loop without
// branches so that the compiler's waits name exactly the tile that is needed;
// with a branch around every load they covered the page just asked for as
// well: stage 4 of 128 rows of 116 pages 25.1 -> 24.7 us, of 32 rows of 324
// pages 19.0 -> 17.5, of 96 rows of 116 pages 21.4 -> 20.7).  A wavefront
// fetches the slot ids and masks of its pages with one load up front, together
// with the queries and the row's counts, so the only dependent memory round
// trips per wavefront are that one and the first page.
//
// Wavefront partials (m, l, O) are merged through LDS in wave order.  With
// more than one split the workgroup partials go to the workspace and the
// last workgroup of the row to arrive (a ticket counter in the workspace
// header) merges them in split order, so results are reproducible.
#include <mutex>

#include "spin_token_tiles_dev.h"

template <int WAVES, int DEPTH>
__global__ __launch_bounds__(WAVES * 64) void spin_decode_kernel(
    const uint16_t *__restrict__ q, const uint4 *__restrict__ pool, int64_t pool_slots,
    const int32_t *__restrict__ slots, const uint16_t *__restrict__ masks,
    const int32_t *__restrict__ npages, int page_stride, int G, int Hq, int Hkv, int nsplit, int pstride,
    const int32_t *__restrict__ skip, int mode, int nside, float scale_log2e, float *part_ml, float *part_acc, int32_t *tickets,
    uint16_t *__restrict__ out, float *__restrict__ lse, int32_t *status) {
  const int row = blockIdx.x / nsplit;
  decode_row<WAVES, DEPTH>(row, blockIdx.x - row * nsplit, q, pool, pool_slots, slots, masks, npages, page_stride, G, Hq, Hkv,
                           nsplit, pstride, skip, mode, nside, scale_log2e, part_ml, part_acc, tickets, out, lse, status,
                           [](int, unsigned mask) { return mask; });
}

// ---------------------------------------------------------------------------
// Partitions smaller than a page (token-major slots): most attended pages hold one or two
// attended tokens, so a tile is not a physical page but 16 ATTENDED tokens gathered from
// wherever they live.  A wavefront expands the masks of its pages (dealt round-robin exactly as
// above) into a token list in LDS -- page order, then token order, so the accumulation order is
// fixed -- and then treats every 16 list entries as one tile: lane (n, c) fetches 64 contiguous
// bytes of the key of tile row n per load, and 16 bytes of each of the value rows 4c .. 4c+3, which
// it transposes in registers into the operands of P V (a lane's output channels then are 8n .. 8n+7,
// eight neighbours, where the page kernel's are 16 apart).  The gather of 256-byte rows bounds this.
// Against 2-byte loads straight into the operands (32 a tile, whose packing waited for all of them
// before the next tile was asked for), whole steps, us: 64 rows of 65536 tokens, 1024 attended
// 54.5 -> 53.7; 96 rows, 2048 attended 91.9 -> 90.3; 8 rows, 2048 attended 41.9 -> 41.1; 16 rows of
// 8003, 300 attended 21.6 -> 21.3.  Three tiles under way are worse than two (55.0 / 91.3 / 41.4 /
// 21.6 us), keys and values read with the same hint as well (nt 54.9 us, none 93.9 in the second).  Per
// attended token that is the algorithmic 512 bytes (two cache lines of K, two of V) instead of
// the page's 8 KiB, and sixteen times fewer matrix tiles.  Logits, softmax and merge are the
// code of the page kernel.
#define TOK_LIST 1024   // list entries per wavefront and batch of 64 pages

template <int WAVES>
__global__ __launch_bounds__(WAVES * 64) void spin_decode_tokens_kernel(
    const uint16_t *__restrict__ q, const uint4 *__restrict__ pool, int64_t pool_slots,
    const int32_t *__restrict__ slots, const uint16_t *__restrict__ masks,
    const int32_t *__restrict__ npages, int page_stride, int G, int Hq, int Hkv, int nsplit, int pstride,
    const int32_t *__restrict__ skip, float scale_log2e, float *part_ml, float *part_acc, int32_t *tickets,
    uint16_t *__restrict__ out, float *__restrict__ lse, int32_t *status) {
  extern __shared__ __align__(16) float smem[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the token lists live behind the merge buffers of decode_finish
  uint32_t *tok = (uint32_t *)(smem + WAVES * G * (SPIN_HEAD_DIM + 2)) + wave * TOK_LIST;

  const int row = blockIdx.x / nsplit;
  const int split = blockIdx.x - row * nsplit;
  const int lane = threadIdx.x & 63;
  const int n = lane & 15, c = lane >> 4;
  const int b = row / Hkv;
  const int h = row - b * Hkv;
  const int32_t *rslots = slots + (size_t)row * page_stride;
  const uint16_t *rmask = masks + (size_t)row * page_stride;
  const int first = wave * nsplit + split, stride = WAVES * nsplit;
  int np = npages[row];
  np = np < 0 ? 0 : (np > page_stride ? page_stride : np);

  // this wavefront's pages: first + i * stride, i < nw; the entries of the first 64 are asked for ahead of all else
  int p = first + lane * stride;
  int next_slot = rslots[min(p, page_stride - 1)];
  unsigned next_mask = rmask[min(p, page_stride - 1)];
  spin_bf16x8 qf[4];
  load_queries(qf, q, b, h, G, Hq, n, c);
  softmax_state st;
  softmax_reset(st);

  const int nw = np > first ? (np - first + stride - 1) / stride : 0;
  for (int base = 0; base < nw; base += 64) {
    int myslot = 0;
    unsigned mymask = 0;
    if (base + lane < nw) {
      if (next_slot < 0 || (int64_t)next_slot >= pool_slots) {
        spin_raise(status, SPIN_ERR_SLOT_RANGE);
      } else {
        myslot = next_slot;
        mymask = next_mask;
      }
    }
    p += 64 * stride;
    if (base + 64 < nw) {
      next_slot = rslots[min(p, page_stride - 1)];
      next_mask = rmask[min(p, page_stride - 1)];
    }
    // token list of this batch of pages: page order, then token order
    const int mine = __popc(mymask);
    const int incl = spin_wave_inclusive_scan(mine);
    const int total = __builtin_amdgcn_readlane(incl, 63);
    {
      int pos = incl - mine;
      unsigned m = mymask;
      while (m) {
        const int t = __ffs(m) - 1;
        m &= m - 1;
        tok[pos++] = ((uint32_t)myslot << 4) | (uint32_t)t;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the wavefront reads its own list: program order
    if (total > 0) attend_token_tiles<2>(st, pool, tok, total, lane, c, qf, scale_log2e, [] {});
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // before the next batch overwrites the list
  }
  __syncthreads();   // the merge buffers are separate from the lists, but keep the phases apart
  decode_finish<WAVES, false, true>(st, row, split, b, h, lane, wave, n, c, G, Hq, nsplit, pstride, part_ml, part_acc,
                                    tickets, out, lse);
}

// Host side of stage 4: checks, then the launch; the split-K scratch (row tickets, (m, l) pairs and
// accumulators of the workgroup partials) and the status word are handed in by the two entry points.
// skip != NULL: the row's always-attended pages were attended by the launch of stages 2+3, whose partial sits
// behind the splits' partials and whose list positions are named in skip[row][2].
int decode_launch(spin_ctx *ctx, int32_t batch, const void *q, const void *kv_pool, int64_t pool_slots,
                  const int32_t *slots, const uint16_t *valid_mask, const int32_t *npages, void *out, float *lse,
                  float *part_ml, float *part_acc, int32_t *tickets, int32_t *status, const int32_t *skip, int mode,
                  int nside, void *stream) {
  const int rows = batch * ctx->cfg.num_kv_heads;
  const int G = ctx->group, nsplit = ctx->splits;
  const int pstride = ctx->pstride;
  const float scale_log2e = ctx->scale * 1.4426950408889634f;
  const int W = ctx->waves;
  const size_t lds = (size_t)W * G * (SPIN_HEAD_DIM + 2) * sizeof(float);
  if (ctx->k_token_major) {
    if (mode) return SPIN_ERR_UNSUPPORTED;   // the gathered-token kernel runs whole rows only
    // token-major slots: tiles of gathered tokens (always 8 wavefronts: the waves and depth knobs do not
    // apply, and the merge buffers are sized for 8 whatever the waves knob says)
    const size_t lds_tok = (size_t)8 * G * (SPIN_HEAD_DIM + 2) * sizeof(float) + (size_t)8 * TOK_LIST * sizeof(uint32_t);
    spin_launch(ctx, SPIN_K_DECODE, spin_decode_tokens_kernel<8>, dim3((unsigned)(rows * nsplit)), dim3(512), lds_tok,
                (hipStream_t)stream, (const uint16_t *)q, (const uint4 *)kv_pool, pool_slots, slots, valid_mask, npages,
                ctx->page_stride, G, ctx->cfg.num_q_heads, ctx->cfg.num_kv_heads, nsplit, pstride, skip, scale_log2e,
                part_ml, part_acc, tickets, (uint16_t *)out, lse, status);
    return spin_launch_status();
  }
#define SPIN_DECODE_LAUNCH2(WV, DP)                                                                              \
  spin_launch(ctx, SPIN_K_DECODE, spin_decode_kernel<WV, DP>, dim3((unsigned)(rows * nsplit)), dim3(WV * 64), lds, \
              (hipStream_t)stream, (const uint16_t *)q, (const uint4 *)kv_pool, pool_slots, slots, valid_mask,   \
              npages, ctx->page_stride, G, ctx->cfg.num_q_heads, ctx->cfg.num_kv_heads, nsplit, pstride, skip,   \
              mode, nside, scale_log2e, part_ml, part_acc, tickets, (uint16_t *)out, lse, status)
#define SPIN_DECODE_LAUNCH(WV)                          \
  do {                                                  \
    if (ctx->depth == 2) SPIN_DECODE_LAUNCH2(WV, 2);    \
    else if (ctx->depth == 4) SPIN_DECODE_LAUNCH2(WV, 4); \
    else SPIN_DECODE_LAUNCH2(WV, 3);                    \
  } while (0)
  if (W == 2) SPIN_DECODE_LAUNCH(2);
  else if (W == 8) SPIN_DECODE_LAUNCH(8);
  else SPIN_DECODE_LAUNCH(4);
#undef SPIN_DECODE_LAUNCH
#undef SPIN_DECODE_LAUNCH2
  return spin_launch_status();
}

extern "C" int spin_sparse_decode(spin_ctx *ctx, int32_t batch, const void *q, const void *kv_pool,
                                  int64_t pool_slots, const int32_t *slots, const uint16_t *valid_mask,
                                  const int32_t *npages, void *out, float *lse, void *workspace,
                                  void *stream) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch || pool_slots <= 0) return SPIN_ERR_INVALID;
  if (batch == 0) return SPIN_OK;
  if (!q || !kv_pool || !slots || !valid_mask || !npages || !out) return SPIN_ERR_INVALID;
  if (!workspace) return SPIN_ERR_WORKSPACE;
  char *ws = (char *)workspace;
  return decode_launch(ctx, batch, q, kv_pool, pool_slots, slots, valid_mask, npages, out, lse,
                       (float *)(ws + ctx->ws_ml_off), (float *)(ws + ctx->ws_acc_off),
                       (int32_t *)(ws + ctx->ws_ticket_off), (int32_t *)workspace, nullptr, 0, 0, stream);
}

// Attention in two passes over one page list: the first attends the tokens its masks name and leaves
// the row's merged partial (m, l, O) in the workspace, the second starts from it.
static int decode_two_pass(spin_ctx *ctx, int32_t batch, const void *q, const void *kv_pool, int64_t pool_slots,
                           const int32_t *slots, const uint16_t *valid_mask, const int32_t *npages, void *out,
                           float *lse, void *workspace, int mode, void *stream) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch || pool_slots <= 0) return SPIN_ERR_INVALID;
  if (ctx->k_token_major) return SPIN_ERR_UNSUPPORTED;
  if (batch == 0) return SPIN_OK;
  if (!q || !kv_pool || !slots || !valid_mask || !npages || (!out && !(mode & SPIN_DECODE_TO_PARTIAL)))
    return SPIN_ERR_INVALID;
  if (!workspace) return SPIN_ERR_WORKSPACE;
  char *ws = (char *)workspace;
  return decode_launch(ctx, batch, q, kv_pool, pool_slots, slots, valid_mask, npages, out, lse,
                       (float *)(ws + ctx->ws_ml_off), (float *)(ws + ctx->ws_acc_off),
                       (int32_t *)(ws + ctx->ws_ticket_off), (int32_t *)workspace, nullptr, mode, 1, stream);
}

extern "C" int spin_sparse_decode_begin(spin_ctx *ctx, int32_t batch, const void *q, const void *kv_pool,
                                        int64_t pool_slots, const int32_t *slots, const uint16_t *valid_mask,
                                        const int32_t *npages, void *workspace, void *stream) {
  return decode_two_pass(ctx, batch, q, kv_pool, pool_slots, slots, valid_mask, npages, nullptr, nullptr, workspace,
                         SPIN_DECODE_TO_PARTIAL, stream);
}

extern "C" int spin_sparse_decode_finish(spin_ctx *ctx, int32_t batch, const void *q, const void *kv_pool,
                                         int64_t pool_slots, const int32_t *slots, const uint16_t *valid_mask,
                                         const int32_t *npages, void *out, float *lse, void *workspace,
                                         void *stream) {
  return decode_two_pass(ctx, batch, q, kv_pool, pool_slots, slots, valid_mask, npages, out, lse, workspace,
                         SPIN_DECODE_FROM_PARTIAL, stream);
}

// Stage 4 over what spin_select_resolve_forced left: the pages other than the always-attended ones, merged
// with the partial that launch stored for them.
extern "C" int spin_sparse_decode_rest(spin_ctx *ctx, int32_t batch, const void *q, const void *kv_pool,
                                       int64_t pool_slots, const int32_t *slots, const uint16_t *valid_mask,
                                       const int32_t *npages, void *out, float *lse, void *workspace,
                                       void *stream) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch || pool_slots <= 0) return SPIN_ERR_INVALID;
  if (!spin_forced_split_supported(ctx)) return SPIN_ERR_UNSUPPORTED;
  if (batch == 0) return SPIN_OK;
  if (!q || !kv_pool || !slots || !valid_mask || !npages || !out) return SPIN_ERR_INVALID;
  if (!workspace) return SPIN_ERR_WORKSPACE;
  char *ws = (char *)workspace;
  return decode_launch(ctx, batch, q, kv_pool, pool_slots, slots, valid_mask, npages, out, lse,
                       (float *)(ws + ctx->ws_ml_off), (float *)(ws + ctx->ws_acc_off),
                       (int32_t *)(ws + ctx->ws_ticket_off), (int32_t *)workspace,
                       (const int32_t *)(ws + ctx->ws_skip_off), SPIN_DECODE_FROM_PARTIAL, ctx->side_wgs, stream);
}

// ---------------------------------------------------------------------------
// Stage 4 for callers that cannot hand over (or allocate) a workspace: the split-K scratch lives in
// a device array of the library itself.  Every GPU the library runs on holds its own copy of the
// array, at its own address, until the process ends.
#define SPIN_STATIC_SCRATCH_DEVICES 64
static __device__ __align__(256) unsigned char scratch[SPIN_STATIC_SCRATCH_BYTES];

// `scratch` above is only a host-side handle in host code: the device address is asked for once per
// device (with that device current) and kept; host code uses that address and never the symbol's name.
static void *g_scratch_ptr[SPIN_STATIC_SCRATCH_DEVICES];
static std::mutex g_scratch_mutex;

static int static_scratch(void **ptr) {
  int dev = -1;
  SPIN_HIP_CHECK(hipGetDevice(&dev));
  if (dev < 0 || dev >= SPIN_STATIC_SCRATCH_DEVICES) return SPIN_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    SPIN_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return SPIN_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return SPIN_OK;
}

int spin_static_scratch_prepare(void) {
  void *p = nullptr;
  return static_scratch(&p);
}

// clears the words that must be zero when the attention kernel starts (a kernel, not a memset, so
// that a caller may record the call into a HIP graph)
__global__ void spin_static_clear_kernel(int32_t *p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

extern "C" int spin_sparse_decode_static(spin_ctx *ctx, int32_t batch, const void *q, const void *kv_pool,
                                         int64_t pool_slots, const int32_t *slots, const uint16_t *valid_mask,
                                         const int32_t *npages, void *out, float *lse, int32_t *status,
                                         void *stream) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch || pool_slots <= 0) return SPIN_ERR_INVALID;
  if (batch == 0) return SPIN_OK;
  if (!q || !kv_pool || !slots || !valid_mask || !npages || !out) return SPIN_ERR_INVALID;
  // layout inside the array, sized for this call's rows: [status word, 256 B][tickets][(m, l)][accumulators]
  const size_t rows = (size_t)batch * ctx->cfg.num_kv_heads;
  const size_t partials = rows * ctx->pstride * ctx->group;   // the layout of the workspace (spare partials are not used here)
  const size_t ticket_off = SPIN_WS_HEADER;
  const size_t ml_off = (ticket_off + rows * sizeof(int32_t) + 255) & ~(size_t)255;
  const size_t acc_off = (ml_off + partials * 2 * sizeof(float) + 255) & ~(size_t)255;
  const size_t need = acc_off + partials * SPIN_HEAD_DIM * sizeof(float);
  if (need > SPIN_STATIC_SCRATCH_BYTES) return SPIN_ERR_STATIC_LIMIT;
  void *base = nullptr;
  const int rc = static_scratch(&base);
  if (rc != SPIN_OK) return rc;
  char *sc = (char *)base;
  // the array keeps the last call's contents: the status word and the row tickets start at zero
  const int nclear = (int)(ml_off / sizeof(int32_t));
  hipLaunchKernelGGL(spin_static_clear_kernel, dim3((nclear + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                     (int32_t *)sc, nclear);
  if (hipGetLastError() != hipSuccess) return SPIN_ERR_HIP;
  return decode_launch(ctx, batch, q, kv_pool, pool_slots, slots, valid_mask, npages, out, lse,
                       (float *)(sc + ml_off), (float *)(sc + acc_off), (int32_t *)(sc + ticket_off),
                       status ? status : (int32_t *)sc, nullptr, 0, 0, stream);
}
