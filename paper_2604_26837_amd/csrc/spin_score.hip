// Stage 1: score every partition of every row against the current query
// (Section 4.1, Select; Table 1, score(q, k_sums)).
//
// Each score kind is a contraction of a summary row with a query-derived
// vector, so a tile of 16 summary rows is one matrix-core tile
// S[head][row] = sum_k Q[head][k] * A[row][k]:
//   MINMAX  sum_d max(q*min, q*max) = sum_d ( max(q,0)*max_d + min(q,0)*min_d ),
//           i.e. the row [max | min] (256 elements) against [q+ | q-]; one of the
//           two products per channel is exactly zero, so nothing is added that
//           the definition does not add.  8 x (16x16x32) instructions.
//   REPMAX  representative . q over 128 channels, 4 x (16x16x32); then a
//           maximum over the partition's 4 rows.
//   SKETCH  16 sketched channels, 1 x (16x16x16).
// bf16 x bf16 products are exact in fp32; accumulation is fp32 inside the
// matrix core.  The queries are the first operand, so a lane holds one summary
// row's values for four heads and the maximum over the group's heads needs no
// exchange for groups of up to four heads (two otherwise).  Summary tiles are
// stored chunk-major so each load is a contiguous wavefront transaction.
#include "spin_score_dev.h"

#define SCORE_WAVES 4

template <int NJ, bool MINMAX, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void spin_score_k32_kernel(
    const uint16_t *__restrict__ q, const uint4 *__restrict__ summ, const int32_t *__restrict__ part_offsets,
    int Hq, int Hkv, int G, int rows_per_part, int tiles_per_wg, int wgs_per_row, float *__restrict__ scores,
    tile_maxima tm) {
  const int row = blockIdx.x / wgs_per_row, chunk = blockIdx.x - row * wgs_per_row;
  score_row_tiles<NJ, MINMAX, WAVES>(q, summ, part_offsets, Hq, Hkv, G, rows_per_part, tiles_per_wg, row, chunk,
                                     scores, tm);
}

template <int NJ, bool MINMAX, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void spin_score_k32_single_kernel(
    const uint16_t *__restrict__ q, const uint4 *__restrict__ summ, const int32_t *__restrict__ part_offsets,
    int Hq, int Hkv, int G, int rows_per_part, int tiles_per_wg, int wgs_per_row, float *__restrict__ scores,
    tile_maxima tm) {
  (void)tiles_per_wg;   // == WAVES
  const int row = blockIdx.x / wgs_per_row, chunk = blockIdx.x - row * wgs_per_row;
  score_row_single_tile<NJ, MINMAX, WAVES>(q, summ, part_offsets, Hq, Hkv, G, rows_per_part, row, chunk, scores, tm);
}

// SKETCH: one 16x16x16 instruction per tile of 16 tokens (512 bytes).  MAXIMA: tm.at is there (asked for at
// run time, it slows the loop: 16 rows of 16000 tokens, groups of 16, 10.0 -> 10.9 us).
template <bool MAXIMA>
__global__ __launch_bounds__(SCORE_WAVES * 64) void spin_score_sketch_kernel(
    const uint16_t *__restrict__ q, const uint2 *__restrict__ summ, const int32_t *__restrict__ chan,
    const int32_t *__restrict__ part_offsets, int Hq, int Hkv, int G, int tiles_per_wg, int wgs_per_row,
    float *__restrict__ scores, tile_maxima tm) {
  const int row = blockIdx.x / wgs_per_row, chunk = blockIdx.x - row * wgs_per_row;
  const int b = row / Hkv, h = row - b * Hkv;
  const int PP = part_offsets[b + 1] - part_offsets[b];
  const int ntiles = PP / 16;
  const int t_begin = chunk * tiles_per_wg;
  if (t_begin >= ntiles) return;
  const int t_end = min(t_begin + tiles_per_wg, ntiles);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = lane & 15, c = lane >> 4;
  const size_t base = (size_t)Hkv * part_offsets[b] + (size_t)h * PP;

  const uint2 *tiles = summ + base * 4;   // 16 elements = 4 units of 8 bytes per row
  constexpr int U = 8;
  // the first batch of tiles is requested before the query gather below (two dependent loads)
  // has to be waited for
  int t0 = t_begin + wave * U;
  uint2 a[U];
#pragma unroll
  for (int u = 0; u < U; ++u) a[u] = (t0 + u < t_end) ? spin_nt_load2(tiles + (size_t)(t0 + u) * 64 + lane) : make_uint2(0, 0);

  // A operand: row n = head, k = sketched channels 4c..4c+3
  spin_s16x4 qf;
  {
    const uint16_t *qrow = q + ((size_t)(b * Hq + h * G + (n < G ? n : 0))) * SPIN_HEAD_DIM;
    uint16_t e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i] = n < G ? qrow[chan[h * 16 + 4 * c + i]] : (uint16_t)0;
    uint2 pk = make_uint2(e[0] | ((uint32_t)e[1] << 16), e[2] | ((uint32_t)e[3] << 16));
    qf = __builtin_bit_cast(spin_s16x4, pk);
  }
  for (; t0 < t_end; t0 += SCORE_WAVES * U) {
    // the next batch is in flight while this one is consumed
    uint2 nx[U];
    const int t1 = t0 + SCORE_WAVES * U;
#pragma unroll
    for (int u = 0; u < U; ++u) nx[u] = (t1 + u < t_end) ? spin_nt_load2(tiles + (size_t)(t1 + u) * 64 + lane) : make_uint2(0, 0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (t0 + u >= t_end) break;
      spin_f32x4 s = {0.f, 0.f, 0.f, 0.f};
      s = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(qf, __builtin_bit_cast(spin_s16x4, a[u]), s, 0, 0, 0);
      const float m = spin_head_max(s, c, G);   // lane (n, c): heads 4c+i of token n
      if (c == 0) scores[base + (size_t)(t0 + u) * 16 + n] = m;
      if (MAXIMA) {
        const float top = spin_row16_max(m);
        if (lane == 0 && t0 + u < tm.stride) tm.at[(size_t)row * tm.stride + t0 + u] = top;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = nx[u];
  }
}

// SKETCH for groups of at most four query heads: 16 bytes per lane and load, four tiles of 16 tokens per accumulator.
// A load of a KiB covers two tiles; lane (n, c) takes channels 4c .. 4c+3 of tokens 2(n%8) and 2(n%8)+1 of tile n/8,
// and each half of it is the second operand of a 16x16x16 instruction whose columns are those 16 tokens of the two
// tiles.  The first operand of instruction j (load j/2, half j%2) holds the group's heads in rows 4j .. 4j+3 and
// zeros elsewhere (exact zero products), so the four instructions of two loads fill one accumulator: lane (n, c) ends
// up with the four heads' scores of one token, the maximum stays in the lane and all 64 lanes store.
// HBM bounds it (64 rows of 65536 tokens, 151 MB read and written: 27.5 us; 28.2 with 8-byte loads in the 16x16x32
// operand's image).
__global__ __launch_bounds__(SCORE_WAVES * 64) void spin_score_sketch4_kernel(
    const uint16_t *__restrict__ q, const uint4 *__restrict__ summ, const int32_t *__restrict__ chan,
    const int32_t *__restrict__ part_offsets, int Hq, int Hkv, int G, int tiles_per_wg, int wgs_per_row,
    float *__restrict__ scores, tile_maxima tm) {
  const int row = blockIdx.x / wgs_per_row, chunk = blockIdx.x - row * wgs_per_row;
  const int b = row / Hkv, h = row - b * Hkv;
  const int PP = part_offsets[b + 1] - part_offsets[b];
  const int ntiles = PP / 16;
  const int t_begin = chunk * tiles_per_wg;       // tiles_per_wg is a multiple of 4
  if (t_begin >= ntiles) return;
  const int t_end = min(t_begin + tiles_per_wg, ntiles);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = lane & 15, c = lane >> 4;
  const size_t base = (size_t)Hkv * part_offsets[b] + (size_t)h * PP;
  const uint4 *tiles = summ + base * 2;           // a tile: [channel quad (4)][token (16)][4 channels], 32 units of 16 bytes
  constexpr int U = 4;                            // groups of four tiles per wavefront and batch
  const int unit = c * 8 + (n & 7);
  struct group4 { uint4 ld[2]; };
  auto load_group = [&](group4 &g4, int t) {
#pragma unroll
    for (int i = 0; i < 2; ++i)                   // tiles past the end are clamped
      g4.ld[i] = spin_nt_load(tiles + (size_t)min(t + 2 * i + (n >> 3), t_end - 1) * 32 + unit);
  };
  int t0 = t_begin + wave * 4 * U;
  group4 cur[U];
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (t0 + 4 * u < t_end) load_group(cur[u], t0 + 4 * u);

  // first operands: lane (r, c) supplies row r = 4j + g, channels 4c .. 4c+3
  spin_s16x4 qa[4];
  {
    const int g = n & 3;
    uint32_t w[2] = {0u, 0u};
    if (g < G) {
      const uint16_t *qrow = q + ((size_t)(b * Hq + h * G + g)) * SPIN_HEAD_DIM;
#pragma unroll
      for (int e = 0; e < 4; e += 2)
        w[e >> 1] = (uint32_t)qrow[chan[h * 16 + 4 * c + e]] | ((uint32_t)qrow[chan[h * 16 + 4 * c + e + 1]] << 16);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      qa[j] = __builtin_bit_cast(spin_s16x4, (n >> 2) == j ? make_uint2(w[0], w[1]) : make_uint2(0u, 0u));
  }
  // the lane's token of the group of four tiles, and whether its tile exists
  const int tok = (c >> 1) * 32 + 2 * n + (c & 1), my_tile = 2 * (c >> 1) + (n >> 3);
  for (; t0 < t_end; t0 += SCORE_WAVES * 4 * U) {
    // the next batch is in flight while this one is consumed
    group4 nxt[U];
    const int t1 = t0 + SCORE_WAVES * 4 * U;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (t1 + 4 * u < t_end) load_group(nxt[u], t1 + 4 * u);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + 4 * u;
      if (t >= t_end) break;
      spin_f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint2 lo = make_uint2(cur[u].ld[i].x, cur[u].ld[i].y), hi = make_uint2(cur[u].ld[i].z, cur[u].ld[i].w);
        s = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(qa[2 * i], __builtin_bit_cast(spin_s16x4, lo), s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(qa[2 * i + 1], __builtin_bit_cast(spin_s16x4, hi), s, 0, 0, 0);
      }
      const float mx = spin_head_max(s, 0, G);    // heads 0..3 of the lane's token
      if (t + my_tile < t_end) scores[base + (size_t)t * 16 + tok] = mx;
      if (tm.at) {                                // uniform; a tile's tokens lie in 8 lanes of two lane rows
        float top = fmaxf(mx, spin_dpp<SPIN_DPP_XOR1>(mx));
        top = fmaxf(top, spin_dpp<SPIN_DPP_XOR2>(top));
        top = fmaxf(top, spin_dpp<SPIN_DPP_HALF_MIRROR>(top));
        top = fmaxf(top, __shfl_xor(top, 16));
        if ((n & 7) == 0 && !(c & 1) && t + my_tile < t_end && t + my_tile < tm.stride)
          tm.at[(size_t)row * tm.stride + t + my_tile] = top;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) cur[u] = nxt[u];
  }
}

int spin_score_impl(spin_ctx *ctx, int32_t batch, const void *q, const void *summaries, const int32_t *chan_idx,
                    const int32_t *part_offsets, const int32_t *seq_lens, float *scores, void *workspace,
                    void *stream, float *maxima) {
  if (!ctx || batch < 0 || batch > ctx->cfg.max_batch) return SPIN_ERR_INVALID;
  if (batch == 0) return SPIN_OK;
  if (!q || !summaries || !part_offsets || !seq_lens || !scores) return SPIN_ERR_INVALID;
  (void)workspace;
  const spin_config &c = ctx->cfg;
  const int rows = batch * c.num_kv_heads;
  const int max_pp = ((ctx->max_parts + 15) / 16) * 16;
  hipStream_t st = (hipStream_t)stream;
  const int W = c.score_waves ? c.score_waves : 4;
  const tile_maxima tm = {maxima, ctx->max_stride};
  if (c.score_kind == SPIN_SCORE_MINMAX) {
    // one tile per wavefront measured best: the dispatcher streams the workgroups
    const int tiles_per_wg = c.score_tiles_per_wg ? c.score_tiles_per_wg : W, max_tiles = max_pp / 16;
    const int wgs = (max_tiles + tiles_per_wg - 1) / tiles_per_wg;
#define SPIN_SCORE_ARGS(RPP)                                                                                  \
  0, st, (const uint16_t *)q, (const uint4 *)summaries, part_offsets, c.num_q_heads, c.num_kv_heads, ctx->group, \
      RPP, tiles_per_wg, wgs, scores, tm
    if (W == 2 && tiles_per_wg == 2)
      spin_launch(ctx, SPIN_K_SCORE, spin_score_k32_single_kernel<8, true, 2>, dim3((unsigned)rows * wgs), dim3(128),
                  SPIN_SCORE_ARGS(1));
    else if (W == 1 && tiles_per_wg == 1)
      spin_launch(ctx, SPIN_K_SCORE, spin_score_k32_single_kernel<8, true, 1>, dim3((unsigned)rows * wgs), dim3(64),
                  SPIN_SCORE_ARGS(1));
    else if (W == 8 && tiles_per_wg == 8)
      spin_launch(ctx, SPIN_K_SCORE, spin_score_k32_single_kernel<8, true, 8>, dim3((unsigned)rows * wgs), dim3(512),
                  SPIN_SCORE_ARGS(1));
    else if (W == 8)
      spin_launch(ctx, SPIN_K_SCORE, spin_score_k32_kernel<8, true, 8>, dim3((unsigned)rows * wgs), dim3(512),
                  SPIN_SCORE_ARGS(1));
    else if (tiles_per_wg == 4)
      spin_launch(ctx, SPIN_K_SCORE, spin_score_k32_single_kernel<8, true, 4>, dim3((unsigned)rows * wgs), dim3(256),
                  SPIN_SCORE_ARGS(1));
    else
      spin_launch(ctx, SPIN_K_SCORE, spin_score_k32_kernel<8, true, 4>, dim3((unsigned)rows * wgs), dim3(256),
                  SPIN_SCORE_ARGS(1));
  } else if (c.score_kind == SPIN_SCORE_REPMAX) {
    const int R = c.reps_per_partition;
    const int tiles_per_wg = c.score_tiles_per_wg ? c.score_tiles_per_wg : 2 * W, max_tiles = max_pp * R / 16;
    const int wgs = (max_tiles + tiles_per_wg - 1) / tiles_per_wg;
    if (W == 8)
      spin_launch(ctx, SPIN_K_SCORE, spin_score_k32_kernel<4, false, 8>, dim3((unsigned)rows * wgs), dim3(512),
                  SPIN_SCORE_ARGS(R));
    else
      spin_launch(ctx, SPIN_K_SCORE, spin_score_k32_kernel<4, false, 4>, dim3((unsigned)rows * wgs), dim3(256),
                  SPIN_SCORE_ARGS(R));
#undef SPIN_SCORE_ARGS
  } else {
    if (!chan_idx) return SPIN_ERR_INVALID;
    // groups of up to four heads: the four-tile kernel, 256 tiles per workgroup measured best (32 / 64 /
    // 128 / 256 / 512: 28.9 / 27.7 / 28.1 / 27.4 / 28.7 us on 64 rows of 65536 tokens)
    const bool four = ctx->group <= 4 && (c.score_tiles_per_wg % 4) == 0;
    const int tiles_per_wg = c.score_tiles_per_wg ? c.score_tiles_per_wg : (four ? 256 : 128), max_tiles = max_pp / 16;
    const int wgs = (max_tiles + tiles_per_wg - 1) / tiles_per_wg;
#define SPIN_SKETCH_ARGS(UNIT)                                                                                   \
  dim3((unsigned)rows * wgs), dim3(SCORE_WAVES * 64), 0, st, (const uint16_t *)q, (const UNIT *)summaries, chan_idx, \
      part_offsets, c.num_q_heads, c.num_kv_heads, ctx->group, tiles_per_wg, wgs, scores, tm
    if (four) spin_launch(ctx, SPIN_K_SCORE, spin_score_sketch4_kernel, SPIN_SKETCH_ARGS(uint4));
    else if (maxima) spin_launch(ctx, SPIN_K_SCORE, spin_score_sketch_kernel<true>, SPIN_SKETCH_ARGS(uint2));
    else spin_launch(ctx, SPIN_K_SCORE, spin_score_sketch_kernel<false>, SPIN_SKETCH_ARGS(uint2));
#undef SPIN_SKETCH_ARGS
  }
  return spin_launch_status();
}

extern "C" int spin_score_partitions(spin_ctx *ctx, int32_t batch, const void *q, const void *summaries,
                                     const int32_t *chan_idx, const int32_t *part_offsets,
                                     const int32_t *seq_lens, float *scores, void *workspace, void *stream) {
  return spin_score_impl(ctx, batch, q, summaries, chan_idx, part_offsets, seq_lens, scores, workspace, stream, nullptr);
}
