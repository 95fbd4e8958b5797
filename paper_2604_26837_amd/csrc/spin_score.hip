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
#include <algorithm>

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

// SKETCH: where a row's scores begin, how many it has, and channels 4c .. 4c+3 of its KV head's sixteen.  Scalar loads, all
// under way together: the channels do not keep the tiles waiting.
struct sketch_row {
  int off, PP, ch[4];
};
__device__ __forceinline__ sketch_row sketch_row_of(const int32_t *__restrict__ chan, const int32_t *__restrict__ part_offsets,
                                                    int b, int h, int c) {
  int ch[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) ch[i] = chan[h * 16 + i];
  const int off = part_offsets[b], end = part_offsets[b + 1];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 16; ++i) ch[i] = __builtin_amdgcn_readfirstlane(ch[i]);
  sketch_row r = {off, end - off, {}};
#pragma unroll
  for (int i = 0; i < 4; ++i) r.ch[i] = c < 2 ? (c == 0 ? ch[i] : ch[4 + i]) : (c == 2 ? ch[8 + i] : ch[12 + i]);
  return r;
}

// SKETCH, groups of more than four heads: one 16x16x16 instruction per 16 tokens, 16 bytes per lane and load.  A load of a
// KiB covers two tiles; lane (n, c) takes channels 4c .. 4c+3 of tokens 2(n%8) and 2(n%8)+1 of tile n/8, and each half
// of it is the second operand of an instruction whose columns are those 16 tokens of the two tiles.  Rows of heads that
// the group does not have start from -inf instead of zero, so that the maximum needs no test per head; over the lane
// quarters it is taken of both halves at once, after which quarters 0 and 2 store 32 neighbouring scores.
// A wavefront asks for its 16 tiles at once (ONE), no load and no store is behind a branch (see spin_buffer); tiles past
// the last are beyond the buffer by the lane's own offset.  MAXIMA: tm.at is there (asked for at run time, it slowed the
// loop).
// 64 rows of 65536 tokens, groups of 8: 33.3 -> 25.4 us; 16 rows of 16000, groups of 16: 10.3 -> 3.5; 32 rows of 30000,
// groups of 5: 12.4 -> 6.2; against 8-byte loads behind branches, two exchanges through LDS per tile and one tile's
// 16 scores per store.
template <bool MAXIMA, bool ONE>
__global__ __launch_bounds__(SCORE_WAVES * 64) void spin_score_sketch_kernel(
    const uint16_t *__restrict__ q, const uint4 *__restrict__ summ, const int32_t *__restrict__ chan,
    const int32_t *__restrict__ part_offsets, int Hkv, int G, int tiles_per_wg, int b0, int h0,
    float *__restrict__ scores, tile_maxima tm) {
  const int chunk = blockIdx.x, b = b0 + blockIdx.z, h = h0 + blockIdx.y, row = b * Hkv + h;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, c = lane >> 4;
  const sketch_row sr = sketch_row_of(chan, part_offsets, b, h, c);
  const int ntiles = sr.PP / 16;
  const int t_begin = chunk * tiles_per_wg;
  if (t_begin >= ntiles) return;
  const int t_end = min(t_begin + tiles_per_wg, ntiles);
  const size_t base = (size_t)Hkv * sr.off + (size_t)h * sr.PP;
  constexpr int U = 8;                            // pairs of tiles per wavefront and round
  constexpr int ROUND = SCORE_WAVES * 2 * U;
  const uint16_t *qrow = q + ((size_t)(row * G + min(n, G - 1))) * SPIN_HEAD_DIM;
  uint32_t e[4];                                  // asked for ahead of the tiles
#pragma unroll
  for (int i = 0; i < 4; ++i) e[i] = qrow[sr.ch[i]];
  // the workgroup's tiles, 512 bytes each; their scores and maxima
  const __amdgpu_buffer_rsrc_t in = spin_buffer(summ + base * 2 + (size_t)t_begin * 32, (uint32_t)(t_end - t_begin) * 512);
  const __amdgpu_buffer_rsrc_t out = spin_buffer(scores + base + (size_t)t_begin * 16, (uint32_t)(t_end - t_begin) * 64);
  const __amdgpu_buffer_rsrc_t top_out =
      spin_buffer(MAXIMA ? tm.at + (size_t)row * tm.stride + t_begin : nullptr,
                  MAXIMA ? (uint32_t)max(min(t_end, tm.stride) - t_begin, 0) * 4 : 0);
  uint32_t at_in = (uint32_t)(wave * 2 * U + (n >> 3)) * 512 + (uint32_t)(c * 8 + (n & 7)) * 16;
  uint32_t at_out = c & 1 ? 0x80000000u : (uint32_t)((wave * 2 * U + (n >> 3)) * 16 + 2 * (n & 7) + (c >> 1)) * 4;
  uint32_t at_top = (n & 7) || c ? 0x80000000u : (uint32_t)(wave * 2 * U + (n >> 3)) * 4;
  uint4 ld[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    ld[u] = spin_buffer_load(in, at_in + 2 * u * 512, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
  // A operand: row n = head, k = sketched channels 4c..4c+3
  const spin_s16x4 qf =
      __builtin_bit_cast(spin_s16x4, n < G ? make_uint2(e[0] | (e[1] << 16), e[2] | (e[3] << 16)) : make_uint2(0u, 0u));
  spin_f32x4 start;
#pragma unroll
  for (int i = 0; i < 4; ++i) start[i] = 4 * c + i < G ? 0.f : -__builtin_inff();
  for (int t0 = t_begin + wave * 2 * U; t0 < t_end; t0 += ROUND) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint2 lo = make_uint2(ld[u].x, ld[u].y), hi = make_uint2(ld[u].z, ld[u].w);
      const spin_f32x4 s0 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(qf, __builtin_bit_cast(spin_s16x4, lo), start, 0, 0, 0);
      const spin_f32x4 s1 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(qf, __builtin_bit_cast(spin_s16x4, hi), start, 0, 0, 0);
      if (!ONE) ld[u] = spin_buffer_load(in, at_in + (ROUND + 2 * u) * 512, 0);
      const float m0 = fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[2], s0[3]));
      const float m1 = fmaxf(fmaxf(s1[0], s1[1]), fmaxf(s1[2], s1[3]));
      float m = spin_max_xor16(spin_max_xor32(m0, m1));
      m = fmaxf(m, -__builtin_inff());            // (NaN in every head: -inf)
      spin_buffer_store(out, at_out + 2 * u * 64, m);
      if (MAXIMA) {                               // a tile's tokens lie in the 8 lanes of both halves
        float top = fmaxf(m, spin_dpp<SPIN_DPP_XOR1>(m));
        top = fmaxf(top, spin_dpp<SPIN_DPP_XOR2>(top));
        top = fmaxf(top, spin_dpp<SPIN_DPP_HALF_MIRROR>(top));
        spin_buffer_store(top_out, at_top + 2 * u * 4, spin_max_xor32(top));
      }
    }
    if (ONE) break;
    at_in += ROUND * 512;
    at_out += ROUND * 64;
    at_top += ROUND * 4;
  }
}

// SKETCH for groups of at most four query heads: 16 bytes per lane and load, four tiles of 16 tokens per accumulator.
// A load of a KiB covers two tiles; lane (n, c) takes channels 4c .. 4c+3 of tokens 2(n%8) and 2(n%8)+1 of tile n/8,
// and each half of it is the second operand of a 16x16x16 instruction whose columns are those 16 tokens of the two
// tiles.  The first operand of instruction j (load j/2, half j%2) holds the group's heads in rows 4j .. 4j+3 and
// zeros elsewhere (exact zero products), so the four instructions of two loads fill one accumulator: lane (n, c) ends
// up with the four heads' scores of one token, the maximum stays in the lane and all 64 lanes store.
// HBM bounds it.  A wavefront asks for its 16 tiles (8 KiB) at once, behind the group's channels and queries, and has no
// second round (ONE); with more tiles to a workgroup a group's registers are asked for again as soon as they have been
// consumed.  No load and no store is behind a branch (see spin_buffer).  64 rows of 65536 tokens, 151 MB read and
// written: 25.6 us in one round, 26.4 in four; 27.1 with four rounds whose loads, behind branches, were waited for as
// soon as they were issued.
// MAXIMA: tm.at is there.
template <bool MAXIMA, bool ONE>
__global__ __launch_bounds__(SCORE_WAVES * 64) void spin_score_sketch4_kernel(
    const uint16_t *__restrict__ q, const uint4 *__restrict__ summ, const int32_t *__restrict__ chan,
    const int32_t *__restrict__ part_offsets, int Hkv, int G, int tiles_per_wg, int b0, int h0,
    float *__restrict__ scores, tile_maxima tm) {
  const int chunk = blockIdx.x, b = b0 + blockIdx.z, h = h0 + blockIdx.y, row = b * Hkv + h;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, c = lane >> 4;
  const sketch_row sr = sketch_row_of(chan, part_offsets, b, h, c);
  const int ntiles = sr.PP / 16;
  const int t_begin = chunk * tiles_per_wg;       // tiles_per_wg is a multiple of 4
  if (t_begin >= ntiles) return;
  const int t_end = min(t_begin + tiles_per_wg, ntiles);
  const size_t base = (size_t)Hkv * sr.off + (size_t)h * sr.PP;
  constexpr int U = 4;                            // groups of four tiles per wavefront and round
  constexpr int ROUND = SCORE_WAVES * 4 * U;

  // first operands: lane (r, c) supplies row r = 4j + g, channels 4c .. 4c+3; asked for ahead of the tiles
  const uint16_t *qrow = q + ((size_t)(row * G + min(n & 3, G - 1))) * SPIN_HEAD_DIM;
  uint32_t e[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) e[i] = qrow[sr.ch[i]];
  // the workgroup's tiles, a tile being [channel quad (4)][token (16)][4 channels], 512 bytes; their scores and maxima
  const __amdgpu_buffer_rsrc_t in = spin_buffer(summ + base * 2 + (size_t)t_begin * 32, (uint32_t)(t_end - t_begin) * 512);
  const __amdgpu_buffer_rsrc_t out = spin_buffer(scores + base + (size_t)t_begin * 16, (uint32_t)(t_end - t_begin) * 64);
  const __amdgpu_buffer_rsrc_t top_out =
      spin_buffer(MAXIMA ? tm.at + (size_t)row * tm.stride + t_begin : nullptr,
                  MAXIMA ? (uint32_t)max(min(t_end, tm.stride) - t_begin, 0) * 4 : 0);
  const int tok = (c >> 1) * 32 + 2 * n + (c & 1), my_tile = 2 * (c >> 1) + (n >> 3);   // the lane's of a group of four tiles
  uint32_t at_in = (uint32_t)(wave * 4 * U + (n >> 3)) * 512 + (uint32_t)(c * 8 + (n & 7)) * 16;
  uint32_t at_out = (uint32_t)(wave * 4 * U * 16 + tok) * 4;
  // a tile's tokens lie in 8 lanes of two lane rows, the first of which stores their maximum
  uint32_t at_top = (n & 7) == 0 && !(c & 1) ? (uint32_t)(wave * 4 * U + my_tile) * 4 : 0x80000000u;
  uint4 ld[U][2];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      ld[u][i] = spin_buffer_load(in, at_in + (4 * u + 2 * i) * 512, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  spin_s16x4 qa[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
    qa[j] = __builtin_bit_cast(spin_s16x4, (n >> 2) == j && (n & 3) < G ? make_uint2(e[0] | (e[1] << 16), e[2] | (e[3] << 16))
                                                                       : make_uint2(0u, 0u));
  for (int t0 = t_begin + wave * 4 * U; t0 < t_end; t0 += ROUND) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      spin_f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint2 lo = make_uint2(ld[u][i].x, ld[u][i].y), hi = make_uint2(ld[u][i].z, ld[u][i].w);
        s = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(qa[2 * i], __builtin_bit_cast(spin_s16x4, lo), s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(qa[2 * i + 1], __builtin_bit_cast(spin_s16x4, hi), s, 0, 0, 0);
        if (!ONE) ld[u][i] = spin_buffer_load(in, at_in + (ROUND + 4 * u + 2 * i) * 512, 0);
      }
      float mx = -__builtin_inff();               // heads 0..3 of the lane's token
#pragma unroll
      for (int i = 0; i < 4; ++i) mx = i < G ? fmaxf(mx, s[i]) : mx;
      spin_buffer_store(out, at_out + 4 * u * 64, mx);
      if (MAXIMA) {
        float top = fmaxf(mx, spin_dpp<SPIN_DPP_XOR1>(mx));
        top = fmaxf(top, spin_dpp<SPIN_DPP_XOR2>(top));
        top = fmaxf(top, spin_dpp<SPIN_DPP_HALF_MIRROR>(top));
        top = fmaxf(top, __shfl_xor(top, 16));
        spin_buffer_store(top_out, at_top + 4 * u * 4, top);
      }
    }
    if (ONE) break;
    at_in += ROUND * 512;
    at_out += ROUND * 64;
    at_top += ROUND * 4;
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
    // groups of up to four heads: the four-tile kernel, 64 tiles per workgroup, one round (32 / 64 / 128 / 256 / 512:
    // 26.4 / 25.6 / 26.9 / 26.4 / 28.2 us on 64 rows of 65536 tokens)
    const bool four = ctx->group <= 4 && (c.score_tiles_per_wg % 4) == 0;
    // (a workgroup addresses its tiles in 32 bits: half a GiB of them at most)
    const int tiles_per_wg = c.score_tiles_per_wg ? std::min(c.score_tiles_per_wg, 1 << 20) : 64, max_tiles = max_pp / 16;
    // The grid is as long as the context's longest row, so that most workgroups of a context sized for more than is
    // running are empty.  They cost the time to start them, which a grid of three dimensions halves (no divisions), and
    // an odd number of them per row keeps the rows' first workgroups, the only ones with work then, from all going to
    // the same of the 8 dies.  1024 rows of 2000 tokens in contexts for 32768 / 36000: 94 / 22 -> 14 / 15 us; 256 rows of
    // 4096 for 131072 / 1048576: 27 / 106 -> 13.5 / 86; 8 rows of 4096 and 64 of 65536 in contexts of their length 3.9 / 24.5
    // -> 4.0 / 24.2.
    const int wgs = ((max_tiles + tiles_per_wg - 1) / tiles_per_wg) | 1;
    constexpr int MOST = 65535;                   // of the grid's second and third dimension
#define SPIN_SKETCH_LAUNCH1(KERNEL)                                                                              \
  for (int b0 = 0; b0 < batch; b0 += MOST)                                                                       \
    for (int h0 = 0; h0 < c.num_kv_heads; h0 += MOST)                                                            \
      spin_launch(ctx, SPIN_K_SCORE, KERNEL,                                                                     \
                  dim3((unsigned)wgs, (unsigned)std::min(c.num_kv_heads - h0, MOST), (unsigned)std::min(batch - b0, MOST)), \
                  dim3(SCORE_WAVES * 64), 0, st, (const uint16_t *)q, (const uint4 *)summaries, chan_idx, part_offsets, \
                  c.num_kv_heads, ctx->group, tiles_per_wg, b0, h0, scores, tm)
#define SPIN_SKETCH_LAUNCH(KERNEL)                                                            \
  do {                                                                                        \
    if (maxima && tiles_per_wg <= 64) SPIN_SKETCH_LAUNCH1((KERNEL<true, true>));              \
    else if (maxima) SPIN_SKETCH_LAUNCH1((KERNEL<true, false>));                              \
    else if (tiles_per_wg <= 64) SPIN_SKETCH_LAUNCH1((KERNEL<false, true>));                  \
    else SPIN_SKETCH_LAUNCH1((KERNEL<false, false>));                                         \
  } while (0)
    if (four) SPIN_SKETCH_LAUNCH(spin_score_sketch4_kernel);
    else SPIN_SKETCH_LAUNCH(spin_score_sketch_kernel);
#undef SPIN_SKETCH_LAUNCH
#undef SPIN_SKETCH_LAUNCH1
  }
  return spin_launch_status();
}

extern "C" int spin_score_partitions(spin_ctx *ctx, int32_t batch, const void *q, const void *summaries,
                                     const int32_t *chan_idx, const int32_t *part_offsets,
                                     const int32_t *seq_lens, float *scores, void *workspace, void *stream) {
  return spin_score_impl(ctx, batch, q, summaries, chan_idx, part_offsets, seq_lens, scores, workspace, stream, nullptr);
}
