// Tiles of 16 gathered tokens (partitions smaller than a page, token-major slots), shared by stage 4 and by the launch of
// stages 2 to 4.
#pragma once
#include "spin_decode_dev.h"

struct tile_src {
  const uint4 *k;           // key row of tile row n (lane % 16), chunk c (lane / 16): + 4 j
  const uint4 *v[4];        // value rows of tile rows 4c .. 4c+3, channels 8n .. 8n+7
};

// Rows past the end of the list, and tiles past it, repeat its last entry: their loads stay inside attended data (and
// touch few lines), their logits are masked and their probabilities are exactly zero.
__device__ inline tile_src tile_source(const uint4 *__restrict__ pool, const uint32_t *tok, int first, int count, int lane) {
  tile_src s;
  const int n = lane & 15, c = lane >> 4;
  const uint32_t e = tok[min(first + n, count - 1)];     // slot * 16 + token
  s.k = pool + (size_t)(e >> 4) * SPIN_SLOT_U4 + (e & 15u) * 16 + c;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t ev = tok[min(first + 4 * c + i, count - 1)];
    s.v[i] = pool + (size_t)(ev >> 4) * SPIN_SLOT_U4 + SPIN_KTILE_U4 + (ev & 15u) * 16 + n;
  }
  return s;
}

__device__ inline void load_tile(page_regs &r, const tile_src &s) {
#pragma unroll
  for (int j = 0; j < 4; ++j) r.k[j] = spin_nt_load(s.k + 4 * j);
#pragma unroll
  for (int i = 0; i < 4; ++i) r.v[i] = *s.v[i];
}

// The value rows 4c .. 4c+3 a lane holds, as the operands of P V: r.v[jv] = {rows 4c,4c+1 | rows 4c+2,4c+3} of channel
// 8n + 2jv, then of 8n + 2jv+1 (channel block jn has channels 8n + jn here, decode_finish<.., true>).
__device__ __forceinline__ void transpose_values(page_regs &r) {
  const uint32_t w[4][4] = {{r.v[0].x, r.v[0].y, r.v[0].z, r.v[0].w}, {r.v[1].x, r.v[1].y, r.v[1].z, r.v[1].w},
                            {r.v[2].x, r.v[2].y, r.v[2].z, r.v[2].w}, {r.v[3].x, r.v[3].y, r.v[3].z, r.v[3].w}};
#pragma unroll
  for (int jv = 0; jv < 4; ++jv) {
    auto lows = [&](int a, int b) { return (w[a][jv] & 0xffffu) | (w[b][jv] << 16); };
    auto highs = [&](int a, int b) { return (w[a][jv] >> 16) | (w[b][jv] & 0xffff0000u); };
    r.v[jv] = make_uint4(lows(0, 1), lows(2, 3), highs(0, 1), highs(2, 3));
  }
}

// Attends the `total` tokens of a list (without any: the list has an entry to load from all the same) through a ring of D
// register buffers, as attend_lane_pages does pages: the loop has no branch around a load, so that it waits for exactly
// the tile it is about to read.  `asked` runs once the first D tiles have been asked for.
template <int D, typename ASKED>
__device__ __forceinline__ void attend_token_tiles(softmax_state &st, const uint4 *__restrict__ pool, const uint32_t *tok,
                                                   int total, int lane, int c, const spin_bf16x8 (&qf)[4],
                                                   float scale_log2e, ASKED asked) {
  page_regs r[D];
  const int ntiles = (total + 15) >> 4;
  auto load = [&](int d, int k) {
    load_tile(r[d], tile_source(pool, tok, 16 * k, max(total, 1), lane));
    __builtin_amdgcn_sched_barrier(0);   // asked for in the order in which the loop asks again
  };
  auto attend = [&](int d, int k) {
    const int left = total - 16 * k;
    const spin_f32x4 s = tile_logits(r[d], qf);
    transpose_values(r[d]);
    tile_attend(st, s, r[d], left >= 16 ? 0xffffu : ((1u << left) - 1u), c, scale_log2e);
  };
#pragma unroll
  for (int d = 0; d < D; ++d) load(d, d);
  asked();
  int k = 0;
  for (; k + D <= ntiles; k += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      attend(d, k + d);
      load(d, k + d + D);
    }
  }
#pragma unroll
  for (int d = 0; d < D - 1; ++d)
    if (k + d < ntiles) attend(d, k + d);
}
