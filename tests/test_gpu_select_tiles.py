"""Stage 2 by the maxima of the score tiles: bit-exact against the oracle at the row lengths and selection sizes where
a tile straddles the candidates' ends, the tiles become too few for k', the list of scores overflows, or another
kernel variant takes over; and the combined call (maxima from stage 1) against the stage calls."""
import numpy as np
import pytest
import torch

from paper_2604_26837_amd import runner, synth
from test_gpu_stages import _check_select

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (partitions, k, sink pages, recent pages) of the longest row; pages of 16 tokens, one partition each
SIZES = [(16385, 1, 0, 0), (16385, 1024, 15, 17), (16400, 1025, 16, 16), (20000, 1249, 3, 8), (20000, 1300, 3, 8),
         (32768, 2040, 0, 1), (62500, 256, 4, 8), (65535, 3600, 1, 1), (65536, 3700, 0, 0), (65537, 128, 4, 8),
         (131071, 700, 7, 9), (131072, 40, 0, 16),
         # k' hardly below, at and beyond the number of tiles, and nearly all partitions: rows that are walked whole
         (16385, 1000, 0, 0), (16400, 16380, 5, 7), (20000, 6000, 3, 8), (65536, 4095, 0, 0), (65536, 12000, 2, 3),
         (131072, 8192, 1, 1), (131072, 131000, 3, 0)]


@pytest.mark.parametrize("parts,topk,sink,recent", SIZES)
def test_rows_by_tile_maxima(parts, topk, sink, recent):
    rng = np.random.default_rng(parts * 3 + topk)
    lens = (parts * 16, parts * 16 - 5, max(parts // 3, 1) * 16 + 3, 40 * 16)
    w = synth.config0().with_(num_q_heads=4, num_kv_heads=1, seq_lens=lens, topk=topk, topk_includes_forced=True,
                              sink_pages=sink, recent_pages=recent, name="tiles")
    smooth = [(rng.standard_normal(w.partitions(b)) * 10 + 150).astype(np.float32) for b in range(4)]
    ties = [np.round(x / 4).astype(np.float32) for x in smooth]
    equal = [np.full(len(x), 2.0, dtype=np.float32) for x in smooth]
    # whole tiles of large scores: every score of the k' tiles is a candidate
    clustered = [np.where(np.arange(len(x)) // 16 % 37 == 5, x + 1000, -x).astype(np.float32) for x in smooth]
    nans = [np.where(rng.random(len(x)) < 0.995, np.nan, x).astype(np.float32) for x in smooth]
    # most scores lie close together, so that a bin of the first histogram holds more than the list
    narrow = [np.where(rng.random(len(x)) < 0.01, x * 10, 150 + x / 1000).astype(np.float32) for x in smooth]
    low = [np.where(rng.random(len(x)) < 0.999, -np.inf, np.where(rng.random(len(x)) < 0.5, np.nan, x)).astype(np.float32)
           for x in smooth]
    # all tiles' maxima alike, and the greatest scores in the tiles that straddle the candidates' ends
    ends = [np.where((np.arange(len(x)) < 16 * (sink // 16 + 1)) | (np.arange(len(x)) >= len(x) - recent - 16),
                     np.float32(9) + (x > 150), np.float32(2)).astype(np.float32) for x in smooth]
    for rows in (smooth, ties, equal, clustered, nans, low, narrow, ends):
        _check_select(w, rows)


@pytest.mark.parametrize("parts", [20000, 65536])
def test_time_of_large_selections(parts):
    """Stage 2 takes longer for a larger k', for the walks over all scores and the longer output, but not by the many
    times that a path for exceptions costs: the least of 30 launches of k' = half the row's tiles (few scores read)
    against k' = one and a half times the tiles (all read three times).  Measured 1.5 times; scores re-read per digit,
    or by each thread a stretch of its own, 3.7 and 10.6 times.  Nor for scores that are all the same (1.7 to 2.1
    times; each counted by itself in one place 9 and 13)."""
    least = []
    for topk, alike in ((parts // 32, False), (parts * 3 // 32, False), (parts // 32, True)):
        w = synth.config0().with_(num_q_heads=4, num_kv_heads=1, seq_lens=(parts,) * 2, partition_tokens=1,
                                  score_kind=synth.SCORE_SKETCH, topk=topk, sink_pages=0, recent_pages=0, name="large")
        layer = runner.build_device_layer(w)[0]
        layer.step(layer.q0)
        if alike:
            layer.scores.fill_(2.0)
        layer.spin.profile_enable(64)
        for _ in range(30):
            layer.spin.select_topk(w.batch, layer.scores, layer.part_offsets, layer.seq_lens, layer.sel, layer.nsel, layer.ws)
        torch.cuda.synchronize()
        least.append(layer.spin.profile_read("select")[2])
    assert max(least[1:]) < 3 * least[0]


# kernel variants by row length and representatives per partition (tiles of 16, 8 and 4 partitions)
CALLS = [(16385, 1, 120, 1, 1), (20000, 1, 1500, 0, 0), (65536, 1, 2048, 0, 1), (70000, 1, 90, 1, 0),
         (65536, 1, 5000, 0, 1), (20000, 1, 2048, 1, 0), (33000, 4, 9000, 3, 5), (16400, 2, 300, 2, 21), (17000, 4, 1025, 0, 0), (33000, 4, 200, 3, 5)]


@pytest.mark.parametrize("parts,reps,topk,sink,recent", CALLS)
def test_combined_call_by_tile_maxima(parts, reps, topk, sink, recent):
    tp = 16 if reps > 1 else 1
    lens = (parts * tp, parts * tp - 3, parts * tp // 5, 90 * tp)
    kind = synth.SCORE_REPMAX if reps > 1 else synth.SCORE_SKETCH
    if tp == 1:
        sink = recent = min(sink, 1)
    w = synth.config0().with_(num_q_heads=5, num_kv_heads=1, seq_lens=lens, partition_tokens=tp, score_kind=kind,
                              reps_per_partition=reps if reps > 1 else 4, topk=topk, sink_pages=sink,
                              recent_pages=recent, name="tiles_call")
    data = synth.generate(w)
    natural = torch.from_numpy(data.pool_bits.view(np.int16).copy()).to(DEV).view(torch.bfloat16)
    layer = runner.LayerState.from_natural_pool(w, data.slot_of, natural)
    if kind == synth.SCORE_SKETCH:
        layer.set_channels(synth.sketch_channels(data))
    layer.build_summaries()
    names = ("scores", "sel", "nsel", "slots", "page_ids", "valid_mask", "npages", "out", "lse")
    for seed in range(3):
        q = torch.from_numpy(synth.make_queries(w, 40 + seed).view(np.int16)).to(DEV).view(torch.bfloat16)
        layer.step(q)
        torch.cuda.synchronize()
        want = {n: getattr(layer, n).clone() for n in names}
        layer.ws.fill_(0x7f)                       # nothing may depend on what the workspace held, tickets aside
        layer.spin.workspace_init(layer.ws)
        for n in names[1:]:
            getattr(layer, n).fill_(-3)
        layer.step123(q)
        torch.cuda.synchronize()
        assert layer.status() == 0
        keep = torch.arange(layer.slots.shape[1], device=DEV)[None, :] < layer.npages[:, None]
        for n in names:
            got, ref = getattr(layer, n), want[n]
            if n in ("slots", "page_ids", "valid_mask"):
                got, ref = got[keep], ref[keep]
            assert torch.equal(got, ref), (seed, n)
