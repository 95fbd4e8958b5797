"""Stage 2 of rows held in registers, against a sort: the tail's histogram (scores of any spread, few and many outliers, rows
as long as they may be), more than 64 scores in the threshold's step, scores that are not finite, pins in every part of the
row (fewer and more than are wanted), at the sizes where the scores per thread, the groups and the interleaved parts
change."""
import numpy as np
import pytest
import torch

from paper_2604_26837_amd import runner, synth

pytestmark = pytest.mark.gpu


def _scores(kind, n, rng):
    x = rng.standard_normal(n)
    if kind == "ties":
        x = np.round(x * 2)
    elif kind == "spread":
        x = np.sign(x) * np.exp2(60 * np.abs(x))
    elif kind == "outliers":
        x[rng.random(n) < 0.004] = 1e30
    elif kind == "close":
        x = 1000 + x * 1e-3
    elif kind == "rising":
        x = np.arange(n) * 1e-3 + x
    elif kind == "inf":
        x[rng.random(n) < 0.01] = np.inf
        x[rng.random(n) < 0.5] = -np.inf
    elif kind == "pins":
        x[rng.random(n) < 0.03] = np.inf
    elif kind == "pins and outliers":
        x[rng.random(n) < 0.01] *= 1e6
        x[rng.random(n) < 0.01] = np.inf
    elif kind == "zeros":
        x = np.where(rng.random(n) < 0.02, x, np.where(rng.random(n) < 0.5, 0.0, -0.0))
    elif kind == "nan":
        x[rng.random(n) < 0.97] = np.nan
    elif kind == "tiny":
        x *= 1e-40
    return x.astype(np.float32)


@pytest.mark.parametrize("kind", ["normal", "ties", "spread", "outliers", "close", "rising", "inf", "nan", "tiny", "pins",
                                  "pins and outliers", "zeros"])
@pytest.mark.parametrize("pages,topk", [(40, 5), (256, 32), (2048, 62), (2048, 63), (2048, 128), (2047, 1300), (4096, 511),
                                        (4096, 527), (8192, 140), (8191, 4100), (16384, 200), (16384, 3000)])
def test_against_a_sort(pages, topk, kind):
    lens = (pages * 16, pages * 16 - 5, pages * 5 + 1)
    w = synth.Workload(name="tail", seq_lens=lens, num_q_heads=2, num_kv_heads=2, partition_tokens=16,
                       score_kind=synth.SCORE_MINMAX, reps_per_partition=1, topk=topk, topk_includes_forced=True,
                       sink_pages=3, recent_pages=9, planted_frac=0.0, seed=1)
    slot_of = [np.zeros((2, -(-n // 16)), np.int32) for n in lens]
    layer = runner.LayerState(w, slot_of, torch.zeros((1, 4096), dtype=torch.bfloat16, device="cuda:0"))
    rng = np.random.default_rng(pages * 7 + topk)
    scores = _scores(kind, layer.scores.numel(), rng)
    layer.scores.copy_(torch.from_numpy(scores))
    layer.spin.select_topk(w.batch, layer.scores, layer.part_offsets, layer.seq_lens, layer.sel, layer.nsel, layer.ws)
    sel, nsel = layer.sel.cpu().numpy(), layer.nsel.cpu().numpy()
    for b, n in enumerate(lens):
        P = -(-n // 16)
        lo, hi = min(3, P), max(P - 9, 0)
        for h in range(2):
            row = scores[layer.row_base(b, h):][:P].astype(np.float64)
            row = np.where(np.isnan(row), -np.inf, row)
            cand = np.arange(lo, hi)
            best = cand[np.lexsort((cand, -row[cand]))[:max(topk - (lo + P - hi), 0)]]
            want = np.sort(np.concatenate([np.arange(lo), best, np.arange(hi, P)]))
            got = sel[2 * b + h]
            assert nsel[2 * b + h] == len(want) and np.array_equal(got[:len(want)], want) and (got[len(want):] == -1).all()
