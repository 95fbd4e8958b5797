"""The launch of stages 2+3 hands a row's selection and its directory over in LDS; beyond what that
holds they go through memory.  Every output has to have the bits of the separate stage calls, which
know nothing of it: selections as long as what is held, one shorter and one longer, and directories
of as many entries as are staged and of more."""
import numpy as np
import pytest

import torch

pytestmark = pytest.mark.gpu

HELD, DIR = 2304, 256          # SEL_HELD and RES_DIR_LDS of csrc/spin_resolve_dev.h


@pytest.mark.parametrize("part,topk,tokens,leaf", [
    (1, HELD - 1, 4093, 64), (1, HELD, 4093, 64), (1, HELD + 1, 4093, 64),       # rows held in registers
    (1, HELD, 20011, 64), (1, HELD + 1, 20011, 64),                             # by the tiles' maxima
    (16, HELD, 64999, 64), (16, HELD + 1, 64999, 64),                           # whole pages, the forced ones beside it
    (16, 40, DIR * 16, 1), (16, 40, DIR * 16 + 1, 1), (16, 40, 20003, 1),       # one leaf entry per directory entry
    (8, 300, 6001, 4), (2, 77, 3001, 16),                                       # several partitions to a page
    (64, 20, DIR * 16 + 100, 1),
])
def test_fused_equals_stage_calls(part, topk, tokens, leaf):
    from paper_2604_26837_amd import runner, synth
    w = synth.Workload(name="handover", seq_lens=(tokens, max(tokens // 3, 1)), num_q_heads=8, num_kv_heads=2,
                       partition_tokens=part, score_kind=synth.SCORE_SKETCH if part == 1 else synth.SCORE_MINMAX,
                       reps_per_partition=1, topk=topk, topk_includes_forced=True, sink_pages=0 if part == 1 else 1,
                       recent_pages=0 if part == 1 else 2, planted_frac=0.0, leaf_entries=leaf,
                       seed=part * 100003 + topk)
    layer = runner.build_device_layer(w)[0]
    q = layer.q0
    names = ("sel", "nsel", "slots", "page_ids", "valid_mask", "npages")

    def outputs():
        torch.cuda.synchronize()
        assert layer.status() == 0
        return {n: getattr(layer, n).cpu().numpy().copy() for n in names}

    layer.step(q)
    want = outputs()
    for fused in (layer.step123, layer.step_fused):
        for n in names:
            getattr(layer, n).fill_(77)
        fused(q)
        got = outputs()
        for n in names:
            assert np.array_equal(want[n], got[n]), (fused.__name__, n)


@pytest.mark.parametrize("topk", [300, HELD, HELD + 1])
def test_a_row_longer_than_its_context(topk):
    """Such a row has no maxima for all its tiles: it is searched in memory, and handed over like the others."""
    from paper_2604_26837_amd import runner, synth
    lens = (17003, 3001, 16390)
    w = synth.Workload(name="longer", seq_lens=lens, num_q_heads=8, num_kv_heads=2, partition_tokens=1,
                       score_kind=synth.SCORE_SKETCH, reps_per_partition=1, topk=topk, topk_includes_forced=True,
                       sink_pages=0, recent_pages=0, planted_frac=0.0, leaf_entries=2048, seed=topk)
    rng = np.random.default_rng(topk)
    slot_of, at = [], 0
    for n in lens:
        pages = -(-n // 16)
        slot_of.append(at + rng.permutation(2 * pages).astype(np.int32).reshape(2, pages))
        at += 2 * pages
    layer = runner.LayerState(w, slot_of, torch.zeros((at, 4096), dtype=torch.bfloat16, device="cuda:0"),
                              max_context=16400)
    sp = layer.spin
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(topk)
    layer.scores.normal_(generator=gen)
    names = ("sel", "nsel", "slots", "page_ids", "valid_mask", "npages")

    def outputs(call):
        for n in names:
            getattr(layer, n).fill_(77)
        call()
        torch.cuda.synchronize()
        assert layer.status() == 0
        return {n: getattr(layer, n).cpu().numpy().copy() for n in names}

    def stage_calls():
        sp.select_topk(3, layer.scores, layer.part_offsets, layer.seq_lens, layer.sel, layer.nsel, layer.ws)
        sp.resolve_slots(3, 0, layer.sel, layer.nsel, layer.seq_lens, layer.dir, layer.leaf_pool, layer.slots,
                         layer.page_ids, layer.valid_mask, layer.npages, layer.ws)

    def fused():
        sp.select_resolve(3, layer.scores, layer.part_offsets, layer.seq_lens, layer.sel, layer.nsel, layer.dir,
                          layer.leaf_pool, layer.slots, layer.page_ids, layer.valid_mask, layer.npages, layer.ws)

    want, got = outputs(stage_calls), outputs(fused)
    for n in names:
        assert np.array_equal(want[n], got[n]), n
    scores = layer.scores.cpu().numpy().astype(np.float64)
    for b, n in enumerate(lens):
        for h in range(2):
            row = scores[layer.row_base(b, h):][:n]
            best = np.sort(np.lexsort((np.arange(n), -row))[:topk])
            assert np.array_equal(got["sel"][2 * b + h, :len(best)], best)
