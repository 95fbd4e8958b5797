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
