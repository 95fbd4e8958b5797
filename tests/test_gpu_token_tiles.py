"""Stage 4 of partitions smaller than a page: a wavefront's pages become a list of attended tokens,
which is attended 16 at a time through a ring of two tiles.  Lists that are empty, end inside a tile,
fill it, end a round of the ring or begin the next one, and lists of more than 64 pages."""
import pytest

import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# pages per row and attended tokens per page (None: any number, also none); with 2 rows in a context
# for 128 there are 2 x 8 wavefronts to a row, so 16 n pages give each of them n
@pytest.mark.parametrize("npages,per_page", [(1, 1), (1, 16), (5, 15), (16, 16), (17, 16), (32, 8), (32, 9), (48, 16), (49, 16),
                                             (64, 16), (80, 7), (512, 1), (1024, 16), (1040, 1), (1040, None), (333, None)])
@pytest.mark.parametrize("q_heads", [2, 8, 32])
def test_lists_of_every_length(npages, per_page, q_heads):
    from paper_2604_26837_amd import runner, synth
    w = synth.Workload(name="tiles", seq_lens=(1040 * 16,), num_q_heads=q_heads, num_kv_heads=2, partition_tokens=1,
                       score_kind=synth.SCORE_SKETCH, reps_per_partition=1, topk=1040, topk_includes_forced=True,
                       sink_pages=0, recent_pages=0, planted_frac=0.0, seed=npages * 100 + q_heads)
    layer, natural = runner.build_device_layer(w, keep_natural=True, max_batch=64)
    gen = torch.Generator().manual_seed(npages)
    rows, stride = 2, layer.slots.shape[1]
    assert npages <= stride
    keep = torch.zeros((rows, stride, 16), dtype=torch.bool)
    for r in range(rows):
        for p in range(npages):
            n = int(torch.randint(0, 17, (1,), generator=gen)) if per_page is None else per_page
            keep[r, p, torch.randperm(16, generator=gen)[:n]] = True
    mask = (keep.to(torch.int32) << torch.arange(16, dtype=torch.int32)).sum(-1).to(torch.int16)
    slots = torch.full((rows, stride), -1, dtype=torch.int32)
    for r in range(rows):
        slots[r, :npages] = torch.randperm(natural.shape[0], generator=gen)[:npages].to(torch.int32)
    layer.slots.copy_(slots)
    layer.valid_mask.copy_(mask)
    layer.npages.fill_(npages)
    layer.spin.sparse_decode(1, layer.q0, layer.kv_pool, layer.slots, layer.valid_mask, layer.npages, layer.out, layer.lse,
                             layer.ws)
    torch.cuda.synchronize()
    assert layer.status() == 0
    g = q_heads // rows
    for r in range(rows):
        pages = natural.cpu()[slots[r, :npages].long()].double()          # [page][K, V][token][channel]
        k, v = pages[:, 0][keep[r, :npages]], pages[:, 1][keep[r, :npages]]
        qh = layer.q0[0, r * g:(r + 1) * g].cpu().double()
        logits = qh @ k.T * layer.scale
        p = torch.softmax(logits, dim=-1)
        want = p @ v
        # probabilities and outputs are rounded to bf16 once each (2**-9 of their size); as much again for fp32 logits
        bound = 2.0 ** -8 * (p @ v.abs()) + 2.0 ** -8 * want.abs() + 1e-6
        got = layer.out[0, r * g:(r + 1) * g].cpu().double()
        assert bool(((got - want).abs() <= bound).all())
        lse = torch.logsumexp(logits, dim=-1)
        assert torch.allclose(layer.lse[0, r * g:(r + 1) * g].cpu().double(), lse, rtol=0, atol=2e-4)
