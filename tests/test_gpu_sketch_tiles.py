"""Stage 1 of token partitions: tile counts around one round of a workgroup (64 tiles), tiles per workgroup that leave
half a pair or several rounds, every kind of group.  The scores against sums in 64 bits to the order bound of 16
products in 32 bits; nothing is stored past a row's last tile.  Where they are asked for, the tiles' maxima are exactly
those of the stored scores, and a selection that rules tiles out by them is the right one."""
import numpy as np
import pytest
import torch

from paper_2604_26837_amd import binding, synth, tables

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("maxima", [False, True])
@pytest.mark.parametrize("tiles_per_wg", [0, 5, 36, 128])
@pytest.mark.parametrize("group", [1, 3, 4, 5, 8, 16])
def test_scores_and_maxima(group, tiles_per_wg, maxima):
    from gpu_harness import unpack_summary_rows
    kv, lens = 2, (1, 16 * 63, 16 * 64 + 3, 16 * 193 + 1)
    topk = 20 if tiles_per_wg else 200                    # fewer than the longest rows have tiles, and more
    sp = binding.Spin(max_batch=len(lens), num_q_heads=kv * group, num_kv_heads=kv, partition_tokens=1,
                      score_kind=synth.SCORE_SKETCH, topk=topk, sink_pages=0, recent_pages=0, score_tiles_per_wg=tiles_per_wg,
                      max_context=16400 if maxima else max(lens))   # (long enough for stage 2 to go by them)
    off = tables.part_offsets(lens, 1)
    total = int(off[-1]) * kv
    gen = torch.Generator(device=DEV)
    gen.manual_seed(group)
    summ = torch.randn(total * 16, generator=gen, device=DEV).to(torch.bfloat16)
    q = torch.randn((len(lens), kv * group, 128), generator=gen, device=DEV).to(torch.bfloat16)
    chan = torch.stack([torch.randperm(128, generator=gen, device=DEV)[:16] for _ in range(kv)]).to(torch.int32).contiguous()
    scores = torch.full((total + 64,), 7.5, device=DEV)
    seq = torch.tensor(lens, dtype=torch.int32, device=DEV)
    offs = torch.from_numpy(off).to(DEV)
    ws = sp.new_workspace(DEV)
    if maxima:
        sel = torch.zeros((len(lens) * kv, sp.sel_stride), dtype=torch.int32, device=DEV)
        nsel = torch.zeros(len(lens) * kv, dtype=torch.int32, device=DEV)
        sp.score_select_topk(len(lens), q, summ.view(torch.uint8), chan, offs, seq, scores, sel, nsel, ws)
    else:
        sp.score_partitions(len(lens), q, summ.view(torch.uint8), chan, offs, seq, scores, ws)
    torch.cuda.synchronize()
    assert sp.poll_status(ws) == 0
    rows = unpack_summary_rows(summ.view(torch.uint8), 16, 4).astype(np.uint32) << 16
    rows = rows.view(np.float32).astype(np.float64)       # [tokens][16]
    words = ws.cpu().numpy()
    words = words[:words.nbytes // 4 * 4].view(np.float32)
    qf, ch, got = q.double().cpu().numpy(), chan.cpu().numpy(), scores.cpu().numpy()
    for b in range(len(lens)):
        for h in range(kv):
            n = int(off[b + 1] - off[b])
            base = int(off[b]) * kv + h * n
            heads = qf[b, h * group:(h + 1) * group][:, ch[h]]
            terms = rows[base:base + n] @ heads.T
            bound = 16 * 2.0 ** -24 * (np.abs(rows[base:base + n]) @ np.abs(heads).T).max(axis=1)
            assert (np.abs(got[base:base + n] - terms.max(axis=1)) <= bound).all()
            if maxima:                                    # the selection is the k largest of the scores, ties lowest first
                want = np.sort(np.lexsort((np.arange(lens[b]), -got[base:base + lens[b]].astype(np.float64)))[:topk])
                r = b * kv + h
                assert np.array_equal(sel[r, :int(nsel[r])].cpu().numpy(), want)
                tops = got[base:base + n].reshape(-1, 16).max(axis=1)      # a row's stand together in the workspace
                assert any(np.array_equal(words[i:i + len(tops)], tops) for i in np.flatnonzero(words == tops[0]))
    assert (got[total:] == 7.5).all()


@pytest.mark.parametrize("batch,kv", [(65537, 1), (1, 65537), (70, 1000)])
def test_more_requests_or_heads_than_a_grid_dimension_holds(batch, kv):
    sp = binding.Spin(max_batch=batch, num_q_heads=kv, num_kv_heads=kv, partition_tokens=1, score_kind=synth.SCORE_SKETCH,
                      topk=4, sink_pages=0, recent_pages=0, max_context=32)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(batch)
    # one tile per row; whole numbers, whose sums are exact in any order
    summ = torch.randint(-8, 9, (batch, kv, 4, 16, 4), generator=gen, device=DEV).to(torch.bfloat16)
    q = torch.randint(-8, 9, (batch, kv, 128), generator=gen, device=DEV).to(torch.bfloat16)
    chan = torch.randint(0, 128, (kv, 16), generator=gen, device=DEV, dtype=torch.int32)
    off = torch.arange(0, 16 * batch + 1, 16, dtype=torch.int32, device=DEV)
    seq = torch.full((batch,), 16, dtype=torch.int32, device=DEV)
    scores = torch.full((batch * kv * 16,), 7.5, device=DEV)
    ws = sp.new_workspace(DEV)
    sp.score_partitions(batch, q, summ.view(-1).view(torch.uint8), chan, off, seq, scores, ws)
    torch.cuda.synchronize()
    taken = torch.gather(q.float(), 2, chan.long().expand(batch, kv, 16))
    want = torch.zeros((batch, kv, 16), device=DEV)
    for quad in range(4):
        for i in range(4):
            want += taken[:, :, 4 * quad + i, None] * summ[:, :, quad, :, i].float()
    assert torch.equal(scores.view(batch, kv, 16), want)


def test_tiles_of_a_workgroup_beyond_4_gib():
    """One row of 4 GiB and three tiles, all of them asked to be one workgroup's."""
    tiles = (1 << 23) + 3
    sp = binding.Spin(max_batch=1, num_q_heads=1, num_kv_heads=1, partition_tokens=1, score_kind=synth.SCORE_SKETCH, topk=4,
                      sink_pages=0, recent_pages=0, max_context=16 * tiles, score_tiles_per_wg=tiles + 1)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    summ = torch.randint(-8, 9, (tiles, 4, 16, 4), generator=gen, device=DEV, dtype=torch.int8).to(torch.bfloat16)
    q = torch.randint(-8, 9, (1, 1, 128), generator=gen, device=DEV).to(torch.bfloat16)
    chan = torch.randperm(128, generator=gen, device=DEV)[:16].to(torch.int32).view(1, 16)
    off = torch.tensor([0, 16 * tiles], dtype=torch.int32, device=DEV)
    seq = torch.tensor([16 * tiles], dtype=torch.int32, device=DEV)
    scores = torch.full((tiles * 16,), 7.5, device=DEV)
    sp.score_partitions(1, q, summ.view(-1).view(torch.uint8), chan, off, seq, scores, sp.new_workspace(DEV))
    torch.cuda.synchronize()
    want = torch.zeros((tiles, 16), device=DEV)
    for quad in range(4):
        for i in range(4):
            want += q[0, 0, chan[0, 4 * quad + i]].float() * summ[:, quad, :, i].float()
    assert torch.equal(scores.view(tiles, 16), want)
