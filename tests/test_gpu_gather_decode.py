"""The copy of the missed pages with stage 4 beside it, against the copy and then stage 4: the same lists and slots, the
attention to the tolerance of a bf16 output of two summation orders."""
import pytest
import torch

from paper_2604_26837_amd import hier, synth


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [
    dict(lens=(5000, 9001, 700), topk=40),
    dict(lens=(20000,), topk=200, kv=1, heads=16),                    # several splits, one row, 16 heads
    dict(lens=(9000, 4000), part=64, topk=9, score=synth.SCORE_REPMAX, incl=False, recent=6),
    dict(lens=(300, 40), topk=30),                                    # every page attended
])
@pytest.mark.parametrize("over", [dict(), dict(lru_policy=1), dict(decode_splits=3, decode_waves=4)])
def test_equals_the_copy_and_then_stage_4(kw, over):
    part = kw.get("part", 16)
    w = synth.Workload(name="budget", seq_lens=kw["lens"], num_q_heads=kw.get("heads", 8), num_kv_heads=kw.get("kv", 2),
                       partition_tokens=part, score_kind=kw.get("score", synth.SCORE_MINMAX),
                       reps_per_partition=4 if part == 64 else 1, topk=kw["topk"], topk_includes_forced=kw.get("incl", True),
                       sink_pages=1, recent_pages=kw.get("recent", 2), planted_frac=0.0, seed=part + kw["topk"])
    a, b = (hier.HierLayer(w, copy_mode="gather", **over) for _ in range(2))
    sp = b.spin
    qs = [a.q0, a.q0] + [synth.make_queries_on_device(w, s, "cuda:0") for s in range(3)]     # all missed, none, some
    kinds = set()
    for t, q in enumerate(qs):
        a.step(q, t, count=False)
        sp.score_partitions(w.batch, q, b.summaries, None, b.part_offsets, b.seq_lens, b.scores, b.ws)
        sp.select_topk(w.batch, b.scores, b.part_offsets, b.seq_lens, b.sel, b.nsel, b.ws)
        sp.resolve_slots(w.batch, t, b.sel, b.nsel, b.seq_lens, b.dir, b.leaf_pool, b.slots, b.page_ids, b.valid_mask,
                         b.npages, b.ws, rev_table=b.rev, slot_base=b.slot_base, miss_pages=b.miss_pages,
                         miss_slots=b.miss_slots, nmiss=b.nmiss)
        sp.gather_misses(w.batch, b.host_kv, b.host_row_base_dev, b.nmiss, b.miss_pages, b.miss_slots, b.kv_pool, b.ws)
        sp.sparse_decode(w.batch, q, b.kv_pool, b.slots, b.valid_mask, b.npages, b.out, b.lse, b.ws)
        torch.cuda.synchronize()
        assert a.status() == 0 and b.status() == 0
        for n in ("slots", "page_ids", "valid_mask", "npages", "nmiss", "miss_pages", "miss_slots", "kv_pool"):
            assert torch.equal(getattr(a, n), getattr(b, n)), (t, n)
        # probabilities rounded to bf16, and the output once more; lse sums them unrounded
        assert (a.out.float() - b.out.float()).abs().max() <= 2 ** -6 * b.out.float().abs().max(), t
        assert (a.lse - b.lse).abs().max() <= 4e-5, t
        for m, n in zip(a.nmiss.tolist(), a.npages.tolist()):
            kinds.add("none" if m == 0 else "all" if m == n else "some")
    assert kinds == ({"all", "none"} if max(kw["lens"]) <= 300 else {"all", "none", "some"})


@pytest.mark.gpu
@pytest.mark.parametrize("over", [dict(), dict(decode_splits=1), dict(decode_splits=5), dict(decode_splits=3, decode_waves=4)])
def test_lists_of_missed_pages_of_any_length(over):
    """The missed pages are dealt to the wavefronts of a workgroup before the next workgroup's: lists around the multiples
    of 4 and 8."""
    w = synth.Workload(name="budget", seq_lens=(9000, 5000, 2000, 1500), num_q_heads=12, num_kv_heads=3, partition_tokens=16,
                       score_kind=synth.SCORE_MINMAX, reps_per_partition=1, topk=70, topk_includes_forced=True,
                       sink_pages=1, recent_pages=2, planted_frac=0.0, seed=11)
    a = hier.HierLayer(w, copy_mode="gather", **over)
    sp = a.spin
    a.step(a.q0, 0, count=False)
    sp.sparse_decode(w.batch, a.q0, a.kv_pool, a.slots, a.valid_mask, a.npages, a.out, a.lse, a.ws)
    out, lse, pool = a.out.float(), a.lse.clone(), a.kv_pool.clone()
    gen = torch.Generator().manual_seed(5)
    for lens in ([0, 1, 3, 4, 5, 7, 8, 9, 15, 16, 17, 70], [24, 25, 31, 32, 33, 39, 40, 41, 63, 64, 65, 0], [0] * 12):
        a.nmiss.copy_(torch.tensor(lens, dtype=torch.int32))
        a.miss_pages.fill_(-1)
        a.miss_slots.fill_(-1)
        for r, n in enumerate(lens):                                  # what is said to have been missed is fetched once more
            at = torch.randperm(70, generator=gen)[:n].sort().values.cuda()
            a.miss_pages[r, :n], a.miss_slots[r, :n] = a.page_ids[r, at], a.slots[r, at]
            a.kv_pool[a.slots[r, at].long()] = 7.0
        a.mask_misses.fill_(-1)
        a.out.fill_(3.0)
        sp.gather_decode(w.batch, a.q0, a.host_kv, a.host_row_base_dev, a.nmiss, a.miss_pages, a.miss_slots, a.kv_pool,
                         a.slots, a.page_ids, a.valid_mask, a.npages, a.mask_misses, a.out, a.lse, a.ws)
        torch.cuda.synchronize()
        assert a.status() == 0 and torch.equal(a.kv_pool, pool)
        assert (a.out.float() - out).abs().max() <= 2 ** -6 * out.abs().max(), lens
        assert (a.lse - lse).abs().max() <= 4e-5, lens
