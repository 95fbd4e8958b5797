"""Stages 2 to 4 in one launch: the page lists have the bits of the separate stage calls, the attention is theirs to the
tolerance of a bf16 output of two summation orders, whatever the number of workgroups per row."""
import dataclasses

import pytest
import torch

from paper_2604_26837_amd import binding, runner, synth

LISTS = ("sel", "nsel", "slots", "page_ids", "valid_mask", "npages")


def _workload(lens, part=16, topk=40, incl=True, sink=2, recent=5, heads=8, kv=2, leaf=512, score=synth.SCORE_MINMAX):
    return synth.Workload(name="fused", seq_lens=lens, num_q_heads=heads, num_kv_heads=kv, partition_tokens=part,
                          score_kind=score, reps_per_partition=1, topk=topk, topk_includes_forced=incl, sink_pages=sink,
                          recent_pages=recent, planted_frac=0.0, leaf_entries=leaf, seed=part * 1009 + topk)


def _same_as_stage_calls(layer, q):
    _same(layer, q, layer.step, layer.step2)


def _same(layer, q, stage_calls, one_launch):
    def run(step):
        for n in LISTS:
            getattr(layer, n).fill_(77)
        layer.out.fill_(3.0)
        layer.lse.fill_(3.0)
        step(q)
        torch.cuda.synchronize()
        assert layer.status() == 0
        return {n: getattr(layer, n).clone() for n in LISTS + ("out", "lse")}

    want, got, again = run(stage_calls), run(one_launch), run(one_launch)
    for n in LISTS:
        assert torch.equal(want[n], got[n]), n
    for n in LISTS + ("out", "lse"):                                  # (the second: the row tickets are left cleared)
        assert torch.equal(got[n].view(torch.uint8), again[n].view(torch.uint8)), n
    # probabilities are rounded to bf16 (2^-9) before they meet the values, the output once more; lse sums them
    # unrounded: a few hundred roundings of 2^-24, exp2's last bit
    assert (got["out"].float() - want["out"].float()).abs().max() <= 2 ** -6 * want["out"].float().abs().max()
    assert torch.nan_to_num(got["lse"] - want["lse"], nan=0.0).abs().max() <= 4e-5
    assert torch.equal(got["lse"].isinf(), want["lse"].isinf())


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [
    dict(lens=(1, 16, 17, 100, 112, 113, 4096)),                      # rows as short as the windows, and shorter
    dict(lens=(32768, 32753, 20001), topk=33),                        # 2048 partitions: 4 per thread
    dict(lens=(32769, 65536), topk=128, sink=4, recent=8),            # 8
    dict(lens=(65537, 131072, 3000), topk=128, sink=0, recent=1),     # 16
    dict(lens=(131073, 262144, 50000), topk=200, sink=0, recent=0),   # 32
    dict(lens=(6001, 9000), topk=6, part=128, incl=False, recent=68),           # blocks, windows that cut them
    dict(lens=(6001, 9000, 30), topk=3, part=48, incl=False, sink=7, recent=10),
    dict(lens=(20000, 1234), topk=2304),                              # the longest selection held in LDS, or nearly all pages
    dict(lens=(40000,), topk=700, kv=1, sink=300, recent=400),        # more windows than wavefronts have lanes to ask ahead
    dict(lens=(3000, 5000), heads=32, kv=2, topk=60),                 # 16 heads to a group
    dict(lens=(3000, 5000), heads=10, kv=2, topk=60),                 # 5
    dict(lens=(64 * 16 + 1, 300 * 16), leaf=1, topk=30),              # directories of more than 64 and 256 entries
    dict(lens=(20000,), leaf=6, topk=30),
])
@pytest.mark.parametrize("splits", [0, 1, 3])
def test_equals_the_stage_calls(kw, splits):
    layer, _ = runner.build_device_layer(_workload(**kw), decode_splits=splits)
    assert layer.spin.fused_splits >= 1
    _same_as_stage_calls(layer, layer.q0)


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [
    dict(lens=(1, 15, 16, 17, 257, 1000, 4096)),                      # up to two tiles per wavefront, rows without any
    dict(lens=(4096, 4081) * 20, heads=10, topk=20),                  # and where the rows are more
    dict(lens=(1024, 1000, 3) * 25, heads=32),
    dict(lens=(8192, 8177, 700), score=synth.SCORE_REPMAX, sink=0, recent=0),
    dict(lens=(4096, 2049), score=synth.SCORE_REPMAX, reps=2, leaf=4),
    dict(lens=(2048, 2033, 99), score=synth.SCORE_REPMAX, reps=4),
])
@pytest.mark.parametrize("splits", [0, 2])
def test_stage_1_in_the_same_launch(kw, splits):
    w = dataclasses.replace(_workload(**{k: v for k, v in kw.items() if k != "reps"}), reps_per_partition=kw.get("reps", 1))
    layer, _ = runner.build_device_layer(w, decode_splits=splits)
    layer.step(layer.q0)
    want = layer.scores.clone()
    _same_as_stage_calls(layer, layer.q0)
    layer.scores.fill_(7.0)
    layer.step2(layer.q0)
    assert torch.equal(want, layer.scores)


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [
    dict(lens=(1, 15, 16, 17, 33, 100, 512), topk=40),                # rows as short as the windows; 1 to 3 tiles
    dict(lens=(2048, 2047, 700), topk=128, sink=0, recent=0),         # 4 scores per thread
    dict(lens=(4096, 3001), topk=300),                                # 8
    dict(lens=(8192, 5000), topk=1025, sink=1, recent=2),             # 16; more entries than threads
    dict(lens=(16384, 16001, 9), topk=2048),                          # 32
    dict(lens=(8193, 9000, 3), topk=512),                             # by the tiles' maxima: 4 per thread
    dict(lens=(8193, 9000, 3), topk=514),                             # 32 scores per thread: more tiles wanted than there are
    dict(lens=(16385, 40000, 65536, 20), topk=1024, sink=0, recent=0),    # 8 maxima per thread
    dict(lens=(131072, 70001), topk=333),                             # 16
    dict(lens=(17000, 20000), topk=2048, heads=32),                   # walked whole; 16 heads to a group
    dict(lens=(9001, 30), part=2, topk=200, score=synth.SCORE_MINMAX),
    dict(lens=(9001, 29), part=4, topk=99, score=synth.SCORE_MINMAX, incl=False, heads=10),
    dict(lens=(9001, 27), part=8, topk=70, score=synth.SCORE_MINMAX, leaf=3),
    dict(lens=(300000, 140001), part=8, topk=50, score=synth.SCORE_MINMAX),
    dict(lens=(300 * 16, 999), leaf=1, topk=100),                     # a directory of more than 256 entries
])
@pytest.mark.parametrize("splits", [0, 1, 3])
def test_partitions_smaller_than_a_page(kw, splits):
    layer, _ = runner.build_device_layer(_workload(**dict(dict(part=1, score=synth.SCORE_SKETCH), **kw)), decode_splits=splits)
    assert layer.spin.fused_splits >= 1
    _same_as_stage_calls(layer, layer.q0)


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [
    dict(lens=(131073, 262144, 50000), topk=200),                     # 4 maxima per thread, and 32 scores where rows are many:
    dict(lens=(131073,) + (5000,) * 16, topk=200),
    dict(lens=(600000, 262145, 5, 70000), topk=128),                  # 8
    dict(lens=(1048576, 1100001), topk=256, sink=4, recent=8, kv=1, heads=4),    # 16
    dict(lens=(300000,), topk=2000, sink=100, recent=200),            # walked whole; windows of more than a page a wavefront
    dict(lens=(300000, 280001), topk=64, leaf=6),                     # leaves that are no power of two
    dict(lens=(600001, 30000), part=32, topk=30, incl=False, sink=3, recent=9),
])
@pytest.mark.parametrize("splits", [0, 1, 3])
def test_rows_beyond_the_registers(kw, splits):
    layer, _ = runner.build_device_layer(_workload(**kw), decode_splits=splits)
    assert layer.spin.fused_splits >= 1
    _same_as_stage_calls(layer, layer.q0)


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [
    dict(lens=(100, 1, 17, 5000), part=64, topk=5),                   # rows as short as the windows
    dict(lens=(20000, 31001), part=256, topk=32, incl=False, recent=16),    # 4 scores per thread
    dict(lens=(65536, 9000), part=16, topk=100),                      # 8: partitions of at most a page
    dict(lens=(131072, 70000), part=32, topk=60, incl=False, sink=0, recent=0),    # 16
    dict(lens=(262144,), part=64, topk=40, incl=False, sink=9, recent=30, kv=1, heads=16),    # 32; 16 heads to a group
    dict(lens=(30000,), part=128, topk=700, score=synth.SCORE_REPMAX),
])
@pytest.mark.parametrize("splits", [0, 1, 3])
def test_variable_length_partitions(kw, splits):
    w = _workload(**kw)
    dd = synth.generate_on_device(w)
    layer = runner.LayerState.from_natural_pool(w, dd.slot_of, dd.pool, layouts=synth.variable_layouts(w, 5),
                                                decode_splits=splits)
    layer.build_summaries()
    assert layer.spin.fused_splits >= 1
    _same_as_stage_calls(layer, dd.q)


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [
    dict(lens=(30000, 8000), topk=64),
    dict(lens=(30000, 8000), topk=500, part=1, score=synth.SCORE_SKETCH),
    dict(lens=(9000, 8000), topk=300, part=1, score=synth.SCORE_SKETCH),
    dict(lens=(300000, 8000), topk=64),
])
def test_scores_that_tie_or_are_not_finite(kw):
    layer, _ = runner.build_device_layer(_workload(**kw))
    sp, w = layer.spin, layer.w
    for fill in ("ties", "inf", "nan", "spread"):
        gen = torch.Generator(device="cuda:0")
        gen.manual_seed(5)
        layer.scores.normal_(generator=gen)
        pick = torch.rand(layer.scores.shape, generator=gen, device="cuda:0")
        if fill == "ties":
            layer.scores.copy_((layer.scores * 2).round())
        elif fill == "inf":
            layer.scores[pick < 0.01] = float("inf")
            layer.scores[pick > 0.5] = float("-inf")
        elif fill == "nan":
            layer.scores[pick < 0.999] = float("nan")                 # fewer numbers than are wanted
        else:
            layer.scores.mul_(torch.exp2(pick * 200 - 100))
        sp.select_topk(w.batch, layer.scores, layer.part_offsets, layer.seq_lens, layer.sel, layer.nsel, layer.ws)
        want = layer.sel.clone()
        layer.sel.fill_(7)
        sp.select_resolve_decode(w.batch, layer.scores, layer.part_offsets, layer.seq_lens, layer.sel, layer.nsel,
                                 layer.dir, layer.leaf_pool, layer.slots, layer.page_ids, layer.valid_mask, layer.npages,
                                 layer.q0, layer.kv_pool, layer.out, layer.lse, layer.ws)
        assert torch.equal(want, layer.sel), fill
    assert layer.status() == 0


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [dict(), dict(part=1, score=synth.SCORE_SKETCH, topk=90), dict(part=4, topk=60)])
def test_pages_that_are_missing_or_outside_the_pool(kw):
    for slot, code, note in ((-1, -6, "not resident"), (1 << 30, -7, "outside the pool")):
        layer, _ = runner.build_device_layer(_workload((5000, 3000), **dict(dict(topk=30, sink=0, recent=0), **kw)))
        layer.step(layer.q0)
        chosen = int(layer.page_ids[1, 7])                            # row 1: request 0, head 1
        chunk = int(layer.dir[1, chosen // layer.w.leaf_entries])
        layer.leaf_pool[chunk, chosen % layer.w.leaf_entries] = slot
        layer.step(layer.q0)
        want = {n: getattr(layer, n).clone() for n in LISTS + ("out",)}
        assert layer.status() == code
        layer.spin.workspace_init(layer.ws)
        layer.step2(layer.q0)
        assert layer.status() == code, note
        for n in LISTS:
            assert torch.equal(want[n], getattr(layer, n)), (note, n)
        assert (layer.out.float() - want["out"].float()).abs().max() <= 2 ** -6 * want["out"].float().abs().max()


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [
    dict(lens=(5000, 3000)),                                          # stage 1 in the same launch
    dict(lens=(40000, 3000)),                                         # the first forced pages asked for ahead
    dict(lens=(9000, 3000), part=64, topk=9, incl=False),
    dict(lens=(300000, 3000)),                                        # by the tiles' maxima
    dict(lens=(9000, 3000), part=4, topk=90),
])
def test_forced_pages_that_are_missing_or_outside_the_pool(kw):
    for page in (0, 1, -5, -1):                                       # of the sink's two and the window's five
        for slot, code in ((-1, -6), (1 << 30, -7)):
            layer, _ = runner.build_device_layer(_workload(**dict(dict(topk=30), **kw)))
            layer.step(layer.q0)
            page %= -(-kw["lens"][0] // 16)
            chunk = int(layer.dir[1, page // layer.w.leaf_entries])   # row 1: request 0, head 1
            layer.leaf_pool[chunk, page % layer.w.leaf_entries] = slot
            layer.step(layer.q0)
            want = {n: getattr(layer, n).clone() for n in LISTS + ("out",)}
            assert layer.status() == code
            layer.spin.workspace_init(layer.ws)
            layer.step2(layer.q0)
            assert layer.status() == code, (page, slot)
            for n in LISTS:
                assert torch.equal(want[n], getattr(layer, n)), (page, slot, n)
            assert (layer.out.float() - want["out"].float()).abs().max() <= 2 ** -6 * want["out"].float().abs().max()


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [
    dict(lens=(40000, 3000), topk=30),                                # its recent pages are not in the list
    dict(lens=(40000, 3000), topk=300, sink=100, recent=200),         # nor are there as many pages as the windows have
    dict(lens=(9000, 3000), part=64, topk=9),
    dict(lens=(9000, 3000), part=64, topk=20, sink=30, recent=60),
    dict(lens=(300000, 3000), topk=30),
    dict(lens=(5000, 300), topk=30, sink=10, recent=30),
])
@pytest.mark.parametrize("splits", [0, 1, 3])
def test_a_row_longer_than_its_partition_table(kw, splits):
    layer, _ = runner.build_device_layer(_workload(**kw), decode_splits=splits)
    layer.seq_lens[1] = kw["lens"][0] - 100
    layer.step(layer.q0)
    lists = {n: getattr(layer, n).clone() for n in LISTS}
    out, code = layer.out.clone(), layer.status()
    layer.spin.workspace_init(layer.ws)
    layer.step2(layer.q0)
    assert layer.status() == code
    for n in LISTS:
        assert torch.equal(lists[n], getattr(layer, n)), n
    assert (layer.out.float() - out.float()).abs().max() <= 2 ** -6 * out.float().abs().max()


@pytest.mark.gpu
@pytest.mark.parametrize("kw,longest", [
    (dict(lens=(40000, 3000), topk=30, leaf=4096), 32000),            # 2500 pages, of which 4 per thread are 2048
    (dict(lens=(40000, 3000), topk=30, leaf=4096, incl=False), 32000),
    (dict(lens=(32800, 3000), topk=30, leaf=4096, recent=9), 32000),  # 2050: some of the recent ones are kept
    (dict(lens=(70000, 66000), topk=300, leaf=8192, sink=100, recent=250), 60000),    # 8
    (dict(lens=(40000, 3000), topk=30, leaf=4096, part=32), 16 * 2048),
])
def test_a_row_longer_than_its_context(kw, longest):
    w = _workload(**kw)
    dd = synth.generate_on_device(w)
    layer = runner.LayerState.from_natural_pool(w, dd.slot_of, dd.pool, max_context=longest)
    sp, gen = layer.spin, torch.Generator(device="cuda:0")
    gen.manual_seed(3)
    layer.scores.normal_(generator=gen)

    def stage_calls(q):
        sp.select_topk(w.batch, layer.scores, layer.part_offsets, layer.seq_lens, layer.sel, layer.nsel, layer.ws)
        sp.resolve_slots(w.batch, 0, layer.sel, layer.nsel, layer.seq_lens, layer.dir, layer.leaf_pool, layer.slots,
                         layer.page_ids, layer.valid_mask, layer.npages, layer.ws)
        sp.sparse_decode(w.batch, q, layer.kv_pool, layer.slots, layer.valid_mask, layer.npages, layer.out, layer.lse, layer.ws)

    def one_launch(q):
        sp.select_resolve_decode(w.batch, layer.scores, layer.part_offsets, layer.seq_lens, layer.sel, layer.nsel, layer.dir,
                                 layer.leaf_pool, layer.slots, layer.page_ids, layer.valid_mask, layer.npages, q,
                                 layer.kv_pool, layer.out, layer.lse, layer.ws)

    _same(layer, dd.q, stage_calls, one_launch)


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [
    dict(lens=(3000, 4000, 100)),                                     # stage 1 in the same launch
    dict(lens=(40000, 3000, 100)),
    dict(lens=(300000, 3000, 50)),
    dict(lens=(9000, 3000, 70), part=64, topk=9),
    dict(lens=(20000, 900, 8), part=1, score=synth.SCORE_SKETCH),
    dict(lens=(5000, 300, 8), part=4, topk=60),
])
@pytest.mark.parametrize("splits", [0, 3])
def test_rows_without_a_token(kw, splits):
    layer, _ = runner.build_device_layer(_workload(**kw), decode_splits=splits)
    layer.seq_lens[1] = 0
    _same_as_stage_calls(layer, layer.q0)
    assert (layer.out[1] == 0).all() and (layer.lse[1] == float("-inf")).all()


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [dict(lens=(9001, 4000)), dict(lens=(20001, 4000), part=1, score=synth.SCORE_SKETCH)])
def test_replays_of_a_graph(kw):
    layer, _ = runner.build_device_layer(_workload(topk=64, **kw))
    q = layer.q0.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        layer.step2(q)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        layer.step2(q)
    for seed in range(4):
        q.copy_(synth.make_queries_on_device(layer.w, seed, "cuda:0"))
        layer.step2(q)
        want = layer.out.clone()
        layer.out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(layer.out, want)


def test_contexts_that_it_does_not_take():
    base = dict(max_batch=2, num_q_heads=8, num_kv_heads=2, topk=8, max_context=4096)
    assert binding.Spin(**base).fused_splits == 1
    assert binding.Spin(**dict(base, max_batch=1, topk=128, max_context=131072, num_kv_heads=8)).fused_splits == 8
    assert binding.Spin(**dict(base, partition_tokens=8)).fused_splits == 1
    assert binding.Spin(**dict(base, partition_tokens=1, topk=1024, max_context=65536, max_batch=32)).fused_splits == 4
    assert binding.Spin(**dict(base, topk=256, max_context=2097152)).fused_splits == 16
    assert binding.Spin(**dict(base, partition_tokens=64, variable_partitions=1)).fused_splits == 1
    for other in (dict(lru_timestamps=8), dict(decode_waves=4), dict(decode_depth=3), dict(max_context=2097153),
                  dict(partition_tokens=64, variable_partitions=1, max_context=262145), dict(partition_tokens=1, max_context=131073),
                  dict(topk=2305, max_context=65536)):
        sp = binding.Spin(**dict(base, **other))
        assert sp.fused_splits == 0, other
        fake = 4096   # never dereferenced: the call returns before anything is launched
        import ctypes as C
        assert sp.lib.spin_select_resolve_decode(sp.h, 1, fake, fake, fake, fake, fake, fake, fake, C.c_int64(1), fake, fake,
                                                 fake, fake, fake, fake, C.c_int64(1), fake, fake, fake, None) == -2


@pytest.mark.parametrize("kw,launches,kernel", [
    (dict(max_context=32768), 2, "spin_select_decode_kernel<4, true, false, false, 0>"),
    (dict(max_context=4096), 1, "spin_select_decode_kernel<4, true, false, false, 1>"),
    (dict(max_context=4096, score_kind=synth.SCORE_REPMAX, reps_per_partition=1), 1,
     "spin_select_decode_kernel<4, true, false, false, 3>"),
    (dict(max_context=65536), 2, "spin_select_decode_kernel<8, true, false, false, 0>"),
    (dict(max_context=131072), 2, "spin_select_decode_kernel<16, true, false, false, 0>"),
    (dict(max_context=262144), 2, "spin_select_decode_kernel<4, true, true, false, 0>"),
    (dict(max_context=262144, max_batch=17), 2, "spin_select_decode_kernel<32, true, false, false, 0>"),
    (dict(max_context=262144, leaf_entries=6), 2, "spin_select_decode_kernel<4, false, true, false, 0>"),
    (dict(max_context=1000000), 2, "spin_select_decode_kernel<8, true, true, false, 0>"),
    (dict(max_context=65536, partition_tokens=64), 2, "spin_select_decode_kernel<4, false, false, false, 0>"),
    (dict(max_context=65536, partition_tokens=1, topk=1024), 2, "spin_select_decode_tokens_kernel<8, true>"),
    (dict(max_context=8192, partition_tokens=1), 2, "spin_select_decode_tokens_kernel<16, false>"),
    (dict(max_context=4096, lru_timestamps=8), 0, ""),
])
def test_the_kernel_that_a_context_takes(kw, launches, kernel):
    assert binding.Spin(**dict(dict(max_batch=2, num_q_heads=8, num_kv_heads=2, topk=8), **kw)).step_kernel() == (launches, kernel)


@pytest.mark.gpu
def test_the_launches_are_as_many_as_it_says():
    for kw in (dict(lens=(3000, 4000)), dict(lens=(40000, 3000)), dict(lens=(140000, 3000)), dict(lens=(9000,), part=64, topk=9),
               dict(lens=(20000, 900), part=1, score=synth.SCORE_SKETCH)):
        layer, _ = runner.build_device_layer(_workload(**kw))
        sp = layer.spin
        sp.profile_enable(8)
        layer.step2(layer.q0)
        torch.cuda.synchronize()
        ran = {name: sp.profile_read(name)[0] for name in sp.KERNEL_IDS}
        sp.profile_enable(0)
        assert {n: c for n, c in ran.items() if c} == {"select_decode": 1, **({"score": 1} if sp.step_kernel()[0] == 2 else {})}
