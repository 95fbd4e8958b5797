"""Small batches in a context sized for many requests, in every form of stage 4 (plain, after the always-attended
pages, in two passes, with the static scratch): to the tolerance of a bf16 output of two summation orders the attention
of a context with one split, and a request's output bits do not depend on how many others share its call."""
import pytest
import torch

from paper_2604_26837_amd import runner, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("batch,max_batch,heads,kv,topk,tp", [(1, 16, 8, 2, 32, 16), (3, 16, 32, 8, 64, 16), (1, 1, 16, 1, 200, 16),
                                                              (2, 40, 128, 8, 40, 16), (2, 9, 8, 2, 6, 128), (5, 5, 8, 8, 9, 16), (4, 4, 128, 8, 128, 16)])
def test_any_batch_of_a_larger_context(batch, max_batch, heads, kv, topk, tp):
    w = synth.config0().with_(seq_lens=tuple(4003 + 517 * b for b in range(batch)), num_q_heads=heads, num_kv_heads=kv,
                              topk=topk, partition_tokens=tp, sink_pages=2, recent_pages=5, topk_includes_forced=tp == 16,
                              name="small_batch")
    one, _ = runner.build_device_layer(w, decode_splits=1)
    many, _ = runner.build_device_layer(w, max_batch=max_batch)
    one.step(one.q0)
    want = one.out.float()

    def check(out, lse=None):
        torch.cuda.synchronize()
        assert many.status() == 0
        # fp32 sums of unrounded probabilities in two orders: a few hundred roundings of 2^-24, exp2's last bit
        if lse is not None:
            assert (lse - one.lse).abs().max() <= 4e-5
        # probabilities are rounded to bf16 (2^-9) before they meet the values, the output once more: two orders of
        # the same sum differ by a few units of the last place of the largest term
        assert (out.float() - want).abs().max() <= 2 ** -6 * want.abs().max()
        assert torch.equal(many.slots, one.slots) and torch.equal(many.npages, one.npages)

    sp, args = many.spin, (w.batch, many.q0, many.kv_pool, many.slots, many.valid_mask, many.npages)
    for form in (many.step, many.step_fused, many.step_fused):       # (twice: the tickets are left cleared)
        many.out.zero_()
        many.lse.zero_()
        form(many.q0)
        check(many.out, many.lse)
    sp.sparse_decode(*args, many.out, many.lse, many.ws)
    plain = many.out.clone()
    check(plain, many.lse)
    static = torch.zeros_like(plain)
    many.lse.zero_()
    sp.sparse_decode_static(*args, static, many.lse)
    check(static, many.lse)
    assert torch.equal(static, plain)
    first = many.valid_mask.clone()
    first[:, 1::2] = 0
    sp.sparse_decode_begin(*args[:4], first, many.npages, many.ws)
    sp.sparse_decode_finish(*args[:4], many.valid_mask - first, many.npages, many.out, many.lse, many.ws)
    check(many.out, many.lse)


@pytest.mark.parametrize("batch,heads,kv,topk,tp", [(16, 32, 8, 64, 16), (16, 8, 2, 70, 16), (5, 128, 8, 128, 16),
                                                    (16, 8, 2, 6, 128)])
def test_bits_of_a_request_in_any_batch(batch, heads, kv, topk, tp):
    w = synth.config0().with_(seq_lens=tuple(4003 + 17 * b for b in range(batch)), num_q_heads=heads, num_kv_heads=kv,
                              topk=topk, partition_tokens=tp, sink_pages=2, recent_pages=5, topk_includes_forced=tp == 16,
                              name="any_batch")
    layer, _ = runner.build_device_layer(w)
    sp = layer.spin

    def static(q):
        layer.step(q)
        sp.sparse_decode_static(layer.w.batch, q, layer.kv_pool, layer.slots, layer.valid_mask, layer.npages, layer.out,
                                layer.lse)

    def two_passes(q):
        layer.step(q)
        args = (layer.w.batch, q, layer.kv_pool, layer.slots)
        first = layer.valid_mask.clone()
        first[:, 1::2] = 0
        sp.sparse_decode_begin(*args, first, layer.npages, layer.ws)
        sp.sparse_decode_finish(*args, layer.valid_mask - first, layer.npages, layer.out, layer.lse, layer.ws)

    for form in (layer.step, layer.step_fused, static, two_passes):
        layer.w = w
        form(layer.q0)
        out, lse = layer.out.clone(), layer.lse.clone()
        for n in (1, 3, batch // 2):                                 # the first n requests alone
            layer.w = w.with_(seq_lens=w.seq_lens[:n])
            layer.out.zero_()
            form(layer.q0[:n].contiguous())
            assert torch.equal(layer.out[:n], out[:n]) and torch.equal(layer.lse[:n], lse[:n])
    torch.cuda.synchronize()
    assert layer.status() == 0
