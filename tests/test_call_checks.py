"""What the stage calls refuse before anything is launched: tensors that are not on the GPU, not contiguous or of
another type than documented, and arguments that are no tensors or no integers; a tensor subclass is as good as a
plain tensor."""
import numpy as np
import pytest
import torch

from paper_2604_26837_amd import binding, runner, synth


def _spin():
    return binding.Spin(max_batch=1, num_q_heads=4, num_kv_heads=1, topk=4, max_context=1024)


def test_refusals_without_a_gpu():
    sp = _spin()
    t = torch.zeros(64, dtype=torch.int32)
    with pytest.raises(ValueError, match="scores must live on the GPU"):
        sp.select_topk(1, t.float(), t, t, t, t, t)
    with pytest.raises(AttributeError):
        sp.sparse_decode(1, None, None, t, t, t, t, t, t)                 # a pool has a size, so it has to be there
    with pytest.raises(AttributeError):
        sp.select_topk(1, [1.0], t, t, t, t, t)
    for batch in (1.0, "1", None, np.float32(1), torch.tensor(1.0), torch.tensor([1, 1])):
        with pytest.raises(TypeError):
            sp.select_topk(batch, t.float(), t, t, t, t, t)


def test_integers_of_any_kind():
    """A batch or a step is often an element of a numpy array or of a tensor: it is as good as Python's integer (the
    call goes on to the tensors behind it)."""
    sp = _spin()
    t = torch.zeros(64, dtype=torch.int32)
    for one in (1, np.int32(1), np.int64(1), np.uint8(1), torch.tensor(1), np.array([1])[0]):
        with pytest.raises(ValueError, match="scores must live on the GPU"):
            sp.select_topk(one, t.float(), t, t, t, t, t)
        with pytest.raises(ValueError, match="sel must live on the GPU"):
            sp.resolve_slots(one, one, t, t, t, t, t, t, t, t, t, t)


@pytest.mark.gpu
def test_refusals_and_subclasses_on_the_gpu():
    w = synth.config0()
    layer, _ = runner.build_device_layer(w)
    sp, q = layer.spin, layer.q0
    with pytest.raises(binding.SpinError) as e:                           # NULL pointers are the library's to refuse
        sp.select_topk(1, None, None, None, None, None, None)
    assert e.value.code == -1
    sp.select_topk(0, None, None, None, None, None, None)                 # an empty batch is nothing to do
    with pytest.raises(binding.SpinError):
        sp.select_topk(w.batch + 1, None, None, None, None, None, None)   # more than max_batch
    sp.select_topk(np.int64(0), None, None, None, None, None, None)
    with pytest.raises(binding.SpinError):
        sp.select_topk(np.int32(-1), None, None, None, None, None, None)
    args = [np.int64(w.batch), layer.scores, layer.part_offsets, layer.seq_lens, layer.sel, layer.nsel, layer.ws]
    for at, bad, text in ((1, layer.scores.half(), "scores must be torch.float32, got torch.float16"),
                          (2, layer.part_offsets.long(), "part_offsets must be torch.int32, got torch.int64"),
                          (4, layer.sel.t().expand(-1, w.rows), "sel must be contiguous"),
                          (3, layer.seq_lens.cpu(), "seq_lens must live on the GPU")):
        with pytest.raises(ValueError, match=text):
            sp.select_topk(*args[:at], bad, *args[at + 1:])

    class Tagged(torch.Tensor):
        pass

    layer.step_fused(q)
    want = layer.out.clone()
    layer.out.zero_()
    layer.kv_pool, layer.leaf_pool = layer.kv_pool.as_subclass(Tagged), layer.leaf_pool.as_subclass(Tagged)
    layer.step_fused(q.as_subclass(Tagged))
    assert torch.equal(layer.out, want) and want.float().abs().sum() > 0
    with pytest.raises(ValueError, match="q must be torch.bfloat16, got torch.float32"):
        layer.step_fused(q.float().as_subclass(Tagged))
    with pytest.raises(ValueError, match="kv_pool must be contiguous"):
        sp.sparse_decode(w.batch, q, layer.kv_pool[:, ::2], layer.slots, layer.valid_mask, layer.npages, layer.out,
                         layer.lse, layer.ws)
