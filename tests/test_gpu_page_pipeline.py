"""The loop over a wavefront's pages: fewer pages than register buffers, a remainder behind the last full round, more than
one batch of 64, empty and partial masks among them, and a pool at any address its elements can have.  Against the fp64
oracle to stage 4's tolerance; a page with an empty mask is not read, so that NaNs in it go nowhere."""
import numpy as np
import pytest
import torch

from paper_2604_26837_amd import synth
from test_gpu_decode import _compare, _oracle_rows, _run_decode

pytestmark = pytest.mark.gpu


def _lists(w, rng, n):
    pl, ml = [], []
    for r in range(w.rows):
        p = sorted(int(x) for x in rng.choice(w.pages(0), size=n, replace=False))
        m = [0xFFFF] * n
        for i in rng.choice(n, size=n // 3, replace=False):
            m[i] = int(rng.choice((0, int(rng.integers(1, 1 << 16)))))
        pl.append(p)
        ml.append(m)
    return pl, ml


@pytest.mark.parametrize("depth", [2, 3, 4])
@pytest.mark.parametrize("waves,pages", [(8, 1), (8, 7), (8, 9), (8, 16), (8, 23), (8, 47), (2, 127), (2, 128), (2, 131),
                                         (2, 300)])
def test_any_number_of_pages_per_wavefront(waves, pages, depth):
    from gpu_harness import DeviceWorkload
    w = synth.config0().with_(seq_lens=(16 * 320,), topk=300, name="pipeline")
    dw = DeviceWorkload(synth.generate(w), decode_splits=1, decode_waves=waves, decode_depth=depth)
    rng = np.random.default_rng(100 * pages + depth)
    pl, ml = _lists(w, rng, pages)
    ref, lref = _oracle_rows(dw, pl, ml)
    for r, (p, m) in enumerate(zip(pl, ml)):            # after the oracle's copy of the keys was taken
        for pg, mask in zip(p, m):
            if mask == 0:
                dw.kv_pool[dw.page_map[(r, pg)]] = float("nan")
    got, lgot = _run_decode(dw, pl, ml)
    _compare(got, ref, lgot, lref)


@pytest.mark.parametrize("elements", [1, 2, 3, 8])
def test_pool_at_any_element_offset(elements):
    from gpu_harness import DEV, DeviceWorkload
    w = synth.config0().with_(seq_lens=(16 * 320,), topk=300, name="pipeline")
    dw = DeviceWorkload(synth.generate(w))
    pl, ml = _lists(w, np.random.default_rng(elements), 40)
    want, lwant = _run_decode(dw, pl, ml)
    whole = torch.empty(dw.kv_pool.numel() + 64, dtype=torch.bfloat16, device=DEV)
    moved = whole[elements:elements + dw.kv_pool.numel()].view_as(dw.kv_pool)
    moved.copy_(dw.kv_pool)
    dw.kv_pool = moved
    got, lgot = _run_decode(dw, pl, ml)
    assert np.array_equal(got, want) and np.array_equal(lgot, lwant)
