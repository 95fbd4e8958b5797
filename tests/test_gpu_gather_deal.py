"""The copy kernel deals the pages of all rows to its wavefronts one by one: every listed page arrives, whatever the
rows' counts are (none at all, one row with everything, more rows than one round of prefix sums holds), and nothing
else is touched.  Bytes are moved, so the comparison is exact."""
import numpy as np
import pytest
import torch

from paper_2604_26837_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("to_host", [False, True])
@pytest.mark.parametrize("batch,heads,counts", [(1, 1, "full"), (3, 2, "none"), (8, 8, "few"), (5, 1, "one_row"),
                                                (130, 8, "random"), (257, 4, "random")])
def test_every_listed_page_is_copied(batch, heads, counts, to_host):
    rng = np.random.Generator(np.random.PCG64(batch * 10 + heads))
    sp = binding.Spin(max_batch=batch, num_q_heads=heads, num_kv_heads=heads, score_kind=0, topk=5, max_context=16 * 40)
    rows, stride = batch * heads, sp.page_stride
    n = {"full": np.full(rows, stride), "none": np.zeros(rows, dtype=np.int64), "few": rng.integers(0, 3, rows),
         "one_row": np.where(np.arange(rows) == rows - 1, stride, 0), "random": rng.integers(0, stride + 1, rows)}[counts]
    per_row = 7                                        # host pages and slots of a row
    host = torch.empty((rows * per_row, 4096), dtype=torch.int16, pin_memory=True)
    host.copy_(torch.from_numpy(rng.integers(-2 ** 15, 2 ** 15, (rows * per_row, 4096), dtype=np.int16)))
    pool = torch.from_numpy(rng.integers(-2 ** 15, 2 ** 15, (rows * per_row, 4096), dtype=np.int16)).to(DEV)
    base = torch.arange(rows, dtype=torch.int64) * per_row
    slots_all = rng.permutation(rows * per_row).astype(np.int32).reshape(rows, per_row)
    pages, slots = np.full((rows, stride), -1, dtype=np.int32), np.full((rows, stride), -1, dtype=np.int32)
    for r in range(rows):
        pages[r, :n[r]] = np.sort(rng.permutation(per_row)[:n[r]])
        slots[r, :n[r]] = slots_all[r, :n[r]]
    want_host, want_pool = host.numpy().copy(), pool.cpu().numpy()
    for r in range(rows):
        hp = r * per_row + pages[r, :n[r]]
        if to_host:
            want_host[hp] = want_pool[slots[r, :n[r]]]
        else:
            want_pool[slots[r, :n[r]]] = want_host[hp]
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV)
    ws = sp.new_workspace(DEV)
    if to_host:
        sp.offload_pages(batch, pool, host, base.to(DEV), d(n), d(pages), d(slots), ws)
    else:
        sp.gather_misses(batch, host, base.to(DEV), d(n), d(pages), d(slots), pool, ws)
    torch.cuda.synchronize()
    assert sp.poll_status(ws) == 0
    assert np.array_equal(pool.cpu().numpy(), want_pool)
    assert np.array_equal(host.numpy(), want_host)
