"""Stage 2 of rows of 4097 to 16384 partitions: most scores are ruled out by a bound taken from the threads'
largest scores, and the exact search runs on a list of the rest.  Bit-exact against the oracle at the row lengths
and selection sizes where a thread's share, the use of the bound or the list's capacity changes."""
import numpy as np
import pytest

from paper_2604_26837_amd import synth
from test_gpu_stages import _check_select

pytestmark = pytest.mark.gpu

# 512 or 1024 threads with 16 scores each: the bound is used while 1.5 k' threads hold a candidate, the list holds
# 1024 or 2048 entries
SIZES = [(4097, 1), (4097, 171), (4097, 172), (5000, 400), (8191, 340), (8192, 341), (8192, 342), (8193, 128),
         (8193, 343), (12345, 682), (16383, 682), (16384, 683), (16384, 116), (16384, 5000)]


@pytest.mark.parametrize("parts,topk", SIZES)
def test_filtered_rows(parts, topk):
    rng = np.random.default_rng(parts * 7 + topk)
    # the context is sized for the longest row; the others use a part of it
    lens = (parts * 16, parts * 16 - 5, max(parts // 3, 1) * 16, 40 * 16)
    w = synth.config0().with_(num_q_heads=4, num_kv_heads=1, seq_lens=lens, topk=topk, topk_includes_forced=True,
                              sink_pages=2, recent_pages=3, name="filtered")
    smooth = [(rng.standard_normal(w.partitions(b)) * 10 + 150).astype(np.float32) for b in range(4)]
    ties = [np.round(x / 4).astype(np.float32) for x in smooth]
    equal = [np.full(len(x), 2.0, dtype=np.float32) for x in smooth]
    # one thread's share holds everything large: the bound admits the fewest threads
    clustered = [np.where(np.arange(len(x)) // 16 % 37 == 5, x + 1000, -x).astype(np.float32) for x in smooth]
    specials = [x.copy() for x in smooth]
    for x in specials:
        idx = rng.choice(len(x), size=len(x) // 2, replace=False)
        x[idx] = rng.choice(np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 1e-40], dtype=np.float32), size=idx.size)
    nans = [np.where(rng.random(len(x)) < 0.995, np.nan, x).astype(np.float32) for x in smooth]
    for rows in (smooth, ties, equal, clustered, specials, nans):
        _check_select(w, rows)
