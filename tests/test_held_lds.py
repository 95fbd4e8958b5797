"""The launches of stages 2+3 that hand a selection over in memory reserve no LDS for it.  No GPU is needed."""
import os
import re

import pytest

from test_buffer_range import HIPCC, device_assembly

SEL_HELD = 2304                # of csrc/spin_resolve_dev.h


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_selections_in_memory_take_no_lds(tmp_path):
    with open(device_assembly("spin_select_resolve.hip", tmp_path)) as f:
        text = f.read()
    lds = {}
    for size, name, shape, held in re.findall(r"\.group_segment_fixed_size: (\d+)\n(?:.*\n)*?\s+\.name:\s+"
                                              r"_Z\d+(spin_select_resolve\w*?_kernel)I((?:Li\d+E)+)Lb([01])E", text):
        lds[name, shape, held] = int(size)
    in_memory = [k for k in lds if k[2] == "0"]
    assert {k[0] for k in in_memory} == {"spin_select_resolve_kernel", "spin_select_resolve_forced_kernel"}, lds
    for name, shape, _ in in_memory:      # (all but a word of it, and what aligning the rest takes)
        assert lds[name, shape, "1"] - lds[name, shape, "0"] >= (SEL_HELD - 4) * 4, (name, shape, lds)
