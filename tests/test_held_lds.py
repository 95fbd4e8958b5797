"""The launches of stages 2+3 that hand a selection over in memory reserve no LDS for it, and no launch asks for more LDS
than a compute unit has.  No GPU is needed."""
import os
import re
import subprocess

import pytest

from paper_2604_26837_amd import build
from test_buffer_range import HIPCC, device_assembly

READELF = os.path.join(os.path.dirname(HIPCC), "..", "llvm", "bin", "llvm-readelf")
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


def _static_lds(library, tmp_path):
    """Every kernel's own LDS, from the notes of the GPU code objects inside a shared library."""
    with open(library, "rb") as f:
        image = f.read()
    lds = {}
    for m in re.finditer(rb"\x7fELF\x02\x01\x01\x40", image):       # 64-bit, little endian, AMDGPU
        path = tmp_path / "object"
        path.write_bytes(image[m.start():])
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for size, name in re.findall(r"\.group_segment_fixed_size: (\d+)\n(?:.*\n)*?\s+\.name:\s+(_Z\w+)\n", notes):
            lds[name] = int(size)
    return lds


@pytest.mark.skipif(not os.path.exists(READELF), reason="llvm-readelf not installed")
def test_launches_fit_a_compute_unit(tmp_path):
    """A kernel's own LDS beside the most that a context may ask for at its launch."""
    if not os.path.exists(build.LIB_PATH):
        build.build_library()
    with open(os.path.join(build.PKG_DIR, "csrc", "spin_common.h")) as f:
        fused = 1024 * int(re.search(r"#define SPIN_FUSED_LDS \((\d+) \* 1024\)", f.read()).group(1))
    merge = 8 * 16 * (128 + 2) * 4                                    # 8 wavefronts' partials of a group of 16 heads
    most = {"spin_select_decode": fused, "spin_gather_decode": merge, "spin_select_resolve_forced": merge,
            "spin_decode_tokens": merge + 8 * 1024 * 4, "spin_decode": merge}
    seen = dict.fromkeys(most, 0)
    for name, size in _static_lds(build.LIB_PATH, tmp_path).items():
        part = next((p for p in most if re.match(r"_Z\d+" + p + "_", name)), None)
        if part:
            seen[part] += 1
        assert size + most.get(part, 0) <= 160 * 1024, (name, size)
    assert all(seen.values()), seen
