"""A lane of a buffer load or store is kept inside the buffer by a check of its own offset; the scalar offset that the
instruction adds is not sure to be part of it.  Stage 1 of sketches lets that check end a row, so every buffer access of
its kernels has to carry its whole offset per lane.  Read from the assembly of this source: no value can show it, since
what lies past a row is never stored.  No GPU is needed."""
import os
import re
import subprocess

import pytest

from paper_2604_26837_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def device_assembly(source, tmp_path):
    """The assembly of one of the library's sources, compiled as the library is."""
    out = str(tmp_path / (source + ".asm"))
    cmd = [HIPCC, *(f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")), "-S", "--offload-device-only",
           "-I", os.path.join(build.ROOT, "include"), "-I", os.path.join(build.PKG_DIR, "csrc"),
           os.path.join(build.PKG_DIR, "csrc", source), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-3000:]
    return out


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_sketch_kernels_pass_no_scalar_offset(tmp_path):
    kernel, seen = None, {}
    with open(device_assembly("spin_score.hip", tmp_path)) as f:
        for line in f:
            label = re.match(r"(_Z\w*spin_score_sketch\w*):", line)
            if label:
                kernel = label.group(1)
                seen[kernel] = {"load": 0, "store": 0}
            elif line.startswith(".Lfunc_end"):
                kernel = None
            access = kernel and re.match(r"\s+buffer_(load|store)_\w+ (.*)", line)
            if access:
                operands = [x.strip() for x in re.sub(r"\[[^]]*\]", "", access.group(2)).split(",")]
                # data, lane offset, buffer, scalar offset and modifiers
                assert len(operands) == 4 and operands[3].split()[0] == "0", line
                seen[kernel][access.group(1)] += 1
    assert len(seen) == 8 and all(n["load"] and n["store"] for n in seen.values()), seen
