"""Properties of the device code that no run shows reliably, read from the assembly of this build's sources."""
import os
import re
import subprocess

import pytest

from paper_1606_07822_amd import _build

pytestmark = pytest.mark.slow


def kernel_instructions(tmp_path, source, kernel):
    if not os.path.exists(_build.HIPCC):
        pytest.skip("hipcc not found")
    out = str(tmp_path / "k.s")
    subprocess.check_call([_build.HIPCC, *_build.FLAGS, "-S", "--cuda-device-only", os.path.join(_build.CSRC, source),
                           "-o", out], stderr=subprocess.DEVNULL)
    with open(out) as f:
        text = f.read()
    body = re.search(rf"^_Z\w*{kernel}\w*:.*?\n(.*?)^\.Lfunc_end", text, re.M | re.S).group(1)
    return [line.strip() for line in body.splitlines() if re.match(r"\s+[a-z]+_", line)]


def test_tree_merge_waits_for_its_stores_at_the_grid_barrier(tmp_path):
    """Each wavefront's stores have to be in the L2 before one wavefront of the workgroup writes it back for the
    other dies: the workgroup barrier before a write-back follows a wait with no store after it."""
    ins = kernel_instructions(tmp_path, "huffman.hip", "k_huff_merge")
    pending, grid_barriers = False, 0
    for i, op in enumerate(ins):
        if op.startswith("global_store"):
            pending = True
        elif re.search(r"s_waitcnt.*vmcnt\(0\)", op):
            pending = False
        elif op.startswith("s_barrier"):
            after = ins[i + 1:i + 12]
            if any(x.startswith("buffer_wbl2") for x in after) and not any(x.startswith("s_barrier") for x in after):
                grid_barriers += 1
                assert not pending, f"instruction {i}: a store may still be on its way"
    assert grid_barriers == 2   # after the first merge, and at the end of a generation
