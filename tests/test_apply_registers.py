"""The apply kernels' registers as compiled for gfx950 (CPU): at most 96, so
that a seam-estimate wave finds room beside the four waves per SIMD of two
workgroups, and none spilled."""
import os
import re
import subprocess

import pytest

from paper_1910_03517_amd import build as bld


@pytest.mark.skipif(not os.path.exists(bld.HIPCC), reason="needs hipcc")
def test_apply_kernels_fit_their_registers(tmp_path):
    asm = os.path.join(tmp_path, "k_apply.s")
    flags = [f for f in bld.CFLAGS if f != "-fPIC"]
    subprocess.run([bld.HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(bld.CSRC, "k_apply.hip"), "-o", asm],
                   check=True, capture_output=True)
    with open(asm) as f:
        meta = re.findall(r"- \.agpr_count.*?\.wavefront_size", f.read(), re.S)
    assert len(meta) == 7
    for m in meta:
        val = {k: int(re.search(rf"\.{k}:\s+(\d+)", m).group(1)) for k in
               ("vgpr_count", "agpr_count", "vgpr_spill_count", "private_segment_fixed_size")}
        name = re.search(r"\.name:\s+(\S+)", m).group(1)
        assert val["vgpr_count"] + val["agpr_count"] <= 96, (name, val)
        assert val["vgpr_spill_count"] == 0 and val["private_segment_fixed_size"] == 0, (name, val)
