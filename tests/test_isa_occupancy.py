"""Registers of the compositors (CPU): every variant that renders a frame or its
backward leaves room for the four wavefronts per SIMD that their grids assume
(512 registers per SIMD, so at most 128 each) and spills none to memory.  The
variants that count statistics are not held to it."""
import os
import re
import subprocess

import pytest

from paper_2508_03180_amd import build as hipbuild


def kernels(src, tmp):
    out = str(tmp / (src + ".s"))
    subprocess.check_call([hipbuild.HIPCC, *hipbuild.FLAGS, "--cuda-device-only", "-S",
                           os.path.join(hipbuild.CSRC, src), "-o", out], stderr=subprocess.DEVNULL)
    with open(out) as f:
        text = f.read()
    for m in re.finditer(r"\.name:\s+(\S+)\n(.*?)\.wavefront_size", text, re.S):
        field = lambda k: int(re.search(re.escape(k) + r":\s+(\d+)", m.group(2)).group(1))  # noqa: E731
        yield m.group(1), field(".vgpr_count"), field(".private_segment_fixed_size")


@pytest.mark.skipif(not os.path.exists(hipbuild.HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("src,pattern,count", [("backward.hip", r"k_composite_bwd", 4),
                                               ("composite.hip", r"k_compositeILi\dELb0E", 7)])
def test_four_wavefronts_per_simd(tmp_path, src, pattern, count):
    found = [k for k in kernels(src, tmp_path) if re.search(pattern, k[0])]
    assert len(found) == count
    for name, vgprs, scratch in found:
        assert vgprs <= 128 and scratch == 0, (name, vgprs, scratch)
