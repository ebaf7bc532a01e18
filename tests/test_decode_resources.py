"""What the compiler gave the decode kernels (CPU only): an instance whose
blocks are meant to share a CU two and two fits there twice.  A gfx950 CU has
163,840 bytes of LDS and, per SIMD, 512 vector registers per lane; two blocks
of 8 waves (head_dim 128) put four waves on a SIMD, two blocks of 4 (256) two.
Read from the metadata of the built library's own code objects."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2609_17475_amd import build

LLVM = "/opt/rocm/llvm/bin/"
pytestmark = pytest.mark.skipif(not os.path.exists(LLVM + "llvm-readelf"), reason="no ROCm tools")


def kernels(tmp_path):
    """{(d, group, append, column sets, stages): (LDS bytes, registers)}"""
    lib = shutil.copy(build.LIB, tmp_path)
    subprocess.run([LLVM + "llvm-objdump", "--offloading", lib], cwd=tmp_path, check=True,
                   capture_output=True)
    found = {}
    for f in os.listdir(tmp_path):
        if "gfx950" not in f:
            continue
        notes = subprocess.run([LLVM + "llvm-readelf", "--notes", os.path.join(tmp_path, f)],
                               check=True, capture_output=True, text=True).stdout
        for k in notes.split("  - .agpr_count")[1:]:
            name = re.search(r"decode_kernelILi(\d+)ELi(\d+)ELb(\d)ELi(\d)ELi(\d)E", k)
            if name:
                found[tuple(int(x) for x in name.groups())] = tuple(
                    int(re.search(r"\." + key + r": +(\d+)", k).group(1))
                    for key in ("group_segment_fixed_size", "vgpr_count"))
    return found


def test_paired_instances_fit_twice(tmp_path):
    found = kernels(tmp_path)
    pairs = {k: v for k, v in found.items() if k[0] >= 128 and k[4] == 2}
    # head_dim, group, fused append or not
    assert {k[:3] for k in pairs} == {(d, g, a) for d in (128, 256) for g in (32, 64, 128) for a in (0, 1)}
    for (d, *_), (lds, regs) in pairs.items():
        assert 2 * lds <= 163840 and regs <= (128 if d == 128 else 256), (pairs, d, lds, regs)
