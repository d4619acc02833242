"""Lanes of a wave exchange values through LDS in the ray loop (the miss table,
a ray's slot words) without a barrier of the workgroup.  What one lane writes
and another reads has to be ordered by wavefront fences, or the compiler may
keep a lane's own last value of a word that another lane has written."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2309_04393_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")
@pytest.mark.parametrize("inst", ["1, 1, false, 18, 0, 4", "4, 2, false, 34, 2, 4"])
def test_lds_exchange_is_fenced(tmp_path, inst):
    src = tmp_path / "one.hip"
    src.write_text('#define RO_PART 9\n#include "render.hip"\n'
                   "const void *instance() { return (const void *)&ro::k_render<%s>; }\n" % inst)
    out = tmp_path / "one.ll"
    subprocess.run([HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "--cuda-device-only", "-emit-llvm", "-S",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, str(src), "-o", str(out)],
                   check=True, capture_output=True, timeout=300)
    ir = out.read_text()
    # the table's clear, a unit's first words, before and after the visits, and
    # in each of the two flushes before and after the entry is written
    for order in ("release", "acquire"):
        n = len(re.findall(r'fence syncscope\("wavefront"\) ' + order, ir))
        assert n >= 8, (order, n)
