"""The wide passes of exact distances as compiled: all loads of a pass are
issued before the first wait on one of them."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2206_11408_amd import build

PROGRAM = """
#include "search_kernel.h"
namespace finger { namespace {
template __global__ void %s(KArgs);
} }
"""


@pytest.mark.skipif(not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)), reason="needs hipcc")
@pytest.mark.parametrize("kernel,loads", [("k_search_few<FINGER_MODE_PLAIN, FINGER_CODE_F32, 32, 4, 0>", 32),
                                          ("k_search<FINGER_MODE_PLAIN, FINGER_CODE_F32, 64, 4, false, 0, true>", 32),
                                          ("k_search<FINGER_MODE_PLAIN, FINGER_CODE_F32, 64, 8, false, 0, true>", 32),
                                          ("k_search<FINGER_MODE_FINGER, FINGER_CODE_BF16, 64, 4, false, 8, true>", 32)])
def test_wide_pass_loads_together(tmp_path, kernel, loads):
    src, out = tmp_path / "one.hip", tmp_path / "one.s"
    src.write_text(PROGRAM % kernel)
    subprocess.run([build.HIPCC, *build.FLAGS, "-w", "-I", build.CSRC, "-S", "--cuda-device-only", str(src), "-o", str(out)],
                   check=True, capture_output=True)
    run = best = 0
    for line in out.read_text().splitlines():
        line = line.strip()
        if line.startswith("global_load_dwordx4"):
            run += 1
            best = max(best, run)
        elif line.startswith((".LBB", "s_cbranch")) or re.match(r"s_waitcnt .*vmcnt", line):
            run = 0
    assert best >= loads
