"""The passes of exact distances as compiled: all loads of a pass are issued
before the first wait on one of them."""
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

NEEDS_HIPCC = pytest.mark.skipif(not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)), reason="needs hipcc")


def runs_of_loads(tmp_path, kernel):
    """lengths of the runs of 16-byte loads with no branch and no wait between them"""
    src, out = tmp_path / "one.hip", tmp_path / "one.s"
    src.write_text(PROGRAM % kernel)
    subprocess.run([build.HIPCC, *build.FLAGS, "-w", "-I", build.CSRC, "-S", "--cuda-device-only", str(src), "-o", str(out)],
                   check=True, capture_output=True)
    runs = [0]
    for line in out.read_text().splitlines():
        line = line.strip()
        if line.startswith("global_load_dwordx4"):
            runs[-1] += 1
        elif line.startswith((".LBB", "s_cbranch")) or re.match(r"s_waitcnt .*vmcnt", line):
            runs.append(0)
    return runs


@NEEDS_HIPCC
@pytest.mark.parametrize("kernel,loads", [("k_search_few<FINGER_MODE_PLAIN, FINGER_CODE_F32, 32, 4, 0>", 32),
                                          ("k_search<FINGER_MODE_PLAIN, FINGER_CODE_F32, 64, 4, false, 0, true>", 32),
                                          ("k_search<FINGER_MODE_PLAIN, FINGER_CODE_F32, 64, 8, false, 0, true>", 32),
                                          ("k_search<FINGER_MODE_FINGER, FINGER_CODE_BF16, 64, 4, false, 8, true>", 32)])
def test_wide_pass_loads_together(tmp_path, kernel, loads):
    assert max(runs_of_loads(tmp_path, kernel)) >= loads


@NEEDS_HIPCC
@pytest.mark.parametrize("kernel,loads", [("k_search<3, FINGER_CODE_BF16, 64, 8, false, 0, false>", 8),
                                          ("k_search<FINGER_MODE_FINGER, FINGER_CODE_BF16, 64, 8, false, 0, true>", 32),
                                          ("k_search<FINGER_MODE_FINGER, FINGER_CODE_F32, 64, 8, false, 0, true>", 32)])
def test_masked_pass_loads_together(tmp_path, kernel, loads):
    # (once for vectors that the lanes cover exactly, once for any other)
    assert sum(r >= loads for r in runs_of_loads(tmp_path, kernel)) >= 2
