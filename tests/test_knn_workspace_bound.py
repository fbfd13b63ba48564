"""The exact kNN's workspace past its fixed part is a few bytes a point,
whatever the vectors' length (host arithmetic, no GPU)."""
import ctypes as C

import pytest

from paper_2206_11408_amd import _lib as L

GB = 1 << 30


def need(n, m, nq, k):
    nb = C.c_size_t(0)
    assert L.load().finger_exact_knn_workspace_size(n, m, nq, k, C.byref(nb)) == L.FINGER_OK
    return nb.value


@pytest.mark.parametrize("m", [4, 96, 960, 2048])
def test_workspace_is_bounded(m):
    for n, nq in ((1_000, 1), (1_000_000, 10_000), (50_000_000, 10_000), (200_000_000, 1_000_000)):
        for k, fixed in ((10, 2.2 * GB), (128, 3.2 * GB)):
            assert need(n, m, nq, k) <= fixed + 12 * n + 8 * nq
