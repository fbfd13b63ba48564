"""The order of a search distance's sum, bit for bit: four terms of a piece in
the order x, y, z, w (y first at exactly 128, 512 and 2,048 dimensions, the
order that distances there have always had), a lane's pieces one after
another, then the lanes by a fixed tree."""
import ctypes
import ctypes.util

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

_fmaf = ctypes.CDLL(ctypes.util.find_library("m")).fmaf
_fmaf.restype = ctypes.c_float
_fmaf.argtypes = [ctypes.c_float] * 3


def fma(a, b, c):
    return np.float32(_fmaf(float(a), float(b), float(c)))


def distance(q, x, ip):
    m = len(q)
    lanes = 8 if m <= 128 else (32 if m <= 512 else 64)
    y_first = not ip and m in (128, 512, 2048)
    acc = [np.float32(0)] * lanes
    with np.errstate(all="ignore"):
        for j in range(m // 4):
            a, b = q[4 * j:4 * j + 4], x[4 * j:4 * j + 4]
            if ip:
                s = fma(a[3], b[3], fma(a[2], b[2], fma(a[1], b[1], a[0] * b[0])))
                acc[j % lanes] = np.float32(acc[j % lanes] - s)
                continue
            d = a - b
            s = fma(d[0], d[0], d[1] * d[1]) if y_first else fma(d[1], d[1], d[0] * d[0])
            s = fma(d[3], d[3], fma(d[2], d[2], s))
            acc[j % lanes] = np.float32(acc[j % lanes] + s)
        step = 1
        while len(acc) > 1:  # neighbours, pairs, quads, ...: the sums are commutative
            acc = [np.float32(acc[i] + acc[i + 1]) for i in range(0, len(acc), 2)]
    return acc[0]


@pytest.mark.parametrize("metric", [0, 2])
@pytest.mark.parametrize("m", [4, 32, 36, 64, 96, 100, 128, 132, 256, 300, 512, 516, 960, 1024, 1028, 2048])
def test_distance_bits(m, metric):
    from paper_2206_11408_amd import api
    print(f"[gpu] distance bits m={m} metric={metric}", flush=True)
    rng = np.random.default_rng(m)
    n, nq = 64, 3
    data = rng.standard_normal((n, m)).astype(np.float32)
    qs = rng.standard_normal((nq, m)).astype(np.float32)
    G = np.stack([(np.arange(n) + s) % n for s in (1, 5, 17, 30)], axis=1).astype(np.int32)
    tab = api.finger_build_tables(torch.as_tensor(data, device="cuda"), torch.as_tensor(G, device="cuda"), metric=metric)
    ids, dist, _ = api.finger_search(tab, torch.as_tensor(qs, device="cuda"), mode=0, k=8, ef=64, entry=0)
    ids, dist = ids.cpu().numpy(), dist.cpu().numpy()
    for i in range(nq):
        want = np.array([distance(qs[i], data[j], metric == 2) for j in ids[i]], dtype=np.float32)
        np.testing.assert_array_equal(dist[i].view(np.uint32), want.view(np.uint32))
