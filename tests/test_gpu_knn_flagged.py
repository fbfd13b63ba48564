"""Rows that run out of candidate space (points ordered against the scan) are
searched point by point: every metric, short and long vectors, one and many
rows, equal distances, neighbours in the last partial slab of points."""
import math

import numpy as np
import pytest
import torch

from test_gpu_knn import ANGULAR, IP, L2, brute, run

pytestmark = pytest.mark.gpu


def against_the_scan(n, m, metric, late=0.7):
    """Points whose nearness to the queries grows along the scan's order, with
    groups of equal ones."""
    a = max(1, int(0.6180339887498949 * n))
    while math.gcd(a, n) != 1:
        a += 1
    p = np.arange(n, dtype=np.int64)
    near = np.where(p < late * n, 0, 1 + (p - int(late * n)) // 3 % 120).astype(np.float32)
    x = np.zeros((n, m), np.float32)
    if metric == IP:  # near: a large product with the queries' first axis
        x[(p * a) % n, 0] = near
    elif metric == ANGULAR:  # near: a small angle to it
        x[(p * a) % n, 0] = near
        x[:, 1] = 8
    else:
        x[(p * a) % n, 0] = 200 - near
    x[:, 2 % m] += (p % 3).astype(np.float32)
    return x


@pytest.mark.parametrize("metric", [L2, ANGULAR, IP])
@pytest.mark.parametrize("n,m,nq,k", [(20_000, 4, 3, 1), (20_001, 100, 70, 30), (30_257, 132, 5, 100), (9_000, 64, 300, 10)])
def test_flagged_rows(n, m, nq, k, metric):
    x = against_the_scan(n, m, metric)
    q = np.zeros((nq, m), np.float32)
    q[:, 0] = 1 + np.arange(nq) % 7
    x, q = torch.as_tensor(x).cuda(), torch.as_tensor(q).cuda()
    ids, dist = run(x, q, k, metric)
    e = [brute(x, q[s:s + 16], k, metric) for s in range(0, nq, 16)]
    ei, ed = torch.cat([v[0] for v in e]), torch.cat([v[1] for v in e])
    if metric == ANGULAR:  # rounded rows: equal up to the float32 sum's rounding
        tol = 4 * (m / 64 + 10) * 2.0 ** -24
        d = brute(x, q[:1], n, metric)  # (one query is a multiple of every other)
        at = torch.empty(n, dtype=torch.float64, device="cuda")
        at[d[0][0].long()] = d[1][0]
        assert float((dist.double() - ed).abs().max()) <= tol * float(ed.abs().max())
        assert float((at[ids.long()] - ed).abs().max()) <= tol * float(ed.abs().max())
        assert all(len(set(r)) == k for r in ids.cpu().tolist())
    else:
        assert torch.equal(dist.double(), ed) and torch.equal(ids, ei)
