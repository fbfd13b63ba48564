"""A phase of the kNN scan that appends nothing leaves every row's bound as it
is.  The nearest points of all queries come first in the scan's order, so the
later phases append nothing: the rows must not run out of space, and a short
list chosen by scores alone must not pass for a list of all points."""
import math

import numpy as np
import pytest
import torch

from oracle import graph as og

from paper_2206_11408_amd import api
from test_gpu_knn import L2, brute, run

pytestmark = pytest.mark.gpu


def scan_order(n):
    a = max(1, int(0.6180339887498949 * n))
    while math.gcd(a, n) != 1:
        a += 1
    return (np.arange(n, dtype=np.int64) * a) % n


def seconds(x, q, k):
    best = math.inf
    for _ in range(5):
        t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        t[0].record()
        run(x, q, k, L2)
        t[1].record()
        t[1].synchronize()
        best = min(best, t[0].elapsed_time(t[1]) / 1e3)
    return best


@pytest.mark.parametrize("n,m,nq,k", [(200_000, 64, 256, 17), (60_001, 260, 33, 17), (120_000, 96, 3000, 8)])
def test_rows_keep_their_bound(n, m, nq, k):
    """Within 5 times the time of the same points in a random order (searched
    point by point, each row takes more than 20 times as long)."""
    print(f"[gpu] empty phases: {nq} queries x {n} x {m}, k {k}", flush=True)
    rng = np.random.default_rng(n)
    near = 2 * (k + 16)
    x = 40 + rng.integers(0, 4, size=(n, m)).astype(np.float32)
    x[:near] -= 40
    q = rng.integers(0, 4, size=(nq, m)).astype(np.float32)
    early = np.empty_like(x)
    early[scan_order(n)] = x
    mixed = torch.as_tensor(x[rng.permutation(n)]).cuda()
    early, q = torch.as_tensor(early).cuda(), torch.as_tensor(q).cuda()
    ids, dist = run(early, q, k, L2)
    e = [brute(early, q[s:s + 16], k, L2) for s in range(0, min(nq, 64), 16)]
    ei, ed = torch.cat([v[0] for v in e]), torch.cat([v[1] for v in e])
    assert torch.equal(dist[:64].double(), ed) and torch.equal(ids[:64], ei)
    assert seconds(early, q, k) < 5 * seconds(mixed, q, k)


@pytest.mark.parametrize("m,offset", [(64, 4000), (132, 4000)])
def test_repair_does_not_trust_the_short_list(m, offset):
    """Components equally far from each other but for small integers, first in
    the scan's order, whose scores in split bf16 cannot be told apart; further
    ones on a line."""
    print(f"[gpu] graph repair after empty phases: {m} dims at {offset}", flush=True)
    rng = np.random.default_rng(m)
    near, far, size = 20, 40, 18
    x = np.full((near + far, size, m), float(offset))
    x[:, :, near + 1:] += rng.integers(0, 4, size=(near + far, size, m - near - 1))
    for c in range(near):
        x[c, :, c] += 700
    x[near:, :, near] += 1200 + 60 * np.arange(far)[:, None]
    x = x.reshape(-1, m)
    n, first = len(x), near * size
    order = scan_order(n)
    pts = np.empty((n, m), np.float32)
    pts[order[:first]] = x[rng.permutation(first)]
    pts[order[first:]] = x[first + rng.permutation(n - first)]
    entry = int(order[0])
    G, st = api.finger_build_graph(torch.as_tensor(pts, device="cuda"), knn_k=4, max_degree=8, entry=entry)
    O, ost = og.build(pts, 4, 8, entry)
    assert st["components_before_repair"] == ost["components_before_repair"] >= near
    np.testing.assert_array_equal(G.cpu().numpy(), O)
