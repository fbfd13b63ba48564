"""Reachability repair of graphs whose paths are thousands of steps long."""
import numpy as np
import pytest
import torch

from oracle import graph as og

pytestmark = pytest.mark.gpu


def path(n, rng=None):
    """Unit steps that fill a box, rows and planes four apart (coordinates up
    to 250 and more planes: distances exact)."""
    P = np.zeros((n, 4), np.float32)
    x, y, z, dx, dy, c = 0, 0, 0, 1, 1, 0
    while c < n:
        steps = [(x + dx * i, y, z) for i in range(250)]
        x += 249 * dx
        if 0 <= y + 4 * dy <= 248:
            steps += [(x, y + dy * i, z) for i in (1, 2, 3)]
            y += 4 * dy
        else:
            steps += [(x, y, z + i) for i in (1, 2, 3)]
            z += 4
            dy = -dy
        dx = -dx
        take = min(len(steps), n - c)
        P[c:c + take, :3] = steps[:take]
        c += take
    return P


def build(x, entry):
    from paper_2206_11408_amd import api
    return api.finger_build_graph(torch.as_tensor(x, device="cuda"), knn_k=2, max_degree=4, entry=entry)


def test_several_long_paths():
    """Paths that the entry does not reach, in shuffled id order."""
    print("[gpu] several long paths", flush=True)
    rng = np.random.default_rng(5)
    one = path(700)
    x = np.concatenate([one + np.float32([0, 0, 0, 40 * c]) for c in range(4)])
    for order in (np.arange(len(x)), rng.permutation(len(x)), np.arange(len(x))[::-1]):
        y = np.ascontiguousarray(x[order])
        G, st = build(y, 900)
        O, ost = og.build(y, 2, 4, 900)
        np.testing.assert_array_equal(G.cpu().numpy(), O)
        assert st["components_before_repair"] == ost["components_before_repair"]


def test_time_grows_with_the_path():
    """Four times the path takes about four times as long (nine times where
    every node takes part in every sweep)."""
    print("[gpu] path of 300,000 points", flush=True)
    ms = []
    for n in (75_000, 300_000):
        _, st = build(path(n), n // 2)
        assert st["components_before_repair"] <= 2
        ms.append(st["ms_repair"])
    print(ms, flush=True)
    assert ms[1] < 6.0 * ms[0]
