"""The exact kNN where its bf16 planes hold a part of the points at a time,
and the graph build where device memory for the usual workspace is short."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def nearest(x, q, k):
    """(ids, d2) by (d2, id) in float64 (integer points: exact)."""
    xd, qd = x.double(), q.double()
    d = (qd * qd).sum(1)[:, None] + (xd * xd).sum(1)[None] - 2 * qd @ xd.T
    v, i = torch.sort(d, dim=1, stable=True)
    return i[:, :k].int(), v[:, :k]


@pytest.mark.parametrize("n,nq,top", [(131_072, 3, 4), (131_073, 130, 4), (300_001, 40, 300), (140_003, 65_700, 4)])
def test_points_in_windows(n, nq, top):
    """2,048 dimensions: 131,072 points fill the planes."""
    from paper_2206_11408_amd import api
    print(f"[gpu] exact_knn in windows n={n} nq={nq}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randint(0, top, (n, 2048), generator=g, device="cuda", dtype=torch.int32).float()
    q = torch.randint(0, top, (nq, 2048), generator=g, device="cuda", dtype=torch.int32).float()
    if top == 4:
        q[::3] = x[torch.randint(0, n, (nq,), generator=g, device="cuda")][::3] + (torch.arange(2048, device="cuda") % 700 == 0)
    ids, dist = api.finger_exact_knn(x, q, 10)
    for rows in (slice(0, 20), slice(nq - 20 if nq > 20 else 0, nq)):
        ei, ed = nearest(x, q[rows], 10)
        if top == 4:
            assert torch.equal(ids[rows], ei) and torch.equal(dist[rows].double(), ed)
        else:  # (beyond what float32 sums hold exactly)
            assert float((dist[rows].double() - ed).abs().max() / ed.max()) <= (2048 / 64 + 10) * 2.0 ** -24


@pytest.mark.parametrize("grouped", [False, True])
def test_graph_build_with_little_memory(grouped, monkeypatch):
    """Allocations of more than 90 MB fail: the kNN's usual workspace (hundreds
    of MB here, in the self-join and in the repair's search) is one."""
    from paper_2206_11408_amd import api
    print(f"[gpu] graph build with little memory grouped={grouped}", flush=True)
    rng = np.random.default_rng(9)
    centers = rng.integers(0, 250, size=(12_000, 1, 16))
    x = torch.as_tensor((centers + rng.integers(0, 3, size=(12_000, 5, 16))).reshape(-1, 16).astype(np.float32), device="cuda")

    def build():
        if grouped:
            off = np.concatenate([[0], np.arange(30_000, 60_001, 5)])  # one large group, then many of five
            return api.finger_build_graph_grouped(x, off, knn_k=2, max_degree=6, entry=3)
        return api.finger_build_graph(x, knn_k=2, max_degree=6, entry=3)

    G, st = build()
    assert st["components_before_repair"] > 8_000
    monkeypatch.setenv("FINGER_FAULT_INJECT", str("alloc:%d" % (90 << 20)))
    G2, st2 = build()
    assert torch.equal(G, G2) and st2["edges_added"] == st["edges_added"]
    monkeypatch.setenv("FINGER_FAULT_INJECT", "alloc:1000000")
    from paper_2206_11408_amd import _lib as L
    with pytest.raises(L.FingerError) as e:
        build()
    assert e.value.status == L.FINGER_ENOMEM if hasattr(e.value, "status") else "injected" in str(e.value)
