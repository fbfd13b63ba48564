"""The repair joins each start node to its nearest reached node with a free
slot by exact distance, also where the kNN's candidate scores (split bf16)
cannot tell the candidates apart: points far from the origin whose distances
to more candidates than the short list holds differ by less than the scores'
error.  Integer points whose squared distances are exact in float32, so the
graph equals the float64 oracle's node for node."""
import numpy as np
import pytest
import torch

from oracle import graph as og

pytestmark = pytest.mark.gpu


def far_clusters(clusters, size, m, seed, offset=4000, top=4):
    """Clusters on an axis of their own, all equally far from each other but
    for small integers in the remaining coordinates."""
    rng = np.random.default_rng(seed)
    x = np.full((clusters, size, m), float(offset))
    x[:, :, clusters:] += rng.integers(0, top, size=(clusters, size, m - clusters))
    for c in range(clusters):
        x[c, :, c] += 700
    x = x.reshape(-1, m)
    return x[rng.permutation(len(x))].astype(np.float32)


@pytest.mark.parametrize("clusters,size,m,offset", [(14, 12, 36, 4000), (20, 16, 64, 8000), (12, 18, 132, 4000)])
def test_far_from_the_origin(clusters, size, m, offset):
    from paper_2206_11408_amd import api
    print(f"[gpu] graph repair: {clusters} clusters of {size} x {m} at {offset}", flush=True)
    x = far_clusters(clusters, size, m, clusters, offset)
    G, st = api.finger_build_graph(torch.as_tensor(x, device="cuda"), knn_k=4, max_degree=8, entry=3)
    O, ost = og.build(x, 4, 8, 3)
    assert ost["components_before_repair"] == clusters
    assert st["components_before_repair"] == clusters and st["edges_added"] == ost["edges_added"]
    np.testing.assert_array_equal(G.cpu().numpy(), O)


def test_ties_and_outliers():
    """Equal distances go to the smaller id; one point far out does not
    matter to the rest."""
    from paper_2206_11408_amd import api
    print("[gpu] graph repair: ties and an outlier", flush=True)
    x = far_clusters(10, 12, 24, 1, offset=0, top=1)
    x[7, -1] = 60_000.0
    G, st = api.finger_build_graph(torch.as_tensor(x, device="cuda"), knn_k=4, max_degree=8, entry=11)
    O, ost = og.build(x, 4, 8, 11)
    np.testing.assert_array_equal(G.cpu().numpy(), O)
    assert st["edges_added"] == ost["edges_added"]
