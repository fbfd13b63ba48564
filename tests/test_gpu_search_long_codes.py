"""The per-lane screen (code rows longer than 256 bytes or of odd length): the
same bits whatever the call's size, the code requests and the launch, and the
exact distances of the returned points."""
import numpy as np
import pytest
import torch

import test_gpu_search_instances as instances
from paper_2206_11408_amd import api
from test_gpu_knn import IP, L2
from test_gpu_search_shapes import cuda, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("code", [0, 1, 2])
@pytest.mark.parametrize("m,rank,ef", [(128, 96, 70), (132, 96, 16), (256, 96, 70), (260, 128, 16), (300, 96, 70),
                                       (512, 96, 16), (516, 96, 70), (1028, 96, 16), (1028, 128, 70), (2048, 96, 16)])
def test_same_bits(m, rank, ef, code):
    instances.test_every_instance_agrees(m, rank, ef, code)


@pytest.mark.parametrize("metric", [L2, IP])
@pytest.mark.parametrize("m,rank", [(100, 96), (132, 128), (200, 96), (300, 128), (516, 128), (1028, 128), (1536, 96)])
def test_distances(m, rank, metric):
    """Integer points: sums below 2^24, exact in float32 in any order."""
    data, qs, G = workload(m)
    basis = np.linalg.qr(np.random.default_rng(1).standard_normal((m, m)))[0][:rank]
    tab = api.finger_build_tables(cuda(data), cuda(G), rank=rank, basis=basis, metric=metric)
    ids, dist, ctr = api.finger_search(tab, cuda(qs), k=5, ef=40, entry=3, mode=1)
    assert int(ctr[:, 2].sum()) > 0
    x, q = cuda(data).double()[ids.long()], cuda(qs).double()[:, None]
    true = -(x * q).sum(-1) if metric == IP else ((x - q) ** 2).sum(-1)
    assert torch.equal(dist.double(), true)
    assert bool((dist[:, 1:] >= dist[:, :-1]).all())
