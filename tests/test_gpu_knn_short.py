"""One short scan takes the split products without asking; the same query has
the same bits in a call large enough to ask."""
import pytest
import torch

from test_gpu_knn import ANGULAR, IP, L2, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("metric", [L2, ANGULAR, IP])
@pytest.mark.parametrize("points", ["integers", "floats"])
@pytest.mark.parametrize("n,m", [(100, 32), (1000, 96), (1024, 128), (513, 260)])
def test_small_and_large_calls_agree(n, m, points, metric):
    g = torch.Generator().manual_seed(n)
    x, q = torch.randn(n, m, generator=g) * 9, torch.randn(2049, m, generator=g) * 9
    if points == "integers":
        x, q = x.round(), q.round()
    x, q = x.cuda(), q.cuda()
    whole = run(x, q, 7, metric)
    for rows in (1, 130, 2048):
        part = run(x, q[:rows].contiguous(), 7, metric)
        assert torch.equal(part[0], whole[0][:rows]) and torch.equal(part[1], whole[1][:rows])
