"""Every width of the kNN scan (vectors padded to 32, 64, 96, 128 and longer),
with one product and with the split's three, against float64: the neighbours
as well as their distances."""
import numpy as np
import pytest
import torch

from test_gpu_knn import ANGULAR, IP, L2, brute, ints, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [28, 36, 64, 68, 92, 96, 100])
@pytest.mark.parametrize("n,nq,k", [(700, 130, 10), (6000, 40, 33)])
def test_integer_points(n, nq, k, m):
    x, q = ints(n, m, n + m), ints(nq, m, m)
    ids, dist = run(x, q, k)
    ei, ed = brute(x, q, k, L2)
    assert torch.equal(dist.double(), ed) and torch.equal(ids, ei)


@pytest.mark.parametrize("metric", [L2, ANGULAR, IP])
@pytest.mark.parametrize("m", [28, 36, 64, 68, 96, 132])
@pytest.mark.parametrize("n,nq,k", [(900, 70, 10), (7000, 33, 40)])
def test_continuous_points(n, nq, k, m, metric):
    g = torch.Generator().manual_seed(n + m)
    x, q = torch.randn(n, m, generator=g).cuda(), torch.randn(nq, m, generator=g).cuda()
    ids, dist = run(x, q, k, metric)
    ei, ed = brute(x, q, n, metric)  # every point, by (d, id)
    of = torch.empty(nq, n, dtype=torch.float64, device="cuda").scatter_(1, ei.long(), ed)
    got = of.gather(1, ids.long())  # float64 distances of the returned points
    # a distance is a float32 sum: (m / 64 + 10) roundings of its terms' size
    size = (q.norm(dim=1)[:, None] * x.norm(dim=1)[ids.long()]).double() if metric == IP else got
    tol = (m / 64 + 10) * 2.0 ** -24 * (4 if metric == ANGULAR else 1)
    assert bool(((dist.double() - got).abs() <= tol * size).all())
    # the k nearest: no returned point further than the k-th by more than that
    last = ed[:, k - 1:k]
    assert bool((got <= last + 2 * tol * (size if metric == IP else last)).all())
    assert all(len(set(r)) == k for r in ids.cpu().tolist())
    assert bool((dist[:, 1:] >= dist[:, :-1]).all())


@pytest.mark.parametrize("m", [516, 960])
def test_large_integers_with_near_ties(m):
    """Squared norms past 2^24: sums and scores are rounded.  Two hundred
    points almost equally far from each query; distances of what is returned
    are right, and none of the returned is beyond the k-th by more than the
    scores' rounding."""
    rng = np.random.default_rng(m)
    n, nq, k = 4000, 12, 10
    x = rng.integers(0, 256, size=(n, m)).astype(np.float32)
    q = rng.integers(0, 256, size=(nq, m)).astype(np.float32)
    for i in range(nq):
        for t in range(200):
            p = q[i].copy()
            j = rng.integers(0, m, size=40)
            p[j] += np.where(p[j] < 128, 1, -1) * (20 + (t % 5 == 0))
            x[i * 200 + t] = p
    x, q = torch.as_tensor(x).cuda(), torch.as_tensor(q).cuda()
    ids, dist = run(x, q, k)
    ei, ed = brute(x, q, n, L2)
    of = torch.empty(nq, n, dtype=torch.float64, device="cuda").scatter_(1, ei.long(), ed)
    got = of.gather(1, ids.long())
    assert torch.equal(dist.double(), got)  # (below 2^24: exact)
    # score rounding: 3 m additions and the norms, 2^-23 of |q|^2 + |x|^2 each
    norm = float((x.double() ** 2).sum(1).max())
    assert float((got - ed[:, :k]).max()) <= 4 * m * 2.0 ** -23 * norm
    assert all(len(set(r)) == k for r in ids.cpu().tolist())
