"""Every instance of the search beyond 128 dimensions, and those that request
codes with the adjacency row: the same query returns the same bits whatever
the call's size, the code requests and the launch, run after run."""
import numpy as np
import pytest
import torch

from test_gpu_search_shapes import cuda, workload

pytestmark = pytest.mark.gpu


def same(a, b, rows, what):
    for x, y in zip(a, b):
        assert torch.equal(x[torch.arange(y.shape[0], device=y.device) % rows], y), what


@pytest.mark.parametrize("code", [0, 1, 2])
@pytest.mark.parametrize("m,rank,ef", [(32, 32, 20), (64, 64, 20), (96, 64, 20), (128, 64, 70), (132, 64, 16), (192, 128, 70),
                                       (256, 32, 16), (300, 64, 16), (512, 64, 70), (516, 64, 16), (960, 16, 70),
                                       (1024, 64, 20), (1028, 64, 20), (2048, 64, 70)])
def test_every_instance_agrees(m, rank, ef, code):
    from paper_2206_11408_amd import api
    data, qs, G = workload(m)
    basis = np.linalg.qr(np.random.default_rng(1).standard_normal((m, m)))[0][:rank]
    tab = api.finger_build_tables(cuda(data), cuda(G), rank=rank, code_type=code, basis=basis)
    rows = len(qs)
    q = cuda(np.tile(qs, (240, 1)))

    def run(nq, **kw):
        print(f"[gpu] search m={m} code={code} nq={nq} {kw}", flush=True)
        return api.finger_search(tab, q[:nq], k=5, ef=ef, entry=3, **kw)

    cases = [(dict(mode=0), (1, 2048, 2049, 4097, 9300))] if code == 0 else []
    for layout in (0, 2):
        cases.append((dict(mode=1, screen_layout=layout), (1, 2048, 2049, 3073, 9300)))
    for base, sizes in cases:
        ref = run(rows, **base)
        assert base["mode"] == 0 or int(ref[2][:, 2].sum()) > 0
        for nq in sizes:
            same(ref, run(nq, **base), rows, (base, nq))
        variants = [dict(persistent=1), dict(waves_per_cu=3)]
        if base["mode"] == 1:
            variants += [dict(code_prefetch=1), dict(code_prefetch=-1), dict(code_prefetch=1, persistent=1)]
        for v in variants:
            for nq in (rows, 2500, 9300):
                for _ in range(2):
                    same(ref, run(nq, **base, **v), rows, (base, v, nq))
