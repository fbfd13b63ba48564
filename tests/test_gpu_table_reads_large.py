"""Table reads and exports at the size from which they go in slices."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [262_143, 262_144, 262_145, 300_007])
def test_codes_around_the_first_sliced_size(n):
    from paper_2206_11408_amd import _lib as L
    from paper_2206_11408_amd import api
    print(f"[gpu] table read n={n}", flush=True)
    m = r = 32  # codes: 256 bytes a node in float32 (degree 2), 64 MB at 262,144
    g = torch.Generator(device="cuda").manual_seed(n)
    data = torch.randn(n, m, generator=g, device="cuda")
    i = torch.arange(n, device="cuda")
    G = torch.stack([(i + 1) % n, (i + 7) % n], 1).to(torch.int32).contiguous()
    tab = api.finger_build_tables(data, G, rank=r, basis=np.eye(m))
    codes = tab.read(L.T_EDGE_CODES)
    x = data.double()
    for slot, step in ((0, 1), (1, 7)):
        d = x.roll(-step, 0)
        res = d - ((x * d).sum(1) / (x * x).sum(1))[:, None] * x
        want = (res / res.norm(dim=1, keepdim=True)).cpu().numpy()
        np.testing.assert_allclose(codes[:, slot], want, atol=1e-5)
    back = api.finger_tables_import(api.finger_tables_export(tab), data, G)
    assert np.array_equal(back.read(L.T_EDGE_CODES).view(np.uint32), codes.view(np.uint32))
