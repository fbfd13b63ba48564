"""The eigensolver at the edge between the host's form (up to 48 dimensions)
and the GPU's, by the same bounds as its other sizes."""
import pytest

from test_gpu_eigh import test_eigenvectors as eigenvectors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [12, 44, 48, 52])
def test_around_the_host_limit(m):
    eigenvectors(m)
