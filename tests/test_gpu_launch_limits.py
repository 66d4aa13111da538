"""Calls whose launch grid would hold more than 65,536 blocks along y."""
import numpy as np
import pytest

from tests.gpu_util import require_gpu, announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nf", [32 * 32768, 32 * 32768 + 1, 32 * 65536 + 33])
def test_assemble_of_many_shifts(nf):
    """x = z y: one complex product, off by sqrt(5) roundings of 1.1e-16 at most on
    either side."""
    torch = require_gpu()
    import paper_1212_3660_amd as P
    announce(f"assemble nf={nf}")
    rng = np.random.default_rng(1)
    n = 3
    Z = rng.standard_normal((1, n)) + 1j * rng.standard_normal((1, n))
    Y = rng.standard_normal((nf, 1)) + 1j * rng.standard_normal((nf, 1))
    X = torch.full((nf, n), float("nan"), dtype=torch.complex128, device="cuda")
    P.shk_assemble(n, 1, nf, torch.from_numpy(Z).cuda(), torch.from_numpy(Y).cuda(), X)
    assert np.all(np.abs(X.cpu().numpy() - Y * Z) <= 5e-16 * np.abs(Y * Z))
