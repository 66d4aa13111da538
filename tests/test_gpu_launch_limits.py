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


def test_gram_schmidt_against_many_columns():
    """One entry per column, all but the last column zero: w goes into that one."""
    torch = require_gpu()
    import paper_1212_3660_amd as P
    k = 4 * 65536 + 5
    announce(f"gram-schmidt k={k}")
    V = torch.zeros(k + 1, dtype=torch.complex128, device="cuda")
    V[k - 1] = 1.0
    w = torch.full((1,), 0.75 - 0.5j, dtype=torch.complex128, device="cuda")
    h = P.shk_orthogonalize(1, k, V, w)
    want = np.zeros(k + 1, dtype=np.complex128)
    want[k - 1] = 0.75 - 0.5j
    assert np.array_equal(h[0], want)
    assert complex(V[k].cpu()) == 0 and complex(w[0].cpu()) == 0
