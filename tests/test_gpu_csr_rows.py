"""Inner solves of a general sparse K whose rows are shorter, as long as and
longer than what the iteration holds ahead of its sums."""
import numpy as np
import pytest
import scipy.sparse as sp

from tests.gpu_util import announce, require_gpu, to_dev

pytestmark = pytest.mark.gpu


def _graph(n, reach, seed):
    """Symmetric, strictly diagonally dominant: row c couples to c +- 1..reach,
    except that every seventh run of five rows stands alone; with a reach, row 3
    couples to 40 more."""
    rng = np.random.default_rng(seed)
    rows, cols, vals = [np.zeros(0, int)], [np.zeros(0, int)], [np.zeros(0)]
    lone = (np.arange(n) // 5) % 7 == 6
    for d in range(1, reach + 1):
        c = np.arange(n - d)
        c = c[~lone[c] & ~lone[c + d]]
        rows.append(c); cols.append(c + d); vals.append(-rng.uniform(0.2, 1.0, c.size))
    far = np.arange(n // 2, n // 2 + (40 if reach else 0))
    far = far[~lone[far]]
    rows.append(np.full(far.size, 3)); cols.append(far); vals.append(-rng.uniform(0.2, 1.0, far.size))
    W = sp.coo_matrix((np.concatenate(vals), (np.concatenate(rows), np.concatenate(cols))), shape=(n, n)).tocsr()
    W = W + W.T
    return (W + sp.diags(0.3 - np.asarray(W.sum(axis=1)).ravel())).tocsr()


# Reach 0: rows of one entry; 2: at most five; 3: seven, past the six held; 9:
# nineteen.  The last two sizes, of 16 lanes, lie on the two sides of the number
# of wavefronts up to which rows are held ahead (131,072 items).
@pytest.mark.parametrize("n,reach,lanes", [(1, 0, 1), (257, 0, 2), (300, 2, 1), (511, 3, 1), (700, 9, 4),
                                           (8192, 3, 16), (8193, 3, 16)])
@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_rows_of_any_length(n, reach, lanes, prec):
    """The solution is judged by its residual.  K >= 0.3 and its largest
    eigenvalue is below 80, so the recurrence's residual strays from the true
    one by its * 80 / 0.3 * 2^-53 at most, far below eps: twice eps covers it.
    The complex64 path judges its last residual in FP64, by the rule itself."""
    torch = require_gpu()
    import paper_1212_3660_amd as P
    announce(f"csr rows n={n} reach={reach} lanes={lanes} prec={prec}")
    K = _graph(n, reach, n + reach)
    M = np.random.default_rng(n).uniform(0.5, 1.5, n)
    g = np.random.default_rng(n + 1)
    tau, eps = 0.4 + 0.7j, 1e-9
    v = to_dev((g.standard_normal((n, lanes)) + 1j * g.standard_normal((n, lanes))).ravel(), prec)
    z = torch.empty(n * lanes, dtype=torch.complex128, device="cuda")
    w = torch.empty_like(v)
    gp = P.Problem.csr(K.indptr, K.indices, K.data, M)
    P.shk_inner_solve(gp, tau, v, z, w, eps=eps, n_rhs=lanes, precond=P.SHK_PRECOND_JACOBI)
    v, z, w = (a.cpu().numpy().astype(np.complex128).reshape(n, lanes) for a in (v, z, w))
    res = v - (K @ z + tau * M[:, None] * z)
    assert np.all(np.linalg.norm(res, axis=0) <= 2 * eps * np.linalg.norm(v, axis=0))
    ref = M[:, None] * z
    assert np.all(np.abs(w - ref) <= (1e-14 if prec == "c128" else 2e-7) * np.abs(ref))
