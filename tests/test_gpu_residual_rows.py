"""True residual on both sides of the number of entries of X (3 Mi) from which
the kernel that marches rows takes it, with ragged rows, segments and planes,
against the oracle's operator.

Tolerance: FP64 sums of at most 6,000 terms, off by about sqrt(6000) roundings
of 1.1e-16 of sums without cancellation: 1e-12 relative."""
import numpy as np
import pytest

import synth
from oracle import Problem as OProblem
from tests.gpu_util import require_gpu, announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,nf", [((33, 65), 1466), ((33, 65), 1467), ((16, 64), 3072), ((17, 257), 721),
                                      ((2, 300), 5243), ((5, 17, 70), 528), ((5, 17, 70), 529), ((4, 16, 64), 769)])
def test_rows_of_a_march(shape, nf):
    torch = require_gpu()
    import paper_1212_3660_amd as P
    announce(f"residual rows {shape} nf={nf}")
    K = synth.cell_conductivity(shape, -11.5, 1.0, 5, cfg=95, idx=nf)
    op = OProblem.fv(K)
    gp = P.Problem.fv2d(K) if len(shape) == 2 else P.Problem.fv3d(K)
    rng = np.random.default_rng(nf)
    sig = 1j * rng.uniform(0.01, 1.0, nf)
    X = (rng.standard_normal((nf, op.n)) + 1j * rng.standard_normal((nf, op.n))) * 1e4
    b = rng.standard_normal(op.n) + 1j * rng.standard_normal(op.n)
    rel = P.shk_true_residual(gp, sig, torch.from_numpy(b).cuda(), torch.from_numpy(X).cuda())
    for j in range(nf):
        want = np.linalg.norm(b - op.apply(sig[j], X[j])) / np.linalg.norm(b)
        assert abs(rel[j] - want) <= 1e-12 * want
